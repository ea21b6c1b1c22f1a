"""GPU parity of the products of two variables at the edges of their rules: moduli
on both sides of 33/34 and 55/56 bits and at 60, words at q - 1, and a key
switch over more digits than its accumulators take without a cut (32), with whole
and with two-pass transforms, its digits in one workgroup and spread.  Oracle
comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, gpu, host, primes, words  # noqa: F401

pytestmark = pytest.mark.gpu

BITS = [33, 34, 55, 56, 60]


@pytest.mark.parametrize("log_n,batch", [(8, 1), (13, 1), (13, 9)])
def test_key_switch_over_many_digits(gpu, log_n, batch):  # noqa: F811
    import paper_2109_14704_amd as H
    l, n = 34, 1 << log_n
    mods = []
    for bits in BITS:
        mods += primes(bits, log_n, 7)
    print("case many digits log_n=%d batch=%d" % (log_n, batch), flush=True)
    rng = np.random.default_rng(log_n + batch)
    c = words(rng, (batch, 3, l, n), mods[:l])
    ksk = words(rng, (l, 2, l + 1, n), mods)
    got = host(H.relin(H.Tables(log_n, mods), dev(c, gpu), dev(ksk, gpu)))
    for b in {0, batch - 1}:
        assert np.array_equal(got[b:b + 1], oracle.relin(c[b:b + 1], ksk, mods)), b


@pytest.mark.parametrize("log_n", [9, 12, 14, 16])
def test_products_at_the_modulus_rules(gpu, log_n):  # noqa: F811
    import paper_2109_14704_amd as H
    n, mods = 1 << log_n, [primes(b, log_n)[0] for b in BITS]
    print("case products log_n=%d" % log_n, flush=True)
    rng = np.random.default_rng(log_n)
    a, b = (words(rng, (1, len(mods), n), mods) for _ in range(2))
    t = H.Tables(log_n, mods)
    assert np.array_equal(host(H.polymul(t, dev(a, gpu), dev(b, gpu))), oracle.batch_polymul(a, b, mods))
    c, d = (words(rng, (1, 2, len(mods), n), mods) for _ in range(2))
    assert np.array_equal(host(H.ct_tensor(t, dev(c, gpu), dev(d, gpu))), oracle.batch_ct_tensor_coeff(c, d, mods))
