"""GPU parity of the product at N = 2^13 on both sides of its choice between two
passes and whole transforms: units around half and whole generations of 256
CUs, two limbs among them.  Oracle comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,limbs", [(1, 1), (64, 2), (129, 1), (128, 2), (257, 1), (193, 2), (512, 1)])
def test_polymul_generations(gpu, batch, limbs):
    import paper_2109_14704_amd as H
    print("case polymul 2^13 units=%d" % (batch * limbs), flush=True)
    log_n, n = 13, 1 << 13
    mods = (primes(60, log_n) + primes(55, log_n))[:limbs]
    rng = np.random.default_rng(batch)
    x, y = (words(rng, (batch, limbs, n), mods) for _ in range(2))
    got = host(H.polymul(H.Tables(log_n, mods), dev(x, gpu), dev(y, gpu)))
    at = sorted({0, batch // 2, batch - 1, *range(0, batch, 16)})
    assert np.array_equal(got[at], oracle.batch_polymul(x[at], y[at], mods))
