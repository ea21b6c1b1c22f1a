"""GPU parity of the key switch with more digits than its accumulators take uncut
(32), whole and two-pass, and with its digits spread over workgroups at the larger
N.  Oracle comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_n,l,batch,bits", [(6, 35, 2, 55), (9, 33, 1, 33), (9, 40, 1, 60), (13, 35, 4, 55), (13, 33, 4, 60),
                                                (15, 8, 1, 55), (16, 5, 1, 55), (16, 5, 1, 60)])
def test_relin_many_digits(gpu, log_n, l, batch, bits):
    import paper_2109_14704_amd as H
    print("case relin digits log_n=%d l=%d batch=%d bits=%d" % (log_n, l, batch, bits), flush=True)
    mods = primes(bits, log_n, l + 1)
    rng = np.random.default_rng(7 * log_n + l + bits)
    n = 1 << log_n
    c = words(rng, (batch, 3, l, n), mods[:l])
    ksk = words(rng, (l, 2, l + 1, n), mods)
    c[:, 2], ksk[:, :, :, n // 2:] = words(rng, (batch, l, n), mods[:l]), np.array(mods, dtype=np.uint64)[:, None] - 1
    got = H.relin(H.Tables(log_n, mods), dev(c, gpu), dev(ksk, gpu))
    assert np.array_equal(host(got), oracle.relin(c, ksk, mods))
