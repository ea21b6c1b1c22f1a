"""GPU parity of the rescale on both sides of its choice between one column pass
(small calls: every workgroup takes the last limb's inverse column stages as well) and two,
4096 waves, at every two-pass N, moduli of 33, 55 and 60 bits.  Oracle
comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


# units (batch x remaining limbs) at and above 4096 waves: 256 at 2^14, 128, 64, 32 at 2^17
@pytest.mark.parametrize("log_n,batch,limbs", [(14, 128, 2), (14, 129, 2), (15, 64, 2), (15, 65, 2), (16, 32, 2), (16, 33, 2),
                                               (17, 16, 2), (17, 11, 3)])
@pytest.mark.parametrize("last", [33, 55, 60])
def test_rescale_column_passes(gpu, log_n, batch, limbs, last):
    import paper_2109_14704_amd as H
    print("case rescale columns log_n=%d units=%d last=%d" % (log_n, batch * limbs, last), flush=True)
    mods = [primes(b, log_n)[0] for b in (60, 33, 55) if b != last][:limbs]
    mods += primes(50, log_n)[:limbs - len(mods)] + primes(last, log_n)
    rng = np.random.default_rng(10 * log_n + last)
    n, some = 1 << log_n, sorted({0, 1, batch // 2, batch - 1})
    x = np.zeros((batch, limbs + 1, n), dtype=np.uint64)
    x[some] = words(rng, (len(some), limbs + 1, n), mods)
    got = host(H.rescale(H.Tables(log_n, mods), dev(x, gpu), ntt=True))
    assert np.array_equal(got[some], oracle.batch_rescale_ntt(x[some], mods))
    rest = np.ones(batch, dtype=bool)
    rest[some] = False
    assert not got[rest].any()   # round(0 / q) = 0
