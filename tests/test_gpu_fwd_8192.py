"""GPU parity of the forward transform at N = 2^13 on both sides of its choice of
words per lane (more than two units per CU of 256), ragged batches, moduli of every
correction rule.  Oracle comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [128, 129, 171])
@pytest.mark.parametrize("bits", [(33, 34, 55, 56), (60, 59, 58, 57)])
def test_fwd_words_per_lane(gpu, batch, bits):
    import paper_2109_14704_amd as H
    print("case fwd 2^13 units=%d bits=%s" % (batch * 4, bits), flush=True)
    log_n, n = 13, 1 << 13
    mods = [primes(b, log_n)[0] for b in bits]
    x = words(np.random.default_rng(batch), (batch, 4, n), mods)
    got = host(H.ntt_fwd(H.Tables(log_n, mods), dev(x, gpu)))
    assert np.array_equal(got, oracle.batch_ntt(x, mods, +1))
