"""GPU parity of the tensor at N = 2^9 on both sides of its choice of words per lane
(1024 units), alone and grouped, all domain forms, moduli of every correction rule.
Oracle comparison, exact."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [255, 257])
@pytest.mark.parametrize("bits", [(33, 34, 55, 56), (60, 59, 58, 57)])
def test_tensor_words_per_lane(gpu, batch, bits):
    import paper_2109_14704_amd as H
    print("case tensor 2^9 units=%d bits=%s" % (batch * 4, bits), flush=True)
    log_n, n = 9, 1 << 9
    mods = [primes(b, log_n)[0] for b in bits]
    rng = np.random.default_rng(batch)
    c, d = (words(rng, (batch, 2, 4, n), mods) for _ in range(2))
    t = H.Tables(log_n, mods)
    fc, fd = (oracle.batch_ntt(x.reshape(2 * batch, 4, n), mods, +1).reshape(x.shape) for x in (c, d))
    want = oracle.batch_ct_tensor_coeff(c, d, mods)
    fwant = oracle.batch_ntt(want.reshape(3 * batch, 4, n), mods, +1).reshape(want.shape)
    for a, x, y in ((False, c, d), (True, fc, fd)):
        for b, w in ((False, want), (True, fwant)):
            xd, yd = dev(x, gpu), dev(y, gpu)
            assert np.array_equal(host(H.ct_tensor(t, xd, yd, in_ntt=a, out_ntt=b)), w), (a, b)
            out = torch.empty(w.shape, dtype=torch.int64, device=gpu)
            H.ct_tensor_grouped([(t, xd, yd, out)], in_ntt=a, out_ntt=b)
            assert np.array_equal(host(out), w), (a, b)
