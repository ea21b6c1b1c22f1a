"""An allocation failure is reported once: the call after it succeeds, in the
library and in the caller's own use of the GPU."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


def test_no_error_left_behind_after_enomem(gpu):
    """A workspace of 2^49 bytes cannot be had (nothing is enqueued, the pointers
    are not read).  What runs next must not see that failure: a small product by
    the library, and a kernel of the caller's."""
    import paper_2109_14704_amd as H
    print("case after ENOMEM", flush=True)
    log_n, n = 14, 1 << 14
    mods = primes(55, log_n)
    rng = np.random.default_rng(5)
    x, y = words(rng, (1, 1, n), mods), words(rng, (1, 1, n), mods)
    t, a, b = H.Tables(log_n, mods), dev(x, gpu), dev(y, gpu)
    H.polymul(t, a, b)   # this thread's workspace for what follows
    far = ctypes.c_void_p(1 << 54)   # no overlap with a and b: the first check to fail is the allocation
    rc = H.lib().hentt_polymul(t.handle, ctypes.c_void_p(a.data_ptr()), ctypes.c_void_p(b.data_ptr()), far,
                               (1 << 31) - 1, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == -3                  # HENTT_ENOMEM
    assert np.array_equal(host(H.polymul(t, a, b)), oracle.batch_polymul(x, y, mods))
    assert int((torch.ones(8, device=gpu) * 2).sum()) == 16
