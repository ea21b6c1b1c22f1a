"""An allocation failure is reported once: the call after it succeeds, in the
library and in the caller's own use of the GPU."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


def test_no_error_left_behind_after_enomem(gpu):
    """Operands of 4 GiB whose workspace of 8 GiB cannot be had on a device with 4
    GiB left.  What runs next must not see that failure: a product that needs
    less, and a kernel of the caller's."""
    import paper_2109_14704_amd as H
    print("case after ENOMEM", flush=True)
    log_n, n, batch = 14, 1 << 14, 1 << 15
    mods = primes(55, log_n)
    rng = np.random.default_rng(5)
    x, y = words(rng, (1, 1, n), mods), words(rng, (1, 1, n), mods)
    t = H.Tables(log_n, mods)
    a, b, out = (torch.zeros((batch, 1, n), dtype=torch.int64, device=gpu) for _ in range(3))
    a[:1], b[:1] = dev(x, gpu), dev(y, gpu)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    H.pool_trim()
    filler = torch.empty(torch.cuda.mem_get_info()[0] - (4 << 30), dtype=torch.uint8, device=gpu)
    try:
        with pytest.raises(H.HenttError, match=r"\[-3\]"):
            H.polymul(t, a, b, out=out)
        got = H.polymul(t, a[:1], b[:1], out=out[:1])
        assert int((torch.ones(8, device=gpu) * 2).sum()) == 16
        assert np.array_equal(host(got), oracle.batch_polymul(x, y, mods))
    finally:
        del filler, a, b, out
        torch.cuda.empty_cache()
