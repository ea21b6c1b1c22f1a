"""Calls whose launches would reach 2^32 work-items in one piece (the HIP
limit): they run as several.  Zero operands apart from a few batch entries on
both sides of the pieces' borders, which the oracle checks; the rest stays zero."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.fixture
def room():
    """Skips where the GPU has less free memory than the case needs."""
    def need(gib):
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < (gib + 8) << 30:
            pytest.skip("needs %d GiB of free GPU memory" % gib)
    yield need
    torch.cuda.empty_cache()


def put(t, at, x, gpu):
    t[at] = dev(x, gpu)


def zero_elsewhere(t, at):
    """Every entry of t outside `at` is zero, counted in pieces."""
    for i in at:
        t[i] = 0
    flat = t.view(-1)
    return all(int(torch.count_nonzero(flat[i:i + (1 << 30)])) == 0 for i in range(0, flat.numel(), 1 << 30))


def test_matmul_of_2_32_coefficients(gpu, room):
    import paper_2109_14704_amd as H
    log_n, m = 13, 1 << 19                # A 64 GiB, C 96 GiB
    n = 1 << log_n
    print("case matmul of 2^19 rows", flush=True)
    room(160)
    mods = primes(55, log_n)
    rng = np.random.default_rng(3)
    at = [0, (1 << 18) - 1, 1 << 18, m - 1]
    a = words(rng, (len(at), 1, 2, 1, n), mods)
    b = words(rng, (1, 1, 2, 1, n), mods)
    A = torch.zeros((m, 1, 2, 1, n), dtype=torch.int64, device=gpu)
    C = torch.zeros((m, 1, 3, 1, n), dtype=torch.int64, device=gpu)
    put(A, at, a, gpu)
    t = H.Tables(log_n, mods)
    H.ct_matmul(t, A, dev(b, gpu), C)
    want = oracle.ct_matmul(a, b, np.zeros((len(at), 1, 3, 1, n), dtype=np.uint64), mods)
    assert np.array_equal(host(C[at]), want)
    del A
    assert zero_elsewhere(C, at)
