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


def test_transforms_of_2_34_words(gpu, room):
    import paper_2109_14704_amd as H
    log_n, batch = 10, 1 << 24           # 128 GiB, 4 words per lane
    print("case transforms of 2^34 words", flush=True)
    room(128)
    mods = primes(55, log_n)
    at = [0, (1 << 22) - 1, 1 << 22, 3 << 22, batch - 1]
    x = words(np.random.default_rng(1), (len(at), 1, 1 << log_n), mods)
    d = torch.zeros((batch, 1, 1 << log_n), dtype=torch.int64, device=gpu)
    put(d, at, x, gpu)
    t = H.Tables(log_n, mods)
    H.ntt_fwd(t, d)
    assert np.array_equal(host(d[at]), oracle.batch_ntt(x, mods, +1))
    H.ntt_inv(t, d)
    assert np.array_equal(host(d[at]), x)
    assert zero_elsewhere(d, at)


def test_polymul_and_rescale_in_pieces(gpu, room):
    import paper_2109_14704_amd as H
    log_n, batch = 9, (1 << 22) + 5       # two limbs: more than 2^32 words an operand
    print("case polymul and rescale of more than 2^32 words", flush=True)
    room(100)
    mods = primes(55, log_n) + primes(58, log_n)
    rng = np.random.default_rng(2)
    at = [0, (1 << 22) - 1, 1 << 22, batch - 1]
    x, y = (words(rng, (len(at), 2, 1 << log_n), mods) for _ in range(2))
    a, b = (torch.zeros((batch, 2, 1 << log_n), dtype=torch.int64, device=gpu) for _ in range(2))
    put(a, at, x, gpu)
    put(b, at, y, gpu)
    t = H.Tables(log_n, mods)
    out = H.polymul(t, a, b)
    assert np.array_equal(host(out[at]), oracle.batch_polymul(x, y, mods))
    assert zero_elsewhere(out, at)
    del b, out
    out = H.rescale(t, a, ntt=True)
    assert np.array_equal(host(out[at]), oracle.batch_rescale_ntt(x, mods))
    assert zero_elsewhere(out, at)


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
