"""Calls that only take more workspace to be faster run without it: the product at N =
2^13, captured with no buffer in the pool and where the device has no room for one;
the key switch of a small batch, captured with a buffer that holds all but its
partial sums."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu
LOG_N, N = 13, 1 << 13


def test_polymul_captured_without_a_warm_pool(gpu):
    import paper_2109_14704_amd as H
    print("case polymul 2^13 captured, empty pool", flush=True)
    mods = primes(60, LOG_N) + primes(50, LOG_N)
    rng = np.random.default_rng(13)
    t = H.Tables(LOG_N, mods)
    x, y = words(rng, (3, 2, N), mods), words(rng, (3, 2, N), mods)
    a, b = dev(x, gpu), dev(y, gpu)
    out = torch.zeros_like(a)
    torch.cuda.synchronize()
    H.pool_trim()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        H.polymul(t, a, b, out=out)
    for _ in range(3):
        x = words(rng, (3, 2, N), mods)
        a.copy_(dev(x, gpu))
        g.replay()
        torch.cuda.synchronize()
        want = oracle.batch_polymul(x, y, mods)
        assert np.array_equal(host(out), want)
        assert np.array_equal(host(H.polymul(t, a, b)), want)   # eager, between the replays


def test_polymul_without_room_for_the_workspace(gpu):
    import paper_2109_14704_amd as H
    print("case polymul 2^13, no room", flush=True)
    batch = (1 << 16) + 8                 # 4 GiB an operand, 8 GiB of workspace; no whole generations of units
    mods = primes(55, LOG_N)
    t = H.Tables(LOG_N, mods)
    at = [0, 777, batch - 1]
    rng = np.random.default_rng(14)
    x, y = words(rng, (len(at), 1, N), mods), words(rng, (len(at), 1, N), mods)
    a, b, out = (torch.zeros((batch, 1, N), dtype=torch.int64, device=gpu) for _ in range(3))
    a[at], b[at] = dev(x, gpu), dev(y, gpu)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    H.pool_trim()
    filler = torch.empty(torch.cuda.mem_get_info()[0] - (4 << 30), dtype=torch.uint8, device=gpu)
    try:
        H.polymul(t, a, b, out=out)
        assert np.array_equal(host(out[at]), oracle.batch_polymul(x, y, mods))
        assert H.pool_bytes() < 8 << 30
    finally:
        del filler, a, b, out
        torch.cuda.empty_cache()


def test_relin_captured_with_room_for_all_but_the_partial_sums(gpu):
    import paper_2109_14704_amd as H
    print("case relin 2^13 captured, pool short of the partial sums", flush=True)
    l = 8
    mods = primes(55, LOG_N, l + 1)
    rng = np.random.default_rng(15)
    t = H.Tables(LOG_N, mods)
    c, ksk = words(rng, (1, 3, l, N), mods[:l]), words(rng, (l, 2, l + 1, N), mods)
    cd, kd = dev(c, gpu), dev(ksk, gpu)
    out = H.relin(t, cd, kd)              # the level's constants
    big = H.Tables(14, primes(55, 14))
    a = torch.zeros((30, 1, 2 * N), dtype=torch.int64, device=gpu)
    o = torch.empty_like(a)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.pool_trim()
    # the pool's buffers for this stream: 2 N words for the rescale inside, 120 N for the key
    # switch, which needs 98 N and 72 N more for partial sums of 4
    H.rescale(t.view(2), torch.zeros((2, 2, N), dtype=torch.int64, device=gpu), ntt=True, stream=s)
    H.polymul(big, a, a, out=o, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        H.relin(t, cd, kd, out=out)
    for _ in range(3):
        c = words(rng, (1, 3, l, N), mods[:l])
        cd.copy_(dev(c, gpu))
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        want = oracle.relin(c, ksk, mods)
        assert np.array_equal(host(out), want)
        assert np.array_equal(host(H.relin(t, cd, kd)), want)
