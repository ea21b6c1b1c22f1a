"""Device memory of a table handle, and the (W, W') tables that
hentt_tables_device_ptrs hands out."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


class DeviceWords:
    """uint64 words at a device address, for torch.as_tensor."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i8", "data": (ptr, False), "version": 3}


def read(ptr, n, gpu):
    return host(torch.as_tensor(DeviceWords(ptr, n), device=gpu).clone())


def test_footprint(gpu):
    """32 N bytes per limb; 16 MiB are left for constants and the allocator's grain."""
    import paper_2109_14704_amd as H
    print("case table footprint", flush=True)
    log_n, limbs = 17, 24
    mods = primes(55, log_n, limbs)
    H.Tables(6, primes(55, 6)).close()   # the library's code and static memory are loaded on first use
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    t = H.Tables(log_n, mods)
    used = before - torch.cuda.mem_get_info()[0]
    assert used <= (32 * limbs << log_n) + (16 << 20), used
    t.close()


@pytest.mark.parametrize("log_n", [6, 11])
def test_device_ptrs(gpu, log_n):
    """Both tables of every limb, from a table and from a view, before and after other calls."""
    import paper_2109_14704_amd as H
    print("case device_ptrs log_n=%d" % log_n, flush=True)
    mods = primes(40, log_n) + primes(60, log_n)
    n, L = 1 << log_n, 2
    t = H.Tables(log_n, mods)
    x = words(np.random.default_rng(3), (2, L, n), mods)
    assert np.array_equal(host(H.ntt_fwd(t, dev(x, gpu))), oracle.batch_ntt(x, mods, +1))
    fwd, inv, rec = t.device_ptrs()
    assert t.view(1).device_ptrs() == (fwd, inv, rec) == t.device_ptrs()
    assert inv == fwd + 16 * n
    assert read(rec, 12 * L, gpu)[::12].tolist() == mods
    pairs = read(fwd, L * 4 * n, gpu).reshape(L, 2, n, 2)
    for l, q in enumerate(mods):
        p = oracle.psi(q, log_n)
        for d, root in enumerate((p, oracle.invmod(p, q))):
            w = [oracle.powmod(root, oracle.bitrev(k, log_n), q) for k in range(n)]
            assert pairs[l, d, :, 0].tolist() == w
            assert pairs[l, d, :, 1].tolist() == [(v << 64) // q for v in w]
    v = H.ntt_fwd_variant(t, dev(x, gpu), H.VARIANT_NAIVE)
    assert np.array_equal(host(v), oracle.batch_ntt(x, mods, +1))


def test_pairs_made_during_a_capture(gpu):
    """A ladder variant captured as the first thing that needs the pairs."""
    import paper_2109_14704_amd as H
    print("case pairs made during a capture", flush=True)
    log_n = 10
    mods = primes(55, log_n)
    x = words(np.random.default_rng(4), (2, 1, 1 << log_n), mods)
    t, d = H.Tables(log_n, mods), dev(x, gpu)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        H.ntt_fwd_variant(t, d, H.VARIANT_NAIVE)
    want = x
    for _ in range(3):
        want = oracle.batch_ntt(want, mods, +1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(d), want)
