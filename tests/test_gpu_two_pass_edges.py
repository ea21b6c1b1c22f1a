"""GPU parity of the two-pass kernels at their edges: every size at which the
column stages or the words per lane change, moduli on both sides of each
correction rule (33/34, 47/48, 55/56 bits, 60 bits), single and ragged units,
words at q - 1, and operands whose address is a multiple of 8 but not of 16
bytes.  Oracle comparison, exact."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def primes(bits, log_n, count=1):
    m, out = 2 << log_n, []
    q = ((1 << bits) - 1) // m * m + 1
    while len(out) < count:
        if q < (1 << bits) and oracle.is_prime(q):
            out.append(q)
        q -= m
    assert all(v.bit_length() == bits for v in out)
    return out


def words(rng, shape, mods):
    """Uniform residues, with runs of q - 1 and of 0."""
    x = np.empty(shape, dtype=np.uint64)
    for l, q in enumerate(mods):
        x[..., l, :] = rng.integers(0, q, size=shape[:-2] + shape[-1:], dtype=np.uint64)
        x[..., l, : shape[-1] // 4] = q - 1
        x[..., l, shape[-1] // 4: shape[-1] // 4 + 3] = 0
    return x


def dev(a, gpu, offset=0):
    """a's words on the GPU, `offset` words past a 512-byte boundary."""
    flat = torch.empty(a.size + offset, dtype=torch.int64, device=gpu)[offset:]
    flat.copy_(torch.from_numpy(a.reshape(-1).view(np.int64)))
    return flat.view(a.shape)


def host(t):
    return t.cpu().numpy().view(np.uint64)


SIZES = [(6, 26), (10, 34), (11, 33), (12, 47), (13, 48), (14, 55), (14, 56), (15, 60), (16, 59), (17, 55), (17, 60)]


@pytest.mark.parametrize("log_n,bits", SIZES)
@pytest.mark.parametrize("offset", [0, 1])
def test_transforms_products_rescale(gpu, log_n, bits, offset):
    import paper_2109_14704_amd as H
    print("case two-pass edges log_n=%d bits=%d offset=%d" % (log_n, bits, offset), flush=True)
    mods = primes(bits, log_n) + primes(55, log_n)[:1] + primes(50, log_n)
    mods = mods if len(set(mods)) == 3 else primes(bits, log_n, 3)
    rng = np.random.default_rng(100 * log_n + bits + offset)
    n, L, batch = 1 << log_n, 3, 1 if log_n > 14 else 3
    t = H.Tables(log_n, mods)
    x = words(rng, (batch, L, n), mods)
    d = dev(x, gpu)
    fwd = oracle.batch_ntt(x, mods, +1)
    assert np.array_equal(host(H.ntt_fwd(t, d)), fwd)
    assert np.array_equal(host(H.ntt_inv(t, d)), x)
    y = words(rng, (batch, L, n), mods)
    assert np.array_equal(host(H.polymul(t, dev(x, gpu, offset), dev(y, gpu, offset))), oracle.batch_polymul(x, y, mods))
    assert np.array_equal(host(H.rescale(t, dev(fwd, gpu, offset), ntt=True)), oracle.batch_rescale_ntt(fwd, mods))
    if log_n <= 15:
        c, e = words(rng, (batch, 2, L, n), mods), words(rng, (batch, 2, L, n), mods)
        want = oracle.batch_ct_tensor_coeff(c, e, mods)
        assert np.array_equal(host(H.ct_tensor(t, dev(c, gpu, offset), dev(e, gpu, offset))), want)
        out = torch.empty(want.shape, dtype=torch.int64, device=gpu)
        H.ct_tensor_grouped([(t, dev(c, gpu, offset), dev(e, gpu, offset), out)])
        assert np.array_equal(host(out), want)


@pytest.mark.parametrize("log_n,bits", [(12, 33), (13, 34), (14, 56), (15, 60), (16, 55)])
@pytest.mark.parametrize("offset", [0, 1])
def test_relin(gpu, log_n, bits, offset):
    import paper_2109_14704_amd as H
    print("case relin edges log_n=%d bits=%d offset=%d" % (log_n, bits, offset), flush=True)
    mods = primes(bits, log_n, 2) + primes(54, log_n)
    rng = np.random.default_rng(31 * log_n + bits + offset)
    n, l, batch = 1 << log_n, 2, 2
    c = words(rng, (batch, 3, l, n), mods[:l])
    ksk = words(rng, (l, 2, l + 1, n), mods)
    got = H.relin(H.Tables(log_n, mods), dev(c, gpu, offset), dev(ksk, gpu, offset))
    assert np.array_equal(host(got), oracle.relin(c, ksk, mods))


@pytest.mark.parametrize("l,batch,log_n", [(4, 1, 13), (5, 2, 13), (9, 1, 13), (8, 1, 14)])
def test_relin_digits_spread_over_workgroups(gpu, l, batch, log_n):
    """Small batches of four and more digits: partial sums of 2 to 4 workgroups
    per block, even and uneven digit runs, moduli of 33 to 60 bits."""
    import paper_2109_14704_amd as H
    print("case relin digit splits l=%d batch=%d log_n=%d" % (l, batch, log_n), flush=True)
    bits = [60, 55, 56, 33, 34, 50, 58, 47, 54, 59][:l + 1]
    mods = [primes(b, log_n)[0] for b in bits]
    rng = np.random.default_rng(77 * l + batch)
    n = 1 << log_n
    c = words(rng, (batch, 3, l, n), mods[:l])
    ksk = words(rng, (l, 2, l + 1, n), mods)
    got = H.relin(H.Tables(log_n, mods), dev(c, gpu), dev(ksk, gpu))
    assert np.array_equal(host(got), oracle.relin(c, ksk, mods))
