"""Performance cases of the library's public entry points.

Each case is one pass of work that a program using this package does, with the
shapes of the repository's own workloads (workloads/, bench.py, serve.py) and
generic ones between them.  All words are 64-bit residues below their limb's
modulus, drawn uniformly; the moduli are the repository's stored chains
(tests/golden/moduli.json), at the sizes each chain supports:

  plain4096   one 50-bit prime              N <= 2^12
  ckks_level  16 primes of 50 to 60 bits    N <= 2^15
  ct_tensor   24 primes of 55 bits          N <= 2^16
  uneven      32 primes of 50 to 60 bits    N <= 2^17

A case names its operation ("op"), chain, log_n, limbs and batch:

  ntt_fwd       a new batch is copied into the program's buffer and transformed in place
  mul_plain     NTT-domain batch times NTT-domain plaintext, then the inverse transform
  polymul       fused negacyclic products of coefficient-domain batches
  ct_tensor     fused ciphertext tensor, coefficient domain in and out
  rescale       RS in the NTT domain
  mul_relin_rs  the paper's MulLinRS routine: tensor, relinearization, rescale (NTT domain)
  ct_matmul     C = A B on ciphertext matrices (NTT domain), C cleared first
  batch         uneven batch through a captured BatchPlan, forward (+1) or inverse (-1)
  grouped       one serving step: requests of mixed N and level in one grouped tensor call
"""
import functools
import random

import numpy as np
import torch

import paper_2109_14704_amd as H
import workloads

_MAX_LOG = {"plain4096": 12, "ckks_level": 15, "ct_tensor": 16, "uneven": 17}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: one product of two polynomials of 4096 coefficients (bench.py's plain4096)
        {"name": "polymul_4096_one", "op": "polymul", "chain": "plain4096", "log_n": 12, "limbs": 1, "batch": 1},
        # the paper's routine unbatched, N = 2^15 and 8 primes: latency of ten dependent launches
        {"name": "mul_relin_rs_2^15_x1", "op": "mul_relin_rs", "chain": "ct_tensor", "log_n": 15, "limbs": 8, "batch": 1},
        # the same routine over a batch of 32 ciphertexts
        {"name": "mul_relin_rs_2^15_x32", "op": "mul_relin_rs", "chain": "ct_tensor", "log_n": 15, "limbs": 8, "batch": 32},
        # an odd batch at a ragged level, small N: ciphertext times plaintext and back to coefficients
        {"name": "mul_plain_2^13_x37", "op": "mul_plain", "chain": "ckks_level", "log_n": 13, "limbs": 11, "batch": 37},
        # element-wise encrypted matrix product of 8K-coefficient polynomials (section IV-E shape 10 x 9 x 8)
        {"name": "ct_matmul_10x9x8", "op": "ct_matmul", "chain": "ct_tensor", "log_n": 13, "limbs": 4, "batch": 10, "n": 9, "k": 8},
        # one serving step: requests of N = 2^14 .. 2^16 at levels 4 .. 24
        {"name": "grouped_24", "op": "grouped", "chain": "ct_tensor", "log_n": 0, "limbs": 24, "batch": 24, "jobs_seed": 1},
        # the paper's transform benchmark at a quarter of its batch: [256][8][2^15] forward
        {"name": "ntt_fwd_2^15_x256", "op": "ntt_fwd", "chain": "ct_tensor", "log_n": 15, "limbs": 8, "batch": 256},
        # the CKKS-level batch: 128 polynomials per operand, 16 primes of 50 to 60 bits
        {"name": "polymul_2^15_x128", "op": "polymul", "chain": "ckks_level", "log_n": 15, "limbs": 16, "batch": 128},
        # rescale of 32 ciphertexts at the top of the 24-prime chain
        {"name": "rescale_2^16_x64", "op": "rescale", "chain": "ct_tensor", "log_n": 16, "limbs": 24, "batch": 64},
        # ciphertext products: 32 pairs, N = 2^16, 24 primes
        {"name": "ct_tensor_2^16_x32", "op": "ct_tensor", "chain": "ct_tensor", "log_n": 16, "limbs": 24, "batch": 32},
        # the uneven batch: 512 polynomials, N = 2^12 .. 2^17, 1 to 32 limbs, each direction
        {"name": "batch_fwd_512", "op": "batch", "chain": "uneven", "log_n": 0, "limbs": 32, "batch": 512, "dir": 1, "jobs_seed": 0},
        {"name": "batch_inv_512", "op": "batch", "chain": "uneven", "log_n": 0, "limbs": 32, "batch": 512, "dir": -1, "jobs_seed": 0},
    ]


def _log_uniform(rng, lo, hi):
    """An integer in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(2 ** rng.uniform(np.log2(lo), np.log2(hi + 0.49))))))


def draw(rng):
    """Another case of the same ranges: any operation, N from 2^6, odd batches and levels among them."""
    op = rng.choice(["ntt_fwd", "mul_plain", "polymul", "ct_tensor", "rescale", "mul_relin_rs", "ct_matmul", "batch",
                     "grouped"])
    if op == "batch":
        return {"op": op, "chain": "uneven", "log_n": 0, "limbs": rng.randint(4, 32), "batch": _log_uniform(rng, 3, 400),
                "dir": rng.choice([1, -1]), "jobs_seed": rng.randint(2, 10 ** 6)}
    if op == "grouped":
        return {"op": op, "chain": "ct_tensor", "log_n": 0, "limbs": rng.randint(4, 24), "batch": _log_uniform(rng, 1, 48),
                "jobs_seed": rng.randint(2, 10 ** 6)}
    # the sizes of real parameter sets most often, the small ones too
    log_n = rng.choice([12, 13, 14, 15, 16, 17, rng.randint(6, 17)])
    chain = rng.choice([c for c in _MAX_LOG if _MAX_LOG[c] >= log_n])
    top = len(workloads.moduli(chain)) - (1 if op == "mul_relin_rs" else 0)
    if top < 2:
        chain = "ckks_level" if log_n <= 15 else "uneven"
        top = 15
    if op == "mul_relin_rs":
        top = min(top, 12)
    limbs = rng.randint(2, top)
    case = {"op": op, "chain": chain, "log_n": log_n, "limbs": limbs, "batch": 1}
    if op == "ct_matmul":
        case.update(batch=rng.randint(1, 10), n=rng.randint(1, 9), k=rng.randint(1, 8))
        while case["log_n"] > 13 or case["chain"] == "plain4096":
            case.update(log_n=rng.randint(10, 13), chain="ct_tensor", limbs=rng.randint(1, 4))
        case["limbs"] = min(case["limbs"], 4)
        return case
    # words of one batch entry's largest array; the batch keeps the case below the listed ones
    per = {"ntt_fwd": 1, "mul_plain": 2, "polymul": 2, "ct_tensor": 4, "rescale": 1, "mul_relin_rs": 3 * limbs}[op]
    room = (1 << 26) // (per * limbs << log_n)
    case["batch"] = _log_uniform(rng, 1, max(1, min(room, 4096)))
    return case


def _jobs(case):
    """(log_n, limbs) of the jobs of a batch or grouped case."""
    if case["op"] == "batch" and case["jobs_seed"] == 0:
        return workloads.uneven_jobs(case["batch"], 12, 17, case["limbs"])
    r = random.Random(case["jobs_seed"])
    if case["op"] == "batch":
        return [(r.randint(12, 17), r.randint(1, case["limbs"])) for _ in range(case["batch"])]
    return [(r.randint(14, 16), r.randint(min(4, case["limbs"]), case["limbs"])) for _ in range(case["batch"])]


# ------------------------------------------------------------------ state and pass
@functools.lru_cache(maxsize=None)
def _tables(chain, log_n, limbs):
    """A program makes its tables once and uses them for every input."""
    return H.Tables(log_n, workloads.moduli(chain)[:limbs])


def _device():
    return torch.device("cuda:0")


def _inputs(case, seed):
    """Seeded operands on the GPU: uniform residues below each limb's modulus."""
    gen = torch.Generator(device=_device())
    gen.manual_seed(1000003 * seed + 17)
    mods = workloads.moduli(case["chain"])
    op, L, n, b = case["op"], case["limbs"], 1 << case["log_n"], case["batch"]

    def uniform(*lead, limbs=L):
        x = torch.empty(lead + (limbs, n), dtype=torch.int64, device=_device())
        for l in range(limbs):
            x[..., l, :].random_(0, mods[l], generator=gen)
        return x

    if op == "ntt_fwd":
        return [uniform(b)]
    if op in ("mul_plain", "polymul"):
        return [uniform(b), uniform(b)]
    if op == "ct_tensor":
        return [uniform(b, 2), uniform(b, 2)]
    if op == "rescale":
        return [uniform(b)]
    if op == "mul_relin_rs":
        return [uniform(b, 2), uniform(b, 2), uniform(L, 2, limbs=L + 1)]
    if op == "ct_matmul":
        return [uniform(b, case["k"], 2), uniform(case["k"], case["n"], 2)]
    # batch and grouped: one flat buffer per operand, jobs one after another
    polys = 1 if op == "batch" else 2
    jobs = _jobs(case)
    total = sum(polys * lv << ln for ln, lv in jobs)
    q = torch.tensor(mods, dtype=torch.int64, device=_device()).view(-1, 1)
    flats = []
    for _ in range(polys):
        flat = torch.empty(total, dtype=torch.int64, device=_device())
        flat.random_(0, (1 << 63) - 1, generator=gen)
        for x in _split(flat, jobs, polys):
            x.remainder_(q[:x.shape[-2]])
        flats.append(flat)
    return flats


def _split(flat, jobs, polys):
    """Views [polys, limbs, N] ([1, limbs, N] for one polynomial) of each job's words in a flat buffer."""
    out, at = [], 0
    for ln, lv in jobs:
        words = polys * lv << ln
        out.append(flat[at:at + words].view(polys, lv, 1 << ln))
        at += words
    return out


def prepare(case, seed):
    op, L, b, n = case["op"], case["limbs"], case["batch"], 1 << case["log_n"]
    x = _inputs(case, seed)
    s = {"op": op, "x": x}

    def empty(*shape):
        return torch.empty(shape, dtype=torch.int64, device=_device())

    if op == "batch":
        s["buf"] = torch.empty_like(x[0])
        jobs = _jobs(case)
        spec = [(v, _tables(case["chain"], ln, 32), lv) for v, (ln, lv) in zip(_split(s["buf"], jobs, 1), jobs)]
        s["buf"].copy_(x[0])
        s["plan"] = H.BatchPlan(spec, case["dir"])
        s["plan"].capture()
        return s
    if op == "grouped":
        jobs = _jobs(case)
        outs = [empty(1, 3, lv, 1 << ln) for ln, lv in jobs]
        c, d = ([v.unsqueeze(0) for v in _split(f, jobs, 2)] for f in x)
        views = {}
        for ln, lv in jobs:
            if (ln, lv) not in views:
                views[ln, lv] = _tables(case["chain"], ln, 24).view(lv)
        s["jobs"] = [(views[j], cc, dd, o) for j, cc, dd, o in zip(jobs, c, d, outs)]
        s["out"] = outs
        return s
    s["t"] = _tables(case["chain"], case["log_n"], L)
    if op in ("ntt_fwd", "mul_plain", "polymul"):
        s["out"] = empty(b, L, n)
    elif op == "ct_tensor":
        s["out"] = empty(b, 3, L, n)
    elif op == "rescale":
        s["out"] = empty(b, L - 1, n)
    elif op == "ct_matmul":
        s["out"] = empty(b, case["n"], 3, L, n)
    elif op == "mul_relin_rs":
        s["t1"] = _tables(case["chain"], case["log_n"], L + 1)
        s["prod"], s["lin"], s["out"] = empty(b, 3, L, n), empty(b, 2, L, n), empty(2 * b, L - 1, n)
    return s


def run(s):
    op, x = s["op"], s["x"]
    if op == "ntt_fwd":
        s["out"].copy_(x[0])
        return H.ntt_fwd(s["t"], s["out"])
    if op == "mul_plain":
        return H.ntt_inv(s["t"], H.dyadic_mul(s["t"], x[0], x[1], out=s["out"]))
    if op == "polymul":
        return H.polymul(s["t"], x[0], x[1], out=s["out"])
    if op == "ct_tensor":
        return H.ct_tensor(s["t"], x[0], x[1], out=s["out"])
    if op == "rescale":
        return H.rescale(s["t"], x[0], out=s["out"], ntt=True)
    if op == "ct_matmul":
        s["out"].zero_()
        return H.ct_matmul(s["t"], x[0], x[1], s["out"])
    if op == "mul_relin_rs":
        H.ct_tensor(s["t"], x[0], x[1], out=s["prod"], in_ntt=True, out_ntt=True)
        H.relin(s["t1"], s["prod"], x[2], out=s["lin"])
        b, _, L, n = s["lin"].shape
        return H.rescale(s["t"], s["lin"].view(2 * b, L, n), out=s["out"], ntt=True)
    if op == "batch":
        s["buf"].copy_(x[0])
        s["plan"].replay()
        return s["buf"]
    H.ct_tensor_grouped(s["jobs"])
    return s["out"]


def work(case):
    """Compulsory bytes (inputs read once, outputs written once) and 32-bit
    integer multiplies: 10 per butterfly (a 64-bit modular product by a
    constant), 11 per product of two variables, 37 per tensor slot."""
    op, L, b, ln = case["op"], case["limbs"], case["batch"], case["log_n"]
    n = 1 << ln

    def ntt(polys, log_n):
        return 10.0 * polys * (log_n << log_n) / 2

    if op == "ntt_fwd":
        return {"bytes": 16.0 * b * L * n, "flops": ntt(b * L, ln)}
    if op == "mul_plain":
        return {"bytes": 24.0 * b * L * n, "flops": ntt(b * L, ln) + 11.0 * b * L * n}
    if op == "polymul":
        return {"bytes": 24.0 * b * L * n, "flops": 3 * ntt(b * L, ln) + 11.0 * b * L * n}
    if op == "ct_tensor":
        return {"bytes": 56.0 * b * L * n, "flops": 7 * ntt(b * L, ln) + 37.0 * b * L * n}
    if op == "rescale":
        return {"bytes": 8.0 * b * (2 * L - 1) * n, "flops": ntt(b * L, ln) + 20.0 * b * L * n}
    if op == "ct_matmul":
        m, c, k = b, case["n"], case["k"]
        return {"bytes": 8.0 * L * n * (2 * m * k + 2 * k * c + 3 * m * c), "flops": 37.0 * m * c * k * L * n}
    if op == "mul_relin_rs":
        ks = ntt(b * (L + L * (L + 1)), ln) + 22.0 * b * L * (L + 1) * n
        rs = ntt(2 * b * (L + 1), ln) + ntt(2 * b * L, ln)
        return {"bytes": 8.0 * n * (4 * b * L + 2 * L * (L + 1) + 2 * b * (L - 1)), "flops": 37.0 * b * L * n + ks + rs}
    if op == "batch":
        return {"bytes": sum(16.0 * lv * (1 << ln2) for ln2, lv in _jobs(case)),
                "flops": sum(ntt(lv, ln2) for ln2, lv in _jobs(case))}
    return {"bytes": sum(56.0 * lv * (1 << ln2) for ln2, lv in _jobs(case)),
            "flops": sum(7 * ntt(lv, ln2) + 37.0 * lv * (1 << ln2) for ln2, lv in _jobs(case))}


# ------------------------------------------------------------------ plain numpy in 64 bits
def _mulmod(a, b, q):
    """a b mod q for uint64 arrays below q < 2^60: the quotient from 64-bit-mantissa floats, one correction."""
    a, b = np.asarray(a, dtype=np.uint64), np.asarray(b, dtype=np.uint64)
    quot = (a.astype(np.longdouble) * b.astype(np.longdouble) / np.longdouble(q)).astype(np.uint64)
    r = (a * b - quot * np.uint64(q)).view(np.int64)
    r = np.where(r < 0, r + np.int64(q), r)
    return np.where(r >= q, r - np.int64(q), r).view(np.uint64)


@functools.lru_cache(maxsize=None)
def _roots(q, log_n):
    """(powers of psi, powers of psi^-1), psi the smallest primitive 2N-th root of unity mod q."""
    n = 1 << log_n
    g = next(c for c in (pow(r, (q - 1) // (2 * n), q) for r in range(2, 10 ** 6)) if pow(c, n, q) == q - 1)

    def powers(r):
        p = np.ones(1, dtype=np.uint64)
        while p.size < 2 * n:
            p = np.concatenate([p, _mulmod(p, np.uint64(pow(r, p.size, q)), q)])
        return p

    psi = int(powers(g)[1::2].min())
    return powers(psi)[:n], powers(pow(psi, q - 2, q))[:n]


def _brv(n):
    r = np.zeros(1, dtype=np.int64)
    while r.size < n:
        r = np.concatenate([2 * r, 2 * r + 1])
    return r


def _ntt(x, q, inverse=False):
    """Negacyclic transform of the rows of x (uint64 [rows, N]); the NTT domain is bit-reversed."""
    n = x.shape[-1]
    w, wi = _roots(q, n.bit_length() - 1)
    order, x, q_ = _brv(n), x.copy(), np.uint64(q)
    gaps = [n >> (s + 1) for s in range(n.bit_length() - 1)]
    for gap in (reversed(gaps) if inverse else gaps):
        blocks = n // (2 * gap)
        tw = (wi if inverse else w)[order[blocks:2 * blocks] if blocks > 1 else order[1:2]].reshape(1, blocks, 1)
        v = x.reshape(-1, blocks, 2, gap)
        a, b = v[:, :, 0], v[:, :, 1]
        if inverse:
            s, d = (a + b) % q_, (a + q_ - b) % q_
            v[:, :, 0], v[:, :, 1] = s, _mulmod(d, tw, q)
        else:
            t = _mulmod(b, tw, q)
            v[:, :, 0], v[:, :, 1] = (a + t) % q_, (a + q_ - t) % q_
    return _mulmod(x, np.uint64(pow(n, q - 2, q)), q) if inverse else x


def _by_limb(f, mods, *arrays):
    """f(rows of limb l of every array, q_l) for each limb, stacked back; arrays [..., limbs, N]."""
    outs = []
    for l, q in enumerate(mods):
        rows = [a[..., l, :].reshape(-1, a.shape[-1]) for a in arrays]
        outs.append(f(*rows, q))
    lead = arrays[0].shape[:-2]
    return np.stack([o.reshape(lead + (o.shape[-1],)) for o in outs], axis=-2)


def _tensor(c, d, mods):
    def one(c0, c1, d0, d1, q):
        return np.concatenate([_mulmod(c0, d0, q)[:, None], ((_mulmod(c0, d1, q) + _mulmod(c1, d0, q)) % np.uint64(q))[:, None],
                               _mulmod(c1, d1, q)[:, None]], axis=1)
    outs = [one(c[:, 0, l], c[:, 1, l], d[:, 0, l], d[:, 1, l], q) for l, q in enumerate(mods)]
    return np.stack(outs, axis=2)


def _rescale(x, mods):
    """[rows, limbs, N] NTT domain -> [rows, limbs - 1, N]: round(x / q_last)."""
    ql = mods[-1]
    h = (ql - 1) // 2
    r = (_ntt(x[:, -1], ql, inverse=True) + np.uint64(h)) % np.uint64(ql)
    outs = []
    for l, q in enumerate(mods[:-1]):
        q_ = np.uint64(q)
        t = _ntt((r % q_ + q_ - np.uint64(h % q)) % q_, q)
        outs.append(_mulmod((x[:, l] + q_ - t) % q_, np.uint64(pow(ql, q - 2, q)), q))
    return np.stack(outs, axis=1)


def exact(case, seed):
    """The outputs of run() by plain numpy; None where that would take long."""
    if work(case)["flops"] > 1.2e9:
        return None
    op, L, n = case["op"], case["limbs"], 1 << case["log_n"]
    mods = workloads.moduli(case["chain"])
    x = [v.cpu().numpy().view(np.uint64) for v in _inputs(case, seed)]

    def words(a):
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int64))

    def product(a, b, q):
        return _ntt(_mulmod(_ntt(a, q), _ntt(b, q), q), q, inverse=True)

    m = mods[:L]
    if op == "ntt_fwd":
        return words(_by_limb(_ntt, m, x[0]))
    if op == "mul_plain":
        return words(_by_limb(lambda a, b, q: _ntt(_mulmod(a, b, q), q, inverse=True), m, x[0], x[1]))
    if op == "polymul":
        return words(_by_limb(product, m, x[0], x[1]))
    if op in ("ct_tensor", "grouped"):
        def whole(c, d, mm):
            t = _tensor(_by_limb(_ntt, mm, c), _by_limb(_ntt, mm, d), mm)
            return words(_by_limb(lambda a, q: _ntt(a, q, inverse=True), mm, t))
        if op == "ct_tensor":
            return whole(x[0], x[1], m)
        jobs = _jobs(case)
        c, d = ([v.numpy().view(np.uint64) for v in _split(torch.from_numpy(f.view(np.int64)), jobs, 2)] for f in x)
        return [whole(cc[None], dd[None], mods[:lv]) for cc, dd, (_, lv) in zip(c, d, jobs)]
    if op == "rescale":
        return words(_rescale(x[0], m))
    if op == "ct_matmul":
        rows, cols, k = case["batch"], case["n"], case["k"]
        out = np.zeros((rows, cols, 3, L, n), dtype=np.uint64)
        for i in range(rows):
            for l in range(k):
                t = _tensor(np.broadcast_to(x[0][i, l], (cols, 2, L, n)), x[1][l], m)
                out[i] = (out[i] + t) % np.array(m, dtype=np.uint64).reshape(L, 1)
        return words(out)
    if op == "mul_relin_rs":
        m1, b = mods[:L + 1], case["batch"]
        prod = _tensor(x[0], x[1], m)
        digits = [_ntt(prod[:, 2, j], q, inverse=True) for j, q in enumerate(m)]
        acc = np.zeros((b, 2, L + 1, n), dtype=np.uint64)
        for t, q in enumerate(m1):
            for j in range(L):
                v = _ntt(digits[j] % np.uint64(q), q)
                for s in (0, 1):
                    acc[:, s, t] = (acc[:, s, t] + _mulmod(v, x[2][j, s, t], q)) % np.uint64(q)
        lin = _rescale(acc.reshape(2 * b, L + 1, n), m1).reshape(b, 2, L, n)
        lin = _by_limb(lambda a, c, q: (a + c) % np.uint64(q), m, lin, prod[:, :2])
        return words(_rescale(lin.reshape(2 * b, L, n), m))
    flat, at, outs = x[0], 0, []
    for ln, lv in _jobs(case):
        v = flat[at:at + (lv << ln)].reshape(1, lv, 1 << ln)
        outs.append(_by_limb(lambda a, q: _ntt(a, q, inverse=case["dir"] < 0), mods[:lv], v).reshape(-1))
        at += lv << ln
    return words(np.concatenate(outs))
