"""GPU parity of in-place transforms on words whose address is a multiple of 8
but not of 16 bytes: the inverse kernels' first load goes from global memory
straight into LDS, 16 bytes per lane where the address allows it.  Every N at
which a workgroup is at least one wave, every compiled instance, and the
persistent batch.  Oracle comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log_n", [7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17])
def test_transforms_in_place_8_byte_aligned(gpu, log_n):
    import paper_2109_14704_amd as H
    mods = primes(60, log_n) + primes(50, log_n)
    n, L, batch = 1 << log_n, 2, 2 if log_n > 14 else 5
    rng = np.random.default_rng(900 + log_n)
    x = words(rng, (batch, L, n), mods)
    t = H.Tables(log_n, mods)
    want = oracle.batch_ntt(x, mods, +1)
    cls = H.shape_class(batch * L)
    for op in ("fwd", "inv"):
        for choice in range(H.tune_count(op, log_n)):
            print("case 8-byte aligned %s log_n=%d instance=%d" % (op, log_n, choice), flush=True)
            H.tune_select(op, log_n, cls, choice)
            try:
                d = dev(x if op == "fwd" else want, gpu, 1)
                assert d.data_ptr() % 16 == 8
                assert np.array_equal(host((H.ntt_fwd if op == "fwd" else H.ntt_inv)(t, d)), want if op == "fwd" else x)
            finally:
                H.tune_select(op, log_n, cls, 0)


def test_batch_plan_8_byte_aligned(gpu):
    import paper_2109_14704_amd as H
    print("case 8-byte aligned persistent batch", flush=True)
    rng = np.random.default_rng(950)
    jobs, xs, fwd = [], [], []
    for log_n, limbs, batch, offset in [(9, 2, 3, 1), (12, 2, 3, 1), (13, 1, 2, 0), (14, 2, 1, 1), (16, 1, 1, 1)]:
        mods = primes(60, log_n) + primes(50, log_n)
        x = words(rng, (batch, limbs, 1 << log_n), mods[:limbs])
        xs.append(x)
        fwd.append(oracle.batch_ntt(x, mods[:limbs], +1))
        jobs.append((dev(fwd[-1], gpu, offset), H.Tables(log_n, mods), limbs))
    H.ntt_batch(jobs, -1)
    H.ntt_batch_status(jobs, -1)
    for (d, _, _), x in zip(jobs, xs):
        assert np.array_equal(host(d), x)
    H.ntt_batch(jobs, +1)
    H.ntt_batch_status(jobs, +1)
    for (d, _, _), y in zip(jobs, fwd):
        assert np.array_equal(host(d), y)
