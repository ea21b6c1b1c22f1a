"""GPU parity of the matrix product's column runs: single columns on small
matrices, longer and uneven runs as the workgroups fill the chip.  Oracle
comparison, exact."""
import numpy as np
import pytest

import oracle
from test_gpu_two_pass_edges import dev, host, primes, words

pytestmark = pytest.mark.gpu


# with two workgroups per CU wanted (512 on 256 CUs): single columns; runs of 1 and 2;
# of 2 and 3; of 4 and 5; of 5, past the 16 steps of a reduction
@pytest.mark.parametrize("log_n,m,n,k", [(6, 3, 7, 17), (9, 16, 12, 2), (10, 8, 20, 2), (11, 8, 34, 1), (12, 16, 10, 17)])
def test_matmul_runs(gpu, log_n, m, n, k):
    import paper_2109_14704_amd as H
    print("case matmul runs log_n=%d %dx%dx%d" % (log_n, m, n, k), flush=True)
    mods = primes(60, log_n) + primes(55, log_n)
    rng = np.random.default_rng(log_n)
    N, L = 1 << log_n, 2
    A, B, C = (words(rng, (a, b, e, L, N), mods) for a, b, e in ((m, k, 2), (k, n, 2), (m, n, 3)))
    got = H.ct_matmul(H.Tables(log_n, mods), dev(A, gpu), dev(B, gpu), dev(C, gpu))
    assert np.array_equal(host(got), oracle.ct_matmul(A, B, C, mods))
