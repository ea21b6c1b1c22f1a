"""GPU parity of the ciphertext matrix product where its kernel changes course:
column runs of 1 to 5 (n around multiples of 5), reductions every 16 steps (k
around 16 and 32), tiles of 256 coefficients (N below, at and above), moduli on
both sides of the correction rules, words at q - 1.  Oracle comparison, exact."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_two_pass_edges import dev, gpu, host, primes, words  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,log_n", [(1, 1, 1, 6), (2, 4, 16, 7), (3, 5, 17, 8), (1, 6, 15, 9), (2, 11, 33, 8),
                                         (9, 1, 5, 10), (1, 10, 2, 11)])
@pytest.mark.parametrize("bits", [(20, 33, 34), (55, 56, 60)])
def test_matmul_edges(gpu, m, n, k, log_n, bits):  # noqa: F811
    import paper_2109_14704_amd as H
    print("case matmul edges m=%d n=%d k=%d log_n=%d bits=%s" % (m, n, k, log_n, bits), flush=True)
    mods = [primes(b, log_n)[0] for b in bits]
    rng = np.random.default_rng(1000 * m + 100 * n + k)
    N = 1 << log_n
    A, B = words(rng, (m, k, 2, 3, N), mods), words(rng, (k, n, 2, 3, N), mods)
    C = words(rng, (m, n, 3, 3, N), mods)
    got = H.ct_matmul(H.Tables(log_n, mods), dev(A, gpu), dev(B, gpu), dev(C, gpu, 1))
    assert np.array_equal(host(got), oracle.ct_matmul(A, B, C, mods))
