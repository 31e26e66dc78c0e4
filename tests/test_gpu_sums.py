"""Error of fp32 products against the exact one, for plans of few K slices: below that of one fp32 sum per slice, k after k, since
the kernels hold two sums and more for each element.  (Sums of half the length have 0.7 of its error.)"""
import numpy as np
import pytest

import peak_inputs as pi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from tests import gpu_util
    return gpu_util


def _one_sum_per_slice(a, b, k_slice):
    """a: rows x K, b: K x N in fp32; the slices' sums added in fp32 in order."""
    total = np.zeros((a.shape[0], b.shape[1]), np.float32)
    for k0 in range(0, a.shape[1], k_slice):
        acc = np.zeros_like(total)
        for k in range(k0, min(k0 + k_slice, a.shape[1])):
            acc = (acc + a[:, k:k + 1].astype(np.float64) * b[k:k + 1].astype(np.float64)).astype(np.float32)
        total += acc
    return total


@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 1, 26, 5504, 2048), (0, 0, 28, 11328, 2688), (0, 1, 16, 5568, 2176), (0, 0, 8, 10944, 2304),
                                         (0, 1, 192, 4304, 7576), (1, 0, 1043, 2179, 1697), (1, 0, 797, 2311, 673)])
def test_error_below_one_sum_per_slice(gu, ta, tb, M, N, K):
    la, lb = (pi.logical_matrix(90, i, *s, "uniform", 1.0, pi.F32) for i, s in enumerate(((M, K), (K, N))))
    got, _, info = gu.run_gemm(pi.F32, ta, tb, M, N, K, 1.0, 0.0, pi.store(la, bool(ta)), pi.store(lb, bool(tb)), np.zeros((M, N), np.float32))
    fields = dict(w.split("=", 1) for w in info.split() if "=" in w)
    k_slice = int(fields["ktiles/slice"]) * int(fields["tile"].split("x")[2])
    rows, cols = np.linspace(0, M - 1, 6).astype(int), slice(0, 512)
    exact = la[rows].astype(np.float64) @ lb[:, cols].astype(np.float64)
    err = lambda x: np.linalg.norm(x - exact) / np.linalg.norm(exact)
    one = err(_one_sum_per_slice(la[rows], lb[:, cols], k_slice).astype(np.float64))
    mine = err(got[rows][:, cols])
    print(info, "%.2e %.2e %.2f" % (one, mine, mine / one), flush=True)
    assert mine < 0.85 * one, (info, mine, one)
