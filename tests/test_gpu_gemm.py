"""GPU parity of focus_gemm against a float64 matrix product of the same bf16
inputs (a plain NumPy matmul is the definition).  Tolerance: f32 output
rel-L2 <= 1e-5 and max-abs <= 1e-4 * sqrt(k); bf16 output adds the output
rounding (relative 2^-9): rel-L2 <= 5e-3.  Cases: ragged M (tails of the
16-, 64-, 128- and 256-row tiles), several N and K tiles, gathered rows, alpha, leading dimensions larger than the row,
and the projection shapes of an Evo-2-scale layer (d = 4096)."""

import numpy as np
import pytest
import torch

import focus_workloads as fw
import paper_2511_14694_amd as F
from gpu_util import DEV, announce, rel_l2, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(1, 128, 64), (127, 128, 64), (129, 256, 128), (300, 384, 192),
                                   (300, 512, 256), (256, 256, 128), (256, 256, 64), (1000, 512, 1024), (4096, 1024, 4096)])
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
def test_gemm_matches_float64(m, n, k, out_dtype):
    announce(f"gemm m={m} n={n} k={k} out={out_dtype}")
    a = fw.randn((m, k), "bf16", m + k, DEV)
    b = fw.randn((k, n), "bf16", n + 7, DEV)
    od = torch.float32 if out_dtype == "f32" else torch.bfloat16
    c = F.focus_gemm(a, b, out_dtype=od, alpha=0.5)
    torch.cuda.synchronize()
    ref = 0.5 * (to64(a) @ to64(b))
    got = to64(c)
    r = rel_l2(got, ref)
    if out_dtype == "f32":
        assert r <= 1e-5 and np.abs(got - ref).max() <= 1e-4 * np.sqrt(k), r
    else:
        assert r <= 5e-3, r


@pytest.mark.parametrize("m,n,k", [(15, 128, 64), (16, 128, 576), (17, 256, 128), (32, 384, 64), (33, 128, 192),
                                   (65, 640, 64), (200, 12288, 128), (129, 16384, 64), (1025, 4224, 192),
                                   (2100, 4096, 64), (2100, 4352, 192), (4000, 2560, 128), (300, 32768, 192),
                                   (2100, 4096, 192), (4000, 2560, 256), (700, 6144, 192), (700, 6144, 128),
                                   (130, 16384, 128)])
def test_gemm_kernel_edges(m, n, k):
    """Each kernel of the dispatch at its edges: row tiles of 16, 32 and 64 (one
    and several), fewer k-steps than waves, the 128 x 128 tile over several
    rounds, the 256 x 256 tile with whole and partial groups of row stripes, in
    super blocks (N / 256 = 16, 10) and without (17).  Gathered rows in reverse,
    C at a column offset of two in a wider buffer (n + 6: some rows 16-byte
    aligned, some not; n + 8: none), and nothing written around it.  float32 sums
    of k products in any order: as above."""
    announce(f"gemm kernels m={m} n={n} k={k}")
    a = fw.randn((m + 3, k), "bf16", m + k, DEV)
    b = fw.randn((k, n), "bf16", n + 9, DEV)
    idx = torch.arange(m + 2, 2, -1, device=DEV)
    ref = a.float()[idx] @ b.float()
    for dt, tol in ((torch.float32, 1e-5), (torch.bfloat16, 5e-3)):
        whole = F.focus_gemm(a, b, out_dtype=dt, a_rows=idx)
        for pad in (6, 8):
            buf = torch.full((m + 1, n + pad), 7.0, dtype=dt, device=DEV)
            F.focus_gemm(a, b, out=buf[:m, 2:2 + n], a_rows=idx)
            torch.cuda.synchronize()
            assert torch.equal(buf[:m, 2:2 + n], whole)
            assert (buf[:, :2] == 7).all() and (buf[:, 2 + n:] == 7).all() and (buf[m] == 7).all()
        assert float((whole.float() - ref).norm() / ref.norm()) <= tol


def test_gemm_gathered_rows_and_strides():
    announce("gemm gather / strides")
    rows, k, n = 500, 256, 256
    big = fw.randn((rows, k + 64), "bf16", 3, DEV)
    a = big[:, :k]                                  # lda = k + 64
    b = fw.randn((k, n + 128), "bf16", 4, DEV)[:, :n]
    idx = np.random.default_rng(0).integers(0, rows, 333)
    out = torch.zeros(333, n + 128, dtype=torch.float32, device=DEV)[:, :n]
    F.focus_gemm(a, b, out=out, a_rows=idx)
    torch.cuda.synchronize()
    ref = to64(a)[idx] @ to64(b)
    assert rel_l2(to64(out), ref) <= 1e-5


def test_gemm_rejects_unsupported_shapes():
    a = torch.zeros(10, 100, dtype=torch.bfloat16, device=DEV)
    b = torch.zeros(100, 128, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(F.FocusError):
        F.focus_gemm(a, b)                          # k not a multiple of 64
