"""The matrix product's forms at the sizes where each is chosen and where its
tiles end, and the split form outside its range, against the FP64 oracle.

Bar per element as in test_gpu_gemm: |C - C_ref| <= 2 K 2^-24 (|A| |B|)_ij, plus
K times the smallest FP32 number for products below the normal range."""

import sys

import numpy as np
import pytest

import oracle
import paper_2011_03602_amd as ofl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]


def say(*args):
    print("[gpu]", *args, flush=True)
    sys.stdout.flush()


def product(a, b, pads=(0, 0, 0)):
    """C = A B through the C interface, rows padded by the given elements."""
    M, K = a.shape
    N = b.shape[1]
    lda, ldb, ldc = K + pads[0], N + pads[1], N + pads[2]
    da = torch.full((M, lda), float("nan"), device="cuda")
    db = torch.full((K, ldb), float("nan"), device="cuda")
    dc = torch.full((M, ldc), 7.0, device="cuda")
    da[:, :K], db[:, :N] = torch.as_tensor(a), torch.as_tensor(b)
    ofl.ofl_gemm_f32(M, N, K, da.data_ptr(), lda, db.data_ptr(), ldb, dc.data_ptr(), ldc, None)
    torch.cuda.synchronize()
    out = dc.cpu().numpy()
    assert np.all(out[:, N:] == 7.0), "wrote past the row"
    return out[:, :N]


def check_rows(a, b, c, rows):
    a, c = a[rows], c[rows]
    ref = oracle.gemm(a, b)
    K = a.shape[1]
    bound = 2.0 * K * 2.0 ** -24 * oracle.gemm(np.abs(a), np.abs(b)) + K * 2.0 ** -149
    err = np.abs(c.astype(np.float64) - ref)
    assert np.all(err <= bound), f"worst excess {float(np.max(err / bound)):.3f} of the bound"


# 16 x 16, 32 x 16 and 32 x 32 direct tiles and their remainders, K below, at and
# past a chunk of 32 and a turn of all waves; split tiles of 128 with one group
# (small K) and two, whole and ragged in M, N (also N % 4) and K.
SHAPES = [(17, 15, 31), (16, 16, 512), (130, 20, 545), (8192, 16, 64), (2049, 9, 257), (33, 31, 32), (511, 333, 101),
          (1000, 400, 40), (64, 2000, 96), (4096, 2049, 33), (4097, 2048, 64), (2305, 2178, 160), (2050, 1155, 999),
          (2176, 2176, 65)]


@pytest.mark.parametrize("pads", [(0, 0, 0), (3, 1, 5)], ids=["tight", "odd strides"])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_forms_match_oracle(M, N, K, pads):
    say("gemm forms", M, N, K, pads)
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    a = rng.standard_normal((M, K)).astype(np.float32)
    b = rng.standard_normal((K, N)).astype(np.float32)
    c = product(a, b, pads)
    check_rows(a, b, c, sorted({r for r in (0, 1, 15, 16, 31, 32, 63, 64, 127, 128, 129, M // 2, M - 1) if r < M}))


# a split product of two groups with ragged tiles
M_, N_, K_ = 2305, 1155, 320


def operands(seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((M_, K_)).astype(np.float32), rng.standard_normal((K_, N_)).astype(np.float32)


@pytest.mark.parametrize("scale_a,scale_b", [(1e-30, 1e20), (1e-18, 1.0), (1e25, 1e-28), (1e-20, 1e-14), (1e18, 1e17)])
def test_split_range(scale_a, scale_b):
    """Magnitudes inside and outside the range of bfloat16 parts."""
    say("gemm range", scale_a, scale_b)
    a, b = operands(1)
    a, b = (a * np.float32(scale_a)).astype(np.float32), (b * np.float32(scale_b)).astype(np.float32)
    check_rows(a, b, product(a, b), [0, 5, 127, 128, 1000, 2304])


def test_split_mixed_magnitudes_and_zeros():
    """Zeros (no magnitude at all) beside ordinary values, one tiny value in one
    tile, FP32 subnormals, and values near the largest."""
    say("gemm mixed magnitudes")
    a, b = operands(2)
    a[a < 0.3] = 0.0
    a[200, :] = 0.0
    a[3, 7] = np.float32(1e-30)
    a[700, :] = np.float32(1e-41)
    b[:, 5] *= np.float32(1e30)
    a[900, :] = 0.0
    a[900, 11] = np.float32(3.4e38)
    b[11, :] = np.clip(b[11, :], -0.9, 0.9)
    b[11, 5] = np.float32(0.5)
    c = product(a, b)
    check_rows(a, b, c, [0, 3, 127, 200, 700, 900, 2304])
    assert np.all(c[200] == 0.0)


def test_split_infinities_and_nans():
    """Infinite and NaN operands give what the definition gives, element by element."""
    say("gemm inf / nan")
    a, b = operands(3)
    a[10, 3] = np.inf
    a[300, 4] = -np.inf
    a[301, 5] = np.nan
    b[6, 40] = np.inf
    b[7, 41] = np.nan
    c = product(a, b)
    rows = [9, 10, 11, 300, 301, 2304]
    with np.errstate(invalid="ignore"):
        ref = a[rows].astype(np.float64) @ b.astype(np.float64)
    got = c[rows]
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 2.0 * K_ * 2.0 ** -24 * 6.0 * K_)
