"""The matrix product's split form over FP32's whole range, against the FP64 oracle."""

import sys

import numpy as np
import pytest

import oracle
import paper_2011_03602_amd as ofl
from test_gpu_gemm_forms import check_rows, product

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # collected on CPU hosts, skipped there
    pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="needs a GPU")]

# a split product of two groups with ragged tiles, and one of one group
SHAPES = [(2305, 1155, 320), (4097, 2050, 64)]


def say(*args):
    print("[gpu]", *args, flush=True)
    sys.stdout.flush()


def one_per_row(M, K, values):
    """A matrix with one value in each row, the rows in turn over the columns."""
    a = np.zeros((M, K), dtype=np.float32)
    a[np.arange(M), (7 * np.arange(M) + 3) % K] = values
    return a


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_every_magnitude(M, N, K):
    """Single products a b with a from the smallest subnormal numbers to 2^100 and
    b such that a b is normal: a's and b's parts are exact, the products of parts
    left out come to 2^-24 of |a b|, and two roundings to 2^-23 and 2^-24 at most
    (a sum's lower addend is truncated): together 2^-22."""
    say("gemm every magnitude", M, N, K)
    rng = np.random.default_rng(M)
    # rows from 2^-149 to 2^100, columns from 2^-20 to 2^20 and, times 2^60, to
    # 2^80, dealt so that no product leaves 2^-126 .. 2^127
    e = np.linspace(-149.0, 100.0, M)
    a = (np.exp2(e) * rng.choice([-1.0, 1.0], M)).astype(np.float32)
    a[a == 0] = np.float32(2.0 ** -149)
    A = one_per_row(M, K, a)
    low, high = np.exp2(rng.uniform(-20.0, 20.0, (K, N // 2))), np.exp2(rng.uniform(40.0, 80.0, (K, N - N // 2)))
    B = (np.concatenate([low, high], axis=1) * rng.choice([-1.0, 1.0], (K, N))).astype(np.float32)
    c = product(A, B)
    cols = (7 * np.arange(M) + 3) % K
    ref = a.astype(np.float64)[:, None] * B.astype(np.float64)[cols]
    fits = (np.abs(ref) >= 2.0 ** -126) & (np.abs(ref) < 2.0 ** 126)
    assert fits.mean() > 0.6
    err = np.abs(c.astype(np.float64) - ref)
    assert np.all(err[fits] <= 2.0 ** -22 * np.abs(ref[fits]))


def test_sums_around_the_split_form_s_largest():
    """Sums that cross 2^82 only when the two groups' halves of K meet, and sums
    past it, up to FP32's largest and over it."""
    M, N, K = SHAPES[0]
    say("gemm large sums")
    a = np.full((M, K), 2.0 ** 44, dtype=np.float32)
    b = np.full((K, N), 1.0, dtype=np.float32)
    for j, factor in enumerate((0.7, 1.0, 1.5, 2.0, 3.0, 1e3, 1e9, 2.0 ** 45.9)):
        b[:, j::8] = np.float32(2.0 ** 38 / K * factor)
    c = product(a, b)
    ref = a[:1].astype(np.float64) @ b.astype(np.float64)
    assert np.all(np.isfinite(c)) and np.all(np.abs(c - ref) <= 2.0 * K * 2.0 ** -24 * ref)
    b[:, 5] = np.float32(2.0 ** 84)
    c = product(a, b)
    assert np.all(np.isposinf(c[:, 5])) and np.all(np.isfinite(np.delete(c, 5, axis=1)))


def timed(M, N, K, a, b):
    c = torch.zeros((M, N), device="cuda")

    def call():
        ofl.ofl_gemm_f32(M, N, K, a.data_ptr(), K, b.data_ptr(), N, c.data_ptr(), N,
                         torch.cuda.current_stream().cuda_stream)

    for _ in range(3):
        call()
    ms = []
    for _ in range(9):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(4):
            call()
        ev[1].record()
        torch.cuda.synchronize()
        ms.append(ev[0].elapsed_time(ev[1]))
    return min(ms)


@pytest.mark.parametrize("scale", [1e-18, 1e-30, 1e30])
def test_operands_in_any_unit_cost_the_same(scale):
    """An operand in small or large units, and one with a few such values, take one
    run of the tiles as others do (a second one on the FP32 instructions takes over
    twice as long; half as much again is far outside the timing's noise)."""
    M = N = K = 2048
    say("gemm operands' time", scale)
    a, b = torch.randn((M, K), device="cuda"), torch.randn((K, N), device="cuda")
    usual = timed(M, N, K, a, b)
    assert timed(M, N, K, a * scale, b) <= 1.5 * usual
    a[::100, ::50] = scale
    assert timed(M, N, K, a, b) <= 1.5 * usual


def test_large_values_after_the_first_stages():
    """Values whose scaled parts overflow, or whose unscaled ones are subnormal, where
    the first 32 (64) k of the tile did not tell."""
    say("gemm late magnitudes")
    rng = np.random.default_rng(6)
    M, N, K = SHAPES[0]
    a, b = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    a[70, 200:] *= np.float32(2.0 ** 110)   # past the scaled range, from k = 200
    a[900, 3] = np.float32(2.0 ** 60)       # unscaled from the first stage on,
    a[901, :] = np.float32(2.0 ** -120)     # and a row below its range
    b[300, 700] = np.float32(3e38)
    b[301, 701] = np.float32(1e-42)
    c = product(a, b)
    rows = [0, 69, 70, 127, 128, 900, 901, 902, 2304]
    # 3e38 times most values is past FP32's largest: infinite, as it has to be
    with np.errstate(over="ignore"):
        over = np.isinf(oracle.gemm(a[rows], b).astype(np.float32))
    assert over.sum() < 2 * len(rows) and np.all(np.isinf(c[rows][over]))
    c[rows] = np.where(over, 0.0, c[rows])
    ref = np.where(over, 0.0, oracle.gemm(a[rows], b))
    bound = 2.0 * K * 2.0 ** -24 * oracle.gemm(np.abs(a[rows]), np.abs(b)) + K * 2.0 ** -149
    assert np.all(np.abs(c[rows].astype(np.float64) - ref) <= bound)


def test_small_operands_values():
    say("gemm small operands' values")
    rng = np.random.default_rng(5)
    M, N, K = SHAPES[0]
    a, b = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    for scale in (1e-18, 1e-30, 1e-37, 1e-41):
        x = (a * np.float32(scale)).astype(np.float32)
        check_rows(x, b, product(x, b), [0, 5, 127, 128, 1000, 2304])


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_single_products_are_rounded_once(M, N, K):
    """A matrix with one value per row times a dense one, so that every element of C
    is one product: half an ulp as in FP32, plus what the product of the third parts
    (left out: 2^-11 ulp) and the truncated sums of the lower products (four, at most
    2^-7 ulp each) may add, 2^-5."""
    say("gemm single products", M, N, K)
    rng = np.random.default_rng(K)
    A = one_per_row(M, K, rng.standard_normal(M))
    B = rng.standard_normal((K, N)).astype(np.float32)
    c = product(A, B)
    cols = (7 * np.arange(M) + 3) % K
    ref = A[np.arange(M), cols].astype(np.float64)[:, None] * B.astype(np.float64)[cols]
    ulp = np.exp2(np.floor(np.log2(np.abs(ref))) - 23)
    assert np.max(np.abs(c - ref) / ulp) <= 0.5 + 2.0 ** -5


@pytest.mark.parametrize("M,K", [(1, 1), (2, 3)])
def test_rows_of_more_columns_than_small_tiles_reach(M, K):
    """2^28 columns and more: launches of small tiles would hold 2^32 threads."""
    N = (1 << 28) + 40
    say("gemm long rows", M, N, K)
    a = torch.randn((M, K), device="cuda")
    b = torch.randn((K, N), device="cuda")
    c = torch.full((M, N), 7.0, device="cuda")
    ofl.ofl_gemm_f32(M, N, K, a.data_ptr(), K, b.data_ptr(), N, c.data_ptr(), N, None)
    torch.cuda.synchronize()
    for first in range(0, N, 1 << 25):
        part = slice(first, min(first + (1 << 25), N))
        x = b[:, part].double()
        ref = sum(a[:, k:k + 1].double() * x[k:k + 1] for k in range(K))
        mag = sum(a[:, k:k + 1].double().abs() * x[k:k + 1].abs() for k in range(K))
        assert bool(((c[:, part].double() - ref).abs() <= 2.0 * K * 2.0 ** -24 * mag).all())
