"""fp32 products through the bf16 matrix units (three-part operands): every
layout at the tiles' edges, each way of loading, values outside bf16's range
and below it.

Bound per element: the 6 ceil(K / 16) additions of a chain each round by at
most 2^-24 of the running sum, which stays below S = sum_k |a b|; the terms
left out and the rounding inside a matrix instruction are covered by the
factor 2.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_1709_02755_amd import sru

pytestmark = pytest.mark.gpu


def product(op, A, B, M, N, K):
    out = sru.gemm(op, A, B, M, N, K, sru.GEMM_FP32)
    torch.cuda.synchronize()
    return out


def operands(op, M, N, K, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    a_shape = (K, M) if op == sru.OP_TN else (M, K)
    b_shape = (N, K) if op == sru.OP_NT else (K, N)
    return (torch.randn(a_shape, generator=g, device="cuda"),
            torch.randn(b_shape, generator=g, device="cuda"))


def canonical(op, A, B):
    A = A.t() if op == sru.OP_TN else A
    B = B.t() if op == sru.OP_NT else B
    return A.double(), B.double()


# (M, N, K): one element; the small tile's edges; unaligned pitches (dword
# loads); the middle and the large tile with remainders in every dimension
SHAPES = [(1, 1, 1), (63, 65, 31), (64, 64, 32), (65, 61, 129), (100, 260, 36), (128, 384, 128),
          (255, 1023, 77), (2048, 768, 256), (4100, 1028, 260), (5000, 2051, 67)]


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
@pytest.mark.parametrize("shape", SHAPES)
def test_within_fp32_rounding(op, shape):
    M, N, K = shape
    A, B = operands(op, M, N, K)
    out = product(op, A, B, M, N, K)
    a, b = canonical(op, A, B)
    bound = 2 * (6 * -(-K // 16) + 1) * 2.0 ** -24 * (a.abs() @ b.abs())
    err = (out.double() - a @ b).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
def test_unaligned_operands_same_bits(op):
    """4-byte aligned operands (dword loads) give the 16-byte loads' bits."""
    M, N, K = 130, 260, 68
    A, B = operands(op, M, N, K)
    ref = product(op, A, B, M, N, K)

    def shifted(t):
        buf = torch.empty(t.numel() + 1, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)

    out = product(op, shifted(A), shifted(B), M, N, K)
    assert torch.equal(out, ref)


def labelled(call):
    """The call's result and the names of its kernels."""
    events = [torch.cuda.Event(enable_timing=True) for _ in range(16)]
    for e in events:
        e.record()
    handles = (ctypes.c_void_p * 16)(*[e.cuda_event for e in events])
    lib = sru.lib()
    assert lib.sru_timing_begin(handles, 16) == 0
    out = call()
    labels = [lib.sru_timing_label(i).decode() for i in range(lib.sru_timing_end())]
    torch.cuda.synchronize()
    return out, labels


@pytest.mark.parametrize("L,B,d_in,d", [(64, 32, 256, 256), (20, 4, 64, 64), (33, 9, 100, 76)])
@pytest.mark.parametrize("shift_x,shift_w", [(True, False), (False, True), (True, True)])
def test_backward_pair_of_unaligned_operands(L, B, d_in, d, shift_x, shift_w):
    """Sizes whose dX and dW run in one launch: X or W on 4 bytes makes two
    launches of it, and the same bits (the same tiles and parts)."""
    g = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")

    def shifted(t):
        buf = torch.empty(t.numel() + 1, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)

    X, W = rand(L, B, d_in), rand(1, 3 if d == d_in else 4, d, d_in) * d_in ** -0.5
    dH = rand(L, B, d)
    p = [rand(1, d) * 0.3 for _ in range(4)]
    fw = sru.forward(X, W, *p)
    ref, labels = labelled(lambda: sru.backward(X, W, *p, fw["U"], fw["C"], dH))
    assert "gemm_dx_dw" in labels, labels
    out, labels = labelled(lambda: sru.backward(shifted(X) if shift_x else X,
                                                shifted(W) if shift_w else W, *p, fw["U"],
                                                fw["C"], dH))
    assert "gemm_dx" in labels and "gemm_dw" in labels and "gemm_dx_dw" not in labels, labels
    for n in ("dX", "dW", "dv_f", "dv_r", "db_f", "db_r"):
        assert torch.equal(out[n], ref[n]), n


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38, -3.4e38])
def test_values_beyond_bf16(op, value):
    """Infinities, NaN and magnitudes that round to infinity in bf16 come out
    as fp32 arithmetic has them, and other rows keep their values."""
    M, N, K = 200, 140, 50
    A, B = operands(op, M, N, K)
    B = B * 0.25
    where = (3, 150) if op == sru.OP_TN else (150, 3)
    A[where] = value
    out = product(op, A, B, M, N, K).cpu().numpy()
    a, b = canonical(op, A, B)
    ref = (a @ b).cpu().numpy()
    fine = np.isfinite(ref)
    np.testing.assert_array_equal(np.isnan(out), np.isnan(ref))
    np.testing.assert_array_equal(out[~fine & ~np.isnan(ref)], ref[~fine & ~np.isnan(ref)])
    bound = 2 * (K + 1) * 2.0 ** -24 * (a.abs() @ b.abs()).cpu().numpy()
    assert (np.abs(out[fine] - ref[fine]) <= bound[fine]).all()


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
@pytest.mark.parametrize("shape", [(200, 140, 50), (1030, 1028, 260), (4100, 2052, 132)])
def test_finite_results_beside_others_keep_their_bits(op, shape):
    """A row of A and a column of B with values that are not finite change no
    other row and column (one shape for each tile)."""
    M, N, K = shape
    A, B = operands(op, M, N, K)
    ref = product(op, A, B, M, N, K)
    m, n = M // 2 + 3, N // 2 + 5
    (A.t() if op == sru.OP_TN else A)[m, K // 2] = float("inf")
    (B if op == sru.OP_NT else B.t())[n, 7] = float("nan")
    out = product(op, A, B, M, N, K)
    assert not torch.isfinite(out[m]).any() and not torch.isfinite(out[:, n]).any()
    out[m], out[:, n] = ref[m], ref[:, n]
    assert torch.equal(out, ref)


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
@pytest.mark.parametrize("scale", [2.0 ** -112, 2.0 ** -122, 2.0 ** -133])
def test_small_values(op, scale):
    """Operands whose parts would lie below bf16's range, down to fp32's own
    subnormal ones: the bound of any other product, and the rounding of
    results (and of partial sums) below 2^-126."""
    M, N, K = 200, 140, 77
    for tiny in (0, 1):
        pair = list(operands(op, M, N, K))
        pair[tiny] = pair[tiny] * scale
        out = product(op, *pair, M, N, K)
        a, b = canonical(op, *pair)
        bound = (2 * (6 * -(-K // 16) + 1) * 2.0 ** -24 * (a.abs() @ b.abs()) + 64 * 2.0 ** -149)
        err = (out.double() - a @ b).abs()
        assert bool((err <= bound).all()), (tiny, float((err / bound).max()))


def test_small_gradients():
    """A backward pass is linear in dH: 2^-120 of it gives 2^-120 of every
    gradient, to fp32 rounding (2^-149 is 2^-26 of the smaller dU)."""
    L, B, d_in, d = 20, 9, 76, 100
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    X, W, dH = rand(L, B, d_in), rand(1, 4, d, d_in) * d_in ** -0.5, rand(L, B, d)
    p = [rand(1, d) * 0.3 for _ in range(4)]
    fw = sru.forward(X, W, *p)
    whole = sru.backward(X, W, *p, fw["U"], fw["C"], dH)
    small = sru.backward(X, W, *p, fw["U"], fw["C"], dH * 2.0 ** -120)
    torch.cuda.synchronize()
    for n in ("dX", "dW"):
        want, got = whole[n].double(), small[n].double() * 2.0 ** 120
        assert float((got - want).norm() / want.norm()) < 1e-6, n


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
@pytest.mark.parametrize("K", [32, 128, 1000])
def test_no_common_sign_in_errors(op, K):
    """The matrix instruction drops low bits of a small accumulator, always
    downwards; the rows' signs keep that from adding up over rows.  Mean of
    the errors over a column's 12,800 rows, against the standard error of a
    mean of independent ones (288 columns: 5 sigma; left alone about 20)."""
    M, N = 12800, 96
    A, B = operands(op, M, N, K)
    out = product(op, A, B, M, N, K)
    a, b = canonical(op, A, B)
    err = out.double() - a @ b
    z = err.mean(0) / (err.std(0) / M ** 0.5)
    assert float(z.abs().max()) < 5.0, z


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN])
@pytest.mark.parametrize("K", [32, 77, 128, 1000])
@pytest.mark.parametrize("lead,count", [(0.0, 16), (1.0, 8)])
def test_no_common_sign_with_equal_leading_values(op, K, lead, count):
    """The same where every row begins with the same values (fewer than a
    slab of 16 where they are not zero: the rounding of a whole slab of equal
    values is the same in every row, whatever its sign)."""
    M, N = 12800, 96
    A, B = operands(op, M, N, K)
    A[:, :count] = lead
    out = product(op, A, B, M, N, K)
    a, b = canonical(op, A, B)
    err = out.double() - a @ b
    z = err.mean(0) / (err.std(0) / M ** 0.5)
    assert float(z.abs().max()) < 5.0, z


def test_same_bits_at_every_row_and_size():
    """A row's results depend on its values alone, whichever tile runs it."""
    N, K = 768, 200
    A, B = operands(sru.OP_NT, 12800, N, K)
    whole = product(sru.OP_NT, A, B, 12800, N, K)
    for m0, m1 in ((0, 1), (1, 70), (3000, 3333), (5, 6001)):
        part = product(sru.OP_NT, A[m0:m1].contiguous(), B, m1 - m0, N, K)
        assert torch.equal(part, whole[m0:m1]), (m0, m1)


@pytest.mark.parametrize("op", [sru.OP_NT, sru.OP_NN, sru.OP_TN])
def test_rows_of_both_signs(op):
    """Whole numbers: exact, whatever sign a row takes."""
    M, N, K = 300, 40, 33
    A, B = (t.mul(3).round() for t in operands(op, M, N, K))
    out = product(op, A, B, M, N, K)
    a, b = canonical(op, A, B)
    assert torch.equal(out.double(), a @ b)
