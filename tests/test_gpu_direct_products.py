"""The layer's bf16 products (both tile sizes, split and whole, and the
staged pair of dX and dW) against float64
products of the same bf16-rounded operands: U, dX with its addends, dW.

Bound per element: an fp32 chain of K products in 16-k slabs, each rounded at
most twice, plus the partials' sums: (K / 8 + 16) 2^-24 of sum |a b|.
"""
import pytest
import torch

from paper_1709_02755_amd import sru

pytestmark = pytest.mark.gpu

CASES = [
    # (L, B, d_in, d, direction)
    (1, 3, 8, 8, sru.DIR_FWD),            # less than one tile, one K step
    (16, 8, 64, 64, sru.DIR_FWD),         # exactly one mid tile of tokens
    (43, 3, 72, 56, sru.DIR_BI),          # ragged rows, columns and K, two addends absent (k = 4)
    (31, 7, 200, 200, sru.DIR_BI),        # k = 3: two addends
    (64, 16, 512, 512, sru.DIR_FWD),      # whole mid tiles
    (77, 13, 304, 200, sru.DIR_REV),      # few tiles: dX split
    (256, 8, 1024, 1024, sru.DIR_FWD),    # one GPU's shard: dW and dX split, one sum
    (130, 33, 1032, 520, sru.DIR_FWD),    # ragged edges over many tiles
    (128, 64, 1024, 1024, sru.DIR_FWD),   # big tiles
    # dX with dW on staged tiles, W as it lies: rows of whole 8-byte chunks only
    (77, 13, 300, 200, sru.DIR_BI),       # dX alone would run direct
    (9, 5, 76, 36, sru.DIR_FWD),          # less than one tile of tokens
    (33, 9, 100, 100, sru.DIR_REV),       # one addend, N no whole 16-byte chunks
    (61, 19, 84, 84, sru.DIR_BI),         # two addends
    (25, 4, 77, 52, sru.DIR_FWD),         # rows in single elements: not paired
    (256, 64, 301, 301, sru.DIR_FWD),     # the same on big tiles
    (128, 63, 67, 1001, sru.DIR_FWD),
]


def close(got, a, b, add=0.0):
    ref = a @ b + add
    bound = (a.shape[1] / 8 + 16) * 2.0 ** -24 * (a.abs() @ b.abs() + abs(add))
    worst = float(((got.double() - ref).abs() - bound).max())
    assert worst <= 0.0, worst


@pytest.mark.parametrize("case", CASES)
def test_layer_products(case):
    L, B, d_in, d, direction = case
    nd = 2 if direction == sru.DIR_BI else 1
    k = 3 if d_in == d else 4
    g = torch.Generator(device="cuda").manual_seed(L + d)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    X, W = rand(L, B, d_in), rand(nd, k, d, d_in) * d_in ** -0.5
    p = [rand(nd, d) * 0.3 for _ in range(4)]
    dH = rand(L, B, nd * d)
    kw = dict(direction=direction)
    fw = sru.forward(X, W, *p, gemm_dtype=sru.GEMM_BF16, **kw)
    bw = sru.backward(X, W, *p, fw["U"], fw["C"], dH, gemm_dtype=sru.GEMM_BF16, **kw)
    # the caller's rounded copies instead of the workspace's: the same bits
    bc = sru.backward(X, W, *p, fw["U"], fw["C"], dH, gemm_dtype=sru.GEMM_BF16,
                      X_bf16=X.bfloat16(), W_bf16=W.bfloat16(), **kw)
    for n in ("dX", "dW"):
        assert torch.equal(bc[n], bw[n]), n
    sc = sru.scan_backward(fw["U"], X, fw["C"], dH, *p, d_in=d_in, **kw)
    torch.cuda.synchronize()
    r64 = lambda t, *s: t.bfloat16().double().reshape(*s)
    M, N = L * B, nd * k * d
    x, w, du = r64(X, M, d_in), r64(W, N, d_in), r64(sc["dU"], M, N)
    close(fw["U"].reshape(M, N), x, w.t())
    close(bw["dW"].reshape(N, d_in), du.t(), x)
    add = sc["dxh"].double().sum(2).reshape(M, d_in) if k == 3 else 0.0
    ref = du @ w + add
    bound = (N / 8 + 16) * 2.0 ** -24 * (du.abs() @ w.abs() + (add.abs() if k == 3 else 0.0))
    assert bool(((bw["dX"].reshape(M, d_in).double() - ref).abs() <= bound).all())
