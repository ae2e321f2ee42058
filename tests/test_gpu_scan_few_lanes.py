"""Scans of few lanes against the same sequences inside a larger batch, bit for
bit: the forward in two waves (at most 256 workgroups of 64 units) against the
one-wave narrow ring, the time-parallel scans in 32-lane workgroups against
64-lane ones (same chunks), and the gated backward of under 8,192 lanes against
the sequential kernel."""
import pytest
import torch

from paper_1709_02755_amd import sru

pytestmark = pytest.mark.gpu


def inputs(L, B, d_in, d, nd, masked, seed=0):
    k = 3 if d_in == d else 4
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    mask = None
    if masked:  # padding anywhere, not only at the end
        mask = (torch.rand((L, B), generator=g, device="cuda") < 0.3).to(torch.uint8)
    return dict(U=rand(L, B, nd, k, d), X=rand(L, B, d_in), p=[rand(nd, d) * 0.5 for _ in range(4)],
                c0=rand(B, nd * d), mask=mask, dH=rand(L, B, nd * d), dc=rand(B, nd * d))


def first(t, B, dim=1):
    return None if t is None else t.narrow(dim, 0, B).contiguous()


# one group of 16 steps less, exact and more, rings of 3, 4 and 5 groups
@pytest.mark.parametrize("L", [1, 15, 16, 17, 33, 64, 79, 81])
@pytest.mark.parametrize("direction,d_in,masked,reset_new", [
    (sru.DIR_FWD, 64, False, False), (sru.DIR_REV, 64, True, True), (sru.DIR_BI, 96, True, False)])
def test_forward_two_waves(L, direction, d_in, masked, reset_new):
    d, nd = 64, 2 if direction == sru.DIR_BI else 1
    Bl, Bs = 320 // nd, 256 // nd  # workgroups: one per (sequence, direction)
    a = inputs(L, Bl, d_in, d, nd, masked)
    kw = dict(direction=direction, reset_new=reset_new, highway_scale=1.3)

    def run(B):
        out = dict(H=torch.empty((L, B, nd * d), device="cuda"),
                   C=torch.empty((L, B, nd * d), device="cuda"),
                   c_last=torch.empty((B, nd * d), device="cuda"),
                   H_bf16=torch.empty((L, B, nd * d), device="cuda", dtype=torch.bfloat16))
        return sru.scan_forward(first(a["U"], B), first(a["X"], B), *a["p"],
                                c0=first(a["c0"], B, 0), mask=first(a["mask"], B), out=out, **kw)

    large, small = run(Bl), run(Bs)
    torch.cuda.synchronize()
    for n in ("H", "C", "H_bf16"):
        assert torch.equal(small[n], first(large[n], Bs)), n
    assert torch.equal(small["c_last"], first(large["c_last"], Bs, 0))


# 128 lane groups against 256: steps below, at and past one block of 16 chunks
# of 8 (backward) or 12 (linear forward) steps, and past two
@pytest.mark.parametrize("L", [2, 9, 127, 128, 129, 200, 300])
@pytest.mark.parametrize("linear,masked,reset_new", [(False, True, False), (False, False, True),
                                                     (True, True, False)])
def test_time_parallel_half_lanes(L, linear, masked, reset_new):
    d, Bl, Bs = 256, 64, 32
    a = inputs(L, Bl, d, d, 1, masked, seed=L)
    kw = dict(linear=linear, reset_new=reset_new)

    def run(B):
        fw = sru.scan_forward(first(a["U"], B), first(a["X"], B), *a["p"], c0=first(a["c0"], B, 0),
                              mask=first(a["mask"], B), **kw)
        bw = sru.scan_backward(first(a["U"], B), first(a["X"], B), fw["C"], first(a["dH"], B),
                               *a["p"], c0=first(a["c0"], B, 0), dc_last=first(a["dc"], B, 0),
                               mask=first(a["mask"], B), **kw)
        return fw, bw

    (fl, bl), (fs, bs) = run(Bl), run(Bs)
    torch.cuda.synchronize()
    for big, small, names in ((fl, fs, ("H", "C")), (bl, bs, ("dU", "dxh"))):
        for n in names:
            assert torch.equal(small[n], first(big[n], Bs)), n
    assert torch.equal(bs["dc0"], first(bl["dc0"], Bs, 0))


# fewer than 8,192 lanes: chunks of 8 steps carried in order, against the
# sequential kernel of 65,536 lanes; d off the 32-lane groups, steps at the
# edges of a chunk and of a block of 16 chunks
@pytest.mark.parametrize("L", [1, 7, 8, 9, 17, 127, 128, 129, 261])
@pytest.mark.parametrize("direction,d_in,masked,reset_new", [
    (sru.DIR_FWD, 75, False, False), (sru.DIR_REV, 75, True, True),
    (sru.DIR_BI, 96, True, False), (sru.DIR_BI, 75, False, True)])
def test_backward_few_lanes(L, direction, d_in, masked, reset_new):
    d, nd = 75, 2 if direction == sru.DIR_BI else 1
    Bl, Bs = -(-65536 // (nd * d)), 5
    a = inputs(L, Bl, d_in, d, nd, masked, seed=L)
    kw = dict(direction=direction, reset_new=reset_new, highway_scale=1.3)

    def run(B, C):
        return sru.scan_backward(first(a["U"], B), first(a["X"], B), C, first(a["dH"], B), *a["p"],
                                 c0=first(a["c0"], B, 0), dc_last=first(a["dc"], B, 0),
                                 mask=first(a["mask"], B), **kw)

    C = sru.scan_forward(a["U"], a["X"], *a["p"], c0=a["c0"], mask=a["mask"], **kw)["C"]
    large, small = run(Bl, C), run(Bs, first(C, Bs))
    torch.cuda.synchronize()
    for n in ("dU", "dxh"):
        if large.get(n) is not None:
            assert torch.equal(small[n], first(large[n], Bs)), n
    assert torch.equal(small["dc0"], first(large["dc0"], Bs, 0))
    # the bias sums, in another order: fp32 sums of n = L * Bs values are within
    # n units in the last place of the sum of their magnitudes
    k = 4 if d_in != d else 3
    du = small["dU"].double().reshape(L, Bs, nd, k, d)
    n = L * Bs
    for name, i in (("db_f", 1), ("db_r", 2)):
        want = du[:, :, :, i].sum(dim=(0, 1))
        tol = n * 2.0**-23 * du[:, :, :, i].abs().sum(dim=(0, 1)) + 1e-30
        assert ((small[name].double() - want).abs() <= tol).all(), name
