"""GPU parity of the float32 products outside the recurrence (input
projection, dx, dW over rows) at the edges of their tiles: input widths that
are no multiple of the 64-column tile (two operands in one dW launch), row
counts around the 32-row k-tile and the 64-row tile, the 128x128 dW tile with
its two-level sums, the GRU's shifted candidate block.  Each case runs a whole
training step against the float64 oracle (1e-5)."""
import numpy as np
import pytest

from paper_1805_01772_amd import workloads as wl
from paper_1805_01772_amd.runner import DeviceCase
from _helpers import TOL, compare, oracle_reference, say

pytestmark = pytest.mark.gpu

W = wl.Workload
CASES = [W(f"g32_{cell}_b{B}_i{I}_h{H}_t{T}", B=B, I=I, H=H, T_max=T, dtype="f32", len_lo=lo, len_hi=T,
           cell=cell, random_state=True, seed=seed)
         for seed, (cell, B, I, H, T, lo) in enumerate([
             ("lstm", 1, 4, 32, 33, 33), ("lstm", 3, 68, 96, 21, 21), ("lstm", 64, 60, 64, 2, 1),
             ("lstm", 7, 132, 160, 9, 0), ("gru", 5, 12, 96, 13, 0), ("gru", 33, 100, 32, 4, 4),
             ("rnn", 9, 36, 224, 7, 0)], start=401)]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_float32_products_parity(w):
    say(f"[gemm32] {w.name}")
    inp = wl.generate(w)
    dc = DeviceCase(inp, w.H, w.I, 1, "f32", cell=w.cell)
    plan = dc.plan()
    assert plan.geometry()["dw_in_place"] == [True]
    dc.fwd(plan)
    dc.bwd(plan)
    assert plan.status_sync() == 0
    res = dc.results()
    plan.close()
    errs, bad = compare(res, oracle_reference(inp, 1, "f32", cell=w.cell), TOL["f32"])
    say(f"    errors {errs}")
    assert not bad, bad


def test_float32_dw_long_reduction():
    """dW over 32 768 rows on the 128x128 tiles (split, several two-level
    spans): against float64 products of the same operands, which a constant
    input makes cheap: with W_h = 0 and h0 = 0 every row's dz depends on its own
    x row only, so dW_x = X^T DZ with DZ = the gradient of one step's cell."""
    import torch
    T, B, I, H = 256, 128, 512, 512
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(T, B, I, device="cuda", generator=g)
    Wt = torch.zeros(I + H, 4 * H, device="cuda")
    Wt[:I] = (torch.rand(I, 4 * H, device="cuda", generator=g) * 2 - 1) / I ** 0.5
    Wt[:I, H:2 * H] = 0
    bias = torch.zeros(4 * H, device="cuda")
    bias[H:2 * H] = -100.0          # forget gate closed: f = 0, the steps are independent
    dy = torch.randn(T, B, H, device="cuda", generator=g)
    inp = dict(x=x.cpu().numpy(), seq_len=np.full(B, T, np.int32), W=[Wt.cpu().numpy()],
               bias=[bias.cpu().numpy()], dy=dy.cpu().numpy(), h0=None, c0=None, dhT=None, dcT=None)
    dc = DeviceCase(inp, H, I, 1, "f32")
    plan = dc.plan()
    dc.fwd(plan)
    dc.bwd(plan)
    assert plan.status_sync() == 0
    x2, w2 = x.double().view(T * B, I), Wt[:I].double()
    z = x2 @ w2
    i, gg, o = torch.sigmoid(z[:, :H]), torch.tanh(z[:, 2 * H:3 * H]), torch.sigmoid(z[:, 3 * H:])
    tc = torch.tanh(i * gg)
    dh = dy.double().view(T * B, H)
    dc1 = dh * o * (1 - tc * tc)
    dz = torch.cat([dc1 * gg * i * (1 - i), torch.zeros_like(i), dc1 * i * (1 - gg * gg), dh * tc * o * (1 - o)], 1)
    ref = x2.t() @ dz
    got = dc.dW[0][:I].double()
    err = ((got - ref).norm() / ref.norm()).item()
    say(f"[gemm32] dW over {T * B} rows: relative error {err:.2e}")
    # sums of 2048 terms, 8 of them per split, 4 splits: rounding grows like
    # the square root of the 2048-term chain, 2^-24 sqrt(2048) = 2.7e-6
    assert err < 2.7e-6
    plan.close()
