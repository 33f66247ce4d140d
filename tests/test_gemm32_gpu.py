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
    # chains of 256 rows, 32 of them per split, 4 splits: rounding grows at
    # most like the square root of a 2048-term chain, 2^-24 sqrt(2048) = 2.7e-6
    assert err < 2.7e-6
    plan.close()


def _independent_steps(cell, T, B, I, H):
    """Inputs whose steps do not depend on each other (W_h = 0, the gate that
    carries the state closed), h, and dz of the input and the recurrent half
    in closed form and float64: dW = [X; Hprev]^T DZ."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    G = 4 if cell == "lstm" else 3
    uniform = lambda a, *s: (torch.rand(*s, device="cuda", generator=g) * 2 - 1) * a
    x = torch.randn(T, B, I, device="cuda", generator=g)
    dy = torch.randn(T, B, H, device="cuda", generator=g)
    h0 = torch.randn(1, B, H, device="cuda", generator=g)
    Wt = torch.zeros(I + H, G * H, device="cuda")
    Wt[:I] = uniform(I ** -0.5, I, G * H)
    Wt[:I, H:2 * H] = 0
    bias = torch.zeros(4 * H, device="cuda")
    bias[H:2 * H] = -100.0          # LSTM: f = 0; GRU: u = 0
    if cell == "gru":
        bias[3 * H:] = uniform(1.0, H)
    x2, dh = x.double().view(T * B, I), dy.double().view(T * B, H)
    z, zero = x2 @ Wt[:I].double(), torch.zeros(T * B, H, device="cuda", dtype=torch.float64)
    if cell == "lstm":
        i, gg, o = torch.sigmoid(z[:, :H]), torch.tanh(z[:, 2 * H:3 * H]), torch.sigmoid(z[:, 3 * H:])
        tc = torch.tanh(i * gg)
        dc = dh * o * (1 - tc * tc)
        h = o * tc
        dzx = dzh = torch.cat([dc * gg * i * (1 - i), zero, dc * i * (1 - gg * gg), dh * tc * o * (1 - o)], 1)
    else:
        r, bhn = torch.sigmoid(z[:, :H]), bias[3 * H:].double()
        h = torch.tanh(z[:, 2 * H:] + r * bhn)
        dn = dh * (1 - h * h)
        dr = dn * bhn * r * (1 - r)
        dzx, dzh = torch.cat([dr, zero, dn], 1), torch.cat([dr, zero, dn * r], 1)
    c = lambda a: a.cpu().numpy()
    inp = dict(x=c(x), seq_len=np.full(B, T, np.int32), W=[c(Wt)], bias=[c(bias)], dy=c(dy), h0=c(h0), c0=None,
               dhT=None, dcT=None)
    return inp, h.view(T, B, H), dzx, dzh


# (64x64 tiles of one, of several splits and of several spans per split; then
# 128x128 tiles, the second operand's row tiles after a ragged first one, the
# GRU's shifted block on them)
@pytest.mark.parametrize("cell,T,B,I,H", [("lstm", 25, 64, 64, 512), ("lstm", 100, 64, 64, 512),
                                          ("lstm", 100, 64, 256, 256), ("gru", 40, 64, 64, 256),
                                          ("lstm", 256, 128, 516, 512), ("gru", 256, 128, 772, 512)])
def test_float32_dw_error(cell, T, B, I, H):
    """Both halves of dW against float64 products (Hprev from the library's own
    h, the operand it multiplies), with a bound on the error of the sums.  A
    float32 chain of n independent terms is off by 2.5e-8 sqrt(n / 2) of its
    2-norm (a rounding is off by 2.5e-8 of its result, root mean square;
    partial sum k holds k / n of the variance): 2.8e-7 for the 256-row chains,
    2.0e-7 for the sum over up to 128 of them.  dz itself: z from a chain of up
    to 772 terms, 2.8e-7 of its size and with a derivative of about one, and
    the activations and their products, some 2e-7."""
    import torch
    inp, h, dzx, dzh = _independent_steps(cell, T, B, I, H)
    dc = DeviceCase(inp, H, I, 1, "f32", cell=cell)
    plan = dc.plan()
    assert plan.geometry()["dw_in_place"] == [True]
    dc.fwd(plan)
    dc.bwd(plan)
    assert plan.status_sync() == 0
    plan.close()
    assert (dc.y - h).abs().max().item() < 1e-5
    hp = torch.cat([dc.h0, dc.y[:-1]]).double().view(T * B, H)
    ref_x, ref_h = dc.x.double().view(T * B, I).t() @ dzx, hp.t() @ dzh
    for half, got, ref in (("x", dc.dW[0][:I].double(), ref_x), ("h", dc.dW[0][I:].double(), ref_h)):
        err = ((got - ref).norm() / ref.norm()).item()
        say(f"[gemm32] {cell} dW_{half} over {T * B} rows: relative error {err:.2e}")
        assert err < (2.8e-7 ** 2 + 2.0e-7 ** 2 + 2.8e-7 ** 2 + 2e-7 ** 2) ** 0.5


@pytest.mark.parametrize("cell", ["lstm", "gru"])
def test_float32_dw_past_two_gib_takes_the_transposes(cell):
    """H = 512, B = 64, T_max = 4096: the dz rows of the row capacity reach
    2 GiB, past the 32-bit offsets of the product over rows, so the plan takes
    the gather-transposes and the split-K product of the copies (the GRU's in
    three parts).  Short lengths; every output against the oracle."""
    w = W(f"g32_{cell}_b64_i16_h512_t4096", B=64, I=16, H=512, T_max=4096, dtype="f32", len_lo=0, len_hi=5,
          cell=cell, random_state=True, seed=421)
    say(f"[gemm32] {w.name}")
    inp = wl.generate(w)
    dc = DeviceCase(inp, w.H, w.I, 1, "f32", cell=cell)
    plan = dc.plan()
    assert plan.geometry()["dw_in_place"] == [False]
    dc.fwd(plan)
    dc.bwd(plan)
    assert plan.status_sync() == 0
    res = dc.results()
    plan.close()
    errs, bad = compare(res, oracle_reference(inp, 1, "f32", cell=cell), TOL["f32"])
    say(f"    errors {errs}")
    assert not bad, bad
