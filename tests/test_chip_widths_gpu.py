"""GPU parity of the loops at the widths between the powers of two.

XCD-local loops: bfloat16 widths of an odd number of 32 units, one and two
layers, one to four row tiles per XCD.  Chip-wide loops over their whole
range: widths between the powers of two (odd counts of 32 units: shares of the reduction of unequal
length, a last gradient column group that is half filled), and batches at the
edges of the row groups (32) and of the waves' shares (64, 128, 256)."""
import numpy as np
import pytest

from paper_1805_01772_amd import workloads as wl
from paper_1805_01772_amd.lstmloop import LL_EUNSUPPORTED, LoopError, Plan
from paper_1805_01772_amd.runner import DeviceCase
from _helpers import TOL, compare, oracle_reference, say
from test_parity_gpu import run_case

pytestmark = pytest.mark.gpu

W = wl.Workload
CASES = [W(f"chipw_{dtype}_b{B}_i{I}_h{H}_t{T}_l{L}", B=B, I=I, H=H, T_max=T, dtype=dtype, layers=L,
           len_lo=0, len_hi=T, random_state=True, seed=seed)
         for seed, (dtype, B, I, H, T, L) in enumerate([
             ("bf16", 1, 8, 1056, 6, 1), ("bf16", 33, 24, 1184, 5, 1), ("bf16", 64, 16, 1536, 5, 1),
             ("bf16", 65, 40, 1056, 5, 1), ("bf16", 128, 16, 2016, 4, 1), ("bf16", 129, 16, 1088, 5, 1),
             ("bf16", 256, 8, 1280, 4, 2), ("f32", 1, 4, 544, 6, 1), ("f32", 40, 20, 672, 6, 1),
             ("f32", 66, 12, 992, 4, 1), ("f32", 130, 8, 544, 5, 2), ("f32", 256, 8, 608, 4, 1),
             # eight and four shares of the forward's reduction at the full LDS, and their last batch
             ("bf16", 32, 8, 2048, 4, 1), ("bf16", 48, 8, 2048, 4, 1), ("f32", 32, 8, 1024, 4, 1),
             ("f32", 17, 8, 576, 5, 1)], start=301)]
# float32: the gradient's slices shared by four and by none either side of H = 768
CASES += [W(f"chipw_f32_b{B}_i8_h{H}_t{T}", B=B, I=8, H=H, T_max=T, dtype="f32", len_lo=0, len_hi=T,
            random_state=True, seed=seed)
          for seed, (B, H, T) in enumerate([(30, 768, 4), (5, 800, 5), (64, 1024, 4), (97, 896, 4)], start=361)]
# the forward's single row tile up to 16 rows, float32's sixteen waves for five to seven row groups
CASES += [W(f"chipw_{dtype}_b{B}_i8_h{H}_t{T}", B=B, I=8, H=H, T_max=T, dtype=dtype, len_lo=0, len_hi=T,
            random_state=True, seed=seed)
          for seed, (dtype, B, H, T) in enumerate([("bf16", 16, 2048, 5), ("bf16", 17, 1120, 4), ("f32", 16, 544, 5),
                                                   ("f32", 9, 1024, 5), ("f32", 160, 1024, 4), ("f32", 193, 736, 4),
                                                   ("f32", 225, 576, 4), ("f32", 129, 1024, 6)], start=371)]


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_chip_widths_parity(w, monkeypatch):
    monkeypatch.delenv("LSTMLOOP_LOOPS", raising=False)
    say(f"[chip widths] {w.name}")
    inp = wl.generate(w)
    geom = {}
    res, err = run_case(w, inp, geometry=geom)
    assert geom["loops"] == "chip", geom
    assert err == 0
    ref = oracle_reference(inp, w.layers, w.dtype)
    assert res["T_eff"] == ref["T_eff"]
    errs, bad = compare(res, ref, TOL[w.dtype])
    say(f"    errors {errs}")
    assert not bad, bad


ODD = [W(f"odd_bf16_b{B}_i{I}_h{H}_t{T}_l{L}", B=B, I=I, H=H, T_max=T, dtype="bf16", layers=L, len_lo=0,
         len_hi=T, random_state=True, seed=seed)
       for seed, (B, I, H, T, L) in enumerate([
           (1, 8, 32, 9, 1), (17, 24, 96, 11, 1), (130, 16, 160, 7, 2), (300, 8, 288, 5, 1), (40, 40, 608, 6, 2),
           (512, 8, 992, 3, 1)], start=331)]


@pytest.mark.parametrize("w", ODD, ids=[w.name for w in ODD])
def test_odd_widths_parity(w, monkeypatch):
    monkeypatch.delenv("LSTMLOOP_LOOPS", raising=False)
    say(f"[odd widths] {w.name}")
    inp = wl.generate(w)
    geom = {}
    res, err = run_case(w, inp, geometry=geom)
    assert geom["loops"] == "xcd", geom
    assert err == 0
    ref = oracle_reference(inp, w.layers, w.dtype)
    assert res["T_eff"] == ref["T_eff"]
    errs, bad = compare(res, ref, TOL[w.dtype])
    say(f"    errors {errs}")
    assert not bad, bad


@pytest.mark.parametrize("kw", [dict(cell=1), dict(cell=2), dict(cell=3), dict(cell=4, ponder_max=2),
                                dict(spill=1), dict(recompute=1)])
def test_odd_widths_refused_for_other_bodies_and_policies(kw):
    with pytest.raises(LoopError) as e:
        Plan(8, 4, 32, 96, dtype="bf16", **kw)
    assert e.value.status == LL_EUNSUPPORTED


@pytest.mark.parametrize("dtype,wide,narrow,B", [("bf16", 2048, 1056, 40), ("f32", 768, 544, 20)])
def test_wide_plan_runs_after_a_narrow_one_was_made(dtype, wide, narrow, B, monkeypatch):
    """Two live plans of the same kernels whose LDS sizes differ: making the
    narrower one takes nothing from the wider one (bitwise its own results)."""
    monkeypatch.delenv("LSTMLOOP_LOOPS", raising=False)
    say(f"[chip widths] {dtype} H = {wide} after H = {narrow}")
    w = W("wide", B=B, I=8, H=wide, T_max=4, dtype=dtype, len_lo=1, len_hi=4, random_state=True, seed=351)
    dc = DeviceCase(wl.generate(w), w.H, w.I, 1, dtype)
    with dc.plan() as plan:
        dc.fwd(plan)
        dc.bwd(plan)
        assert plan.status_sync() == 0
        first = dc.results()
        with Plan(4, B, 8, narrow, dtype=dtype) as other:
            assert plan.geometry()["loops"] == other.geometry()["loops"] == "chip"
            dc.fwd(plan)
            dc.bwd(plan)
            assert plan.status_sync() == 0
    again = dc.results()
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        np.testing.assert_array_equal(again[k], first[k], err_msg=k)
