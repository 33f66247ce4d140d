"""GPU test of the c values rebuilt for swapped-in chunks: a swapped stack
gives the resident stack's results bitwise, c rebuilt or swapped with the
gates, at the edges of the chunks (a chunk of one step, a last chunk cut short, rows that end on a chunk's first
and last step, rows that never start, random entering states in two layers)."""
import numpy as np
import pytest

from paper_1805_01772_amd import workloads as wl
from paper_1805_01772_amd.lstmloop import Plan
from paper_1805_01772_amd.runner import DeviceCase
from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,layers,B,H,T,C", [("f32", 1, 17, 64, 13, 1), ("f32", 2, 20, 32, 31, 4),
                                                  ("bf16", 1, 33, 64, 24, 6), ("bf16", 1, 130, 128, 22, 3),
                                                  # either side of 3 MiB a chunk, from where c is rebuilt
                                                  ("f32", 1, 64, 512, 23, 4), ("f32", 2, 64, 512, 23, 5),
                                                  ("bf16", 1, 160, 1024, 11, 1), ("bf16", 2, 80, 512, 17, 4)])
def test_swapped_stack_bitwise_at_chunk_edges(dtype, layers, B, H, T, C, monkeypatch):
    monkeypatch.setenv("LSTMLOOP_WAVEFRONT", "off")
    w = wl.Workload("rebuild", B=B, I=24, H=H, T_max=T, dtype=dtype, layers=layers, len_lo=0, len_hi=T,
                    w_scale=0.3, random_state=True, seed=77)
    inp = wl.generate(w)
    edges = [0, 1, C, C + 1, 2 * C, 3 * C, T - 1, T]
    inp["seq_len"][:len(edges)] = np.minimum(edges, T)
    say(f"[spill] rebuilt c, {dtype}, {layers} layer(s), B={B} H={H} T={T} chunks of {C}")
    outs = []
    for kw in ({}, dict(spill=1, spill_chunk_steps=C, device_stack_budget_bytes=1)):
        dc = DeviceCase(inp, H, 24, layers, dtype)
        plan = dc.plan(**kw)
        for _ in range(2):
            dc.fwd(plan)
            dc.bwd(plan)
        assert plan.status_sync() == 0
        outs.append(dc.results())
        plan.close()
    for k in ("y", "hT", "cT", "dx", "dh0", "dc0"):
        np.testing.assert_array_equal(outs[0][k], outs[1][k])
    for a, b in zip(outs[0]["dW"] + outs[0]["dbias"], outs[1]["dW"] + outs[1]["dbias"]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("layers,C", [(1, 1), (2, 4)])
def test_swapped_stack_stays_within_its_budget(layers, C):
    """The plan's device stack is the budget's chunk slots and the h history,
    whatever the number of chunks: nothing grows with T_max beside them."""
    B, H, T, R = 16, 64, 200, 5
    slots = R * C * B * 5 * H * 4
    say(f"[spill] device bytes, {layers} layer(s), chunks of {C}")
    with Plan(T, B, 32, H, layers=layers, dtype="f32", spill=1, spill_chunk_steps=C,
              device_stack_budget_bytes=slots) as plan:
        assert plan.stack_bytes()[0] == layers * (slots + T * B * H * 4)
