"""fp32 gate/up with both adapters' rank rows in one 16-row block (rank <= 8)
against the oracle: both, one or neither of gate and up adapted, ranks 1, 3, 8 and
9 (the last past the packing), on each of the three tile sizes.  Tolerance: the
repository's fp32 bound (1e-4)."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, oracle_window, run_gpu_window

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "r8_gate": (40, 8, ("gate",), 424),
    "r3_up_2x2": (700, 3, ("up", "down"), 424),
    "r1_both_4x4": (700, 1, ("gate", "up"), 1512),
    "r8_up_4x4": (700, 8, ("up",), 1512),
    "r8_neither": (40, 8, ("q", "down"), 424),
    "r9_both": (40, 9, ("gate", "up"), 424),
}


@pytest.mark.parametrize("name", list(CASES))
def test_f32_gate_up_adapters(name):
    from synthetic.device import build_case
    n, rank, targets, f = CASES[name]
    dims = dict(n_layers=2, d_model=136, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ffn=f)
    wl = syn.WORKLOADS["tiny_f32"].with_dims(**dims).with_window(n_tokens=n, l0=0, h=2)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=targets)
    print(f"[case] f32 gate/up {name}", flush=True)
    case = build_case(wl, 59)
    run_gpu_window(case)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"f32 gate/up {name}")
