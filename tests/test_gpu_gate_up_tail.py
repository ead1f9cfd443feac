"""Long windows whose 256x256 tiles leave a last round at most half full, against
the oracle: gate/up with its last panels on 128x128 tiles (a token tail of less
than 128 rows, a last panel half empty because d_ffn is a multiple of 64 only,
adapters on both, one or neither of gate and up).  Bounds: the ideal-bf16 model
on the same inputs (tests/helpers.py).  The tile counts are those of 256
compute units; with others the same shapes take other routes."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, oracle_window, run_gpu_window

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NARROW = dict(n_layers=3, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128)
CASES = {
    # 9 token tiles x 68 panels = 2 rounds + 100 tiles: 12 panels
    "tail_r32": (2049, dict(NARROW, d_ffn=8704), 32, syn.TARGETS),
    # 9 x 69 (the last half empty) = 2 rounds + 109 tiles: 13 panels
    "half_panel_gate": (2300, dict(NARROW, d_ffn=8768), 16, ("q", "gate")),
    "half_panel_none": (2300, dict(NARROW, d_ffn=8768), 16, ("v",)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_last_round_of_large_tiles(name):
    from synthetic.device import build_case
    n, dims, rank, targets = CASES[name]
    wl = syn.WORKLOADS["qwen7b_16k"].with_dims(**dims).with_window(n_tokens=n, l0=1, h=1)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=tuple(targets))
    print(f"[case] last round {name}", flush=True)
    case = build_case(wl, 67, with_bias=True)
    run_gpu_window(case)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"last round {name}")
