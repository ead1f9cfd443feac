"""Long windows whose 256x256 tiles leave a last round at most half full, against
the oracle: gate/up with its last panels on 128x128 tiles (a token tail of less
than 128 rows, a last panel half empty because d_ffn is a multiple of 64 only,
adapters on both, one or neither of gate and up), and a down projection whose
few leftover tiles are split into more than two K-parts, over one round and two.  Bounds: the ideal-bf16
model on the same inputs (tests/helpers.py).  The tile counts are those of 256
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
    # down: 9 x 32 tiles = 1 round + 32 tiles, in 4 K-parts of 8 slices
    "down_parts": (2100, dict(NARROW, d_model=8192, d_ffn=2048), 16, ("q", "down")),
    # down: 9 x 16 tiles, more than half a round, in 3 K-parts of 32 slices over two rounds
    "down_two_rounds": (2100, dict(NARROW, d_model=4096, d_ffn=6144), 16, ("q", "down")),
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
