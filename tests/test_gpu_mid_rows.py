"""The bf16 path at 17 to about a thousand tokens (K-split 128-row tiles and
their reductions) against the oracle at the edges of its tiles: 17, 64/65,
128/129 and 256/257 tokens, the switch from one to two tokens per reduction
thread (512/513), the last count before the 256x256 tiles take over and the
first after it, adapter ranks 8 to 64 on target subsets (adapter columns that
end inside a row tile), d_ffn a multiple of 64 only, head sizes 64 and 128,
biases, and a row wider than one thread's share.  Bounds: the ideal-bf16 model
on the same inputs (tests/helpers.py)."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, oracle_window, run_gpu_window

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

S64 = dict(n_layers=3, d_model=768, n_q_heads=12, n_kv_heads=2, head_dim=64, d_ffn=2112)
S128 = dict(n_layers=3, d_model=1152, n_q_heads=7, n_kv_heads=1, head_dim=128, d_ffn=1088)
WIDE = dict(n_layers=3, d_model=5248, n_q_heads=2, n_kv_heads=2, head_dim=128, d_ffn=512)
# 2 d_ffn / 256 = 171 row tiles: three token tiles (768) are past two rounds of 256 CUs
TALL = dict(n_layers=3, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128, d_ffn=21888)
ALL = syn.TARGETS
CASES = {
    "n17": (17, S64, 16, ALL),
    "n64_r8_qv": (64, S128, 8, ("q", "v")),
    "n65_r24": (65, S64, 24, ALL),
    "n128_r64": (128, S128, 64, ALL),
    "n129_none": (129, S64, 16, ()),
    "n256_r32_kgu": (256, S128, 32, ("k", "gate")),
    "n257_r8_od": (257, S64, 8, ("o", "down")),
    "n513_r48": (513, S128, 48, ALL),
    "n40_wide": (40, WIDE, 16, ALL),
    "n512_tall": (512, TALL, 16, ("up", "down")),
    # two layers on either side of the line that the adapters' deltas draw (rank 64 on all)
    "n2900_r64": (2900, S64, 64, ALL),
    "n4400_r64": (4400, S64, 64, ALL),
    "n513_tall": (513, TALL, 16, ("up", "down")),
}


@pytest.mark.parametrize("name", list(CASES))
def test_mid_rows_tile_edges(name):
    from synthetic.device import build_case
    n, dims, rank, targets = CASES[name]
    wl = syn.WORKLOADS["qwen7b_16k"].with_dims(**dims).with_window(n_tokens=n, l0=1, h=2)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=tuple(targets))
    print(f"[case] mid rows {name}", flush=True)
    case = build_case(wl, 61, with_bias=True)
    run_gpu_window(case)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"mid {name}")
