"""Up to 16 token rows (weight-streaming projections fed U as parts) against the
oracle: windows of 1 to 16 tokens and decoding steps, over adapter ranks on both
sides of 32, target subsets, no adapter, a short prefix (attention without a
merge) and a long one (the merge forms the output adapter's parts, one per
head), head sizes 64 and 128, biases, a down projection whose K is split over
workgroups (K >= 4096 over few workgroups) and one whose last part is short."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, oracle_window, run_gpu_window
from tests.test_gpu_decode import _check_decode

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

S64 = dict(n_layers=2, d_model=640, n_q_heads=10, n_kv_heads=2, head_dim=64, d_ffn=4160)   # 65 pairs of k-steps
S128 = dict(n_layers=2, d_model=1152, n_q_heads=7, n_kv_heads=1, head_dim=128, d_ffn=4480)
ALL = syn.TARGETS
WINDOWS = {
    "n1_r16": (1, S64, 16, ALL),
    "n2_r40": (2, S128, 40, ALL),
    "n7_r8_vod": (7, S64, 8, ("v", "o", "down")),
    "n12_r64": (12, S128, 64, ALL),
    # 13 rows and more with large adapters on gate/up: the kernels of larger counts
    "n13_r64": (13, S128, 64, ALL),
    "n14_r24_up": (14, S128, 24, ("up", "down")),
    "n16_r64": (16, S128, 64, ALL),
    # (too small an adapter: d = 640 has two parts of 2 x 16 columns)
    "n16_r16": (16, S64, 16, ALL),
    "n4_none": (4, S128, 16, ()),
    "n5_none": (5, S128, 16, ()),
    "n13_none": (13, S64, 16, ()),
    "n5_r24_kg": (5, S128, 24, ("k", "gate")),
}


@pytest.mark.parametrize("name", list(WINDOWS))
def test_few_row_windows(name):
    from synthetic.device import build_case
    n, dims, rank, targets = WINDOWS[name]
    wl = syn.WORKLOADS["qwen7b_16k"].with_dims(**dims).with_window(n_tokens=n, l0=0, h=2)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=tuple(targets))
    print(f"[case] few rows {name}", flush=True)
    case = build_case(wl, 67, with_bias=True)
    ctx = run_gpu_window(case)
    for _ in range(3):   # arrival counters are back at zero after every launch
        run_gpu_window(case, ctx=ctx)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"few {name}")


@pytest.mark.parametrize("n,m,shape", [(100, 3, S64), (100, 16, S128), (1500, 1, S64), (1500, 16, S128)])
def test_few_row_decoding(n, m, shape):
    _check_decode(31, n, m, 1, base="qwen7b_16k", shape=shape)
