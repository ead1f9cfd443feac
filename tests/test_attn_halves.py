"""Attention over windows with few query blocks, whose long blocks take their keys
in two parts: the work map and its rule on the host, and windows against the
oracle (an odd tile count, so that a second part begins inside a query block; head
sizes 64 and 128; pages of 16 and 8; a last block of one row)."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, oracle_window, run_gpu_window
from tests.test_schedule_host import _build_and_run

CASES = {
    "hd64": (2900, dict(n_layers=3, d_model=768, n_q_heads=12, n_kv_heads=2, head_dim=64, d_ffn=1024), 16),
    "hd128_page8": (2945, dict(n_layers=3, d_model=256, n_q_heads=12, n_kv_heads=2, head_dim=128, d_ffn=512), 8),
    "group7": (2113, dict(n_layers=3, d_model=256, n_q_heads=28, n_kv_heads=4, head_dim=64, d_ffn=512), 16),
}


def test_every_part_of_every_block_once(tmp_path):
    assert _build_and_run(tmp_path, "attn_halves_check") > 10000


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_window_with_two_key_parts(name):
    torch = pytest.importorskip("torch")
    from synthetic.device import build_case
    n, dims, page = CASES[name]
    wl = syn.WORKLOADS["qwen7b_16k"].with_dims(**dims).with_window(n_tokens=n, l0=1, h=1)
    wl = dataclasses.replace(wl, lora_rank=16, lora_targets=("q", "v"), page_size=page)
    print(f"[case] two key parts {name}", flush=True)
    case = build_case(wl, 71, with_bias=True)
    run_gpu_window(case)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"two key parts {name}")
