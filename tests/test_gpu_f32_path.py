"""The fp32 path at the edges of its tiles against the oracle: token counts
around the 16- and 32-token tiles and one, adapter ranks on both sides of the
fused 16-row block (odd ones among them), widths that are only multiples of 8,
head sizes 64 and 128, tile counts that take the 4 x 4-block kernel, other page
sizes, and a window without hidden_out (K/V of its last layer only).

Tolerance: the repository's fp32 bound (1e-4); every sum is fp32 over at most
a few thousand terms, so errors near 1e-6 are expected."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import assert_window_parity, bits_equal, oracle_window, run_gpu_window

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BASE = dict(n_layers=3, d_model=264, n_q_heads=4, n_kv_heads=2, head_dim=64, d_ffn=424)
CASES = {
    "n1_r8": (1, 8, 16, {}),
    "n15_r16": (15, 16, 16, {}),
    "n17_r17": (17, 17, 16, {}),
    "n33_r5_page1": (33, 5, 1, dict(head_dim=128, n_q_heads=3, n_kv_heads=1)),
    "n129_r64": (129, 64, 16, dict(head_dim=128)),
    # (n / 32) x (rows / 32, gate/up rows / 16) tiles past 2048: 4 x 4 blocks
    "big_gateup_r8": (700, 8, 16, dict(d_model=136, d_ffn=1512)),
    "big_all_r33": (1490, 33, 48, dict(d_model=1416, n_q_heads=9, n_kv_heads=1, head_dim=128, d_ffn=712)),
}


def _case(name):
    from synthetic.device import build_case
    n, rank, page, dims = CASES[name]
    wl = syn.WORKLOADS["tiny_f32"].with_dims(**{**BASE, **dims}).with_window(n_tokens=n, l0=1, h=2)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=syn.TARGETS, page_size=page)
    print(f"[case] f32 path {name}", flush=True)
    return build_case(wl, 53, with_bias=True)


@pytest.mark.parametrize("name", list(CASES))
def test_f32_tile_edges(name):
    case = _case(name)
    run_gpu_window(case)
    torch.cuda.synchronize()
    out, kv = oracle_window(case)
    assert_window_parity(case, out, kv, label=f"f32 {name}")


@pytest.mark.parametrize("name", ["n17_r17", "big_gateup_r8", "big_all_r33"])
def test_f32_window_without_hidden_out_writes_the_same_cache(name):
    case = _case(name)
    run_gpu_window(case)
    torch.cuda.synchronize()
    k, v = case.k_pool.clone(), case.v_pool.clone()
    case.k_pool.fill_(0.0)
    case.v_pool.fill_(0.0)
    l1 = case.window.l0 + case.window.h
    run_gpu_window(case, hidden_out=False)
    torch.cuda.synchronize()
    rows = torch.from_numpy(case.block_table).cuda().long()
    for pool, ref in ((case.k_pool, k), (case.v_pool, v)):
        n = case.window.n_tokens // case.wl.page_size * case.wl.page_size   # whole pages
        got, want = pool[case.window.l0:l1][:, rows], ref[case.window.l0:l1][:, rows]
        full = n // case.wl.page_size
        assert bits_equal(got[:, :full].contiguous(), want[:, :full].contiguous())
