"""fp32 windows with a non-finite token among finite ones: what cannot depend on
the token keeps its value, as under the definition (a key that a query does not
see takes no part in it)."""
import dataclasses

import pytest

import synthetic as syn
from tests.helpers import TOL, gpu_kv, rel_to_rms, run_gpu_window

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(n, page, seed=73, rank=8, targets=("q", "v"), **dims):
    from synthetic.device import build_case
    wl = syn.WORKLOADS["tiny_f32"].with_dims(**{**dict(n_layers=3, n_q_heads=4, n_kv_heads=2, head_dim=64, d_model=264,
                                                       d_ffn=424), **dims}).with_window(n_tokens=n, l0=0, h=2)
    wl = dataclasses.replace(wl, lora_rank=rank, lora_targets=targets, page_size=page)
    return build_case(wl, seed)


# the non-finite token first, in the middle and last of its block of 16 queries,
# in a tile of 32 keys behind others, and on pages of one token
@pytest.mark.parametrize("n,t,page,hd", [(40, 21, 16, 64), (40, 32, 16, 128), (31, 15, 1, 64), (700, 541, 16, 64),
                                         (5, 4, 16, 128)])
def test_non_finite_token_leaves_earlier_tokens_alone(n, t, page, hd):
    print(f"[case] f32 non-finite token {t} of {n}, hd {hd}", flush=True)
    case = _case(n, page, head_dim=hd)
    run_gpu_window(case)
    torch.cuda.synchronize()
    ref = [case.hidden_out.cpu().numpy()] + [x for l in (0, 1) for x in gpu_kv(case, l)]
    case.hidden_dev[t, 3] = float("inf")
    run_gpu_window(case)
    torch.cuda.synchronize()
    got = [case.hidden_out.cpu().numpy()] + [x for l in (0, 1) for x in gpu_kv(case, l)]
    for g, r in zip(got, ref):
        # (the block's keys are added in another order where a value is not finite)
        assert rel_to_rms(g[:t], r[:t]) <= TOL["f32"]
        assert (g[:t // 16 * 16] == r[:t // 16 * 16]).all()
    assert not torch.isfinite(case.hidden_out[t:]).any(dim=1).any()   # every later token sees it


# ranks that leave rows of the adapter's 16-row block unused, and one that fills it
@pytest.mark.parametrize("rank", [1, 3, 13, 16])
def test_infinite_adapter_input_stays_infinite(rank):
    """U of the last rank row overflows to +Inf and its factor is positive: V is
    +Inf, not the NaN of an unused row's zero factor times that U."""
    print(f"[case] f32 infinite U, rank {rank}", flush=True)
    case = _case(20, 16, rank=rank, targets=("v",))
    case.hidden_dev.fill_(1.0)
    a, b = case.lora_dev[0]["targets"]["v"]
    a[rank - 1] = 3e38
    b[:, rank - 1] = 0.5
    run_gpu_window(case, h=1, hidden_out=False)
    torch.cuda.synchronize()
    k, v = gpu_kv(case, 0)
    assert (v == float("inf")).all()
