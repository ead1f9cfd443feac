"""crf_layer_drift over the forms its kernel treats apart, against fp64 numpy:
tensors that do not start on 16 bytes, chunk remainders, more versions than one
group of four, fp32 and bf16, and more chunks than workgroups.  Both sides sum
exact differences in fp64; the outputs are fp32 (2^-24 relative)."""
import numpy as np
import pytest

import synthetic as syn
from tests.helpers import cdims

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (workload, dims, rank, targets, versions, element offset of every tensor)
CASES = {
    "f32_r3_v5": ("tiny_f32", dict(n_layers=3), 3, ("q", "down"), 5, 0),
    "f32_r3_odd": ("tiny_f32", dict(n_layers=3), 3, ("q", "down"), 2, 1),
    "bf16_r8_v1_odd": ("qwen15b_4k", dict(n_layers=2), 8, ("k", "o"), 1, 3),
    "bf16_r16_v6": ("qwen15b_4k", dict(n_layers=5), 16, syn.TARGETS, 6, 0),
    "bf16_r24_chunks": ("qwen15b_4k", dict(n_layers=12, d_ffn=8896), 24, syn.TARGETS, 2, 0),
}


@pytest.mark.parametrize("per_layer_only", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_drift_chunk_forms(name, per_layer_only):
    import paper_2609_30884_amd as crf
    base, kw, rank, targets, V, off = CASES[name]
    dims = syn.WORKLOADS[base].with_dims(**kw).dims
    dt = torch.bfloat16 if dims.dtype == "bf16" else torch.float32
    N = dims.n_layers
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    print(f"[case] drift {name}", flush=True)

    def tensor(shape, std):
        n = shape[0] * shape[1]
        x = std * torch.randn(n + off, generator=g, device="cuda")
        return x.to(dt)[off:].view(shape)

    def state():
        out = []
        for _ in range(N):
            tg = {}
            for t in targets:
                d_out, d_in = dims.target_shape(t)
                tg[t] = (tensor((rank, d_in), 0.125), tensor((d_out, rank), 0.01))
            out.append({"rank": rank, "scale": 1.0, "targets": tg})
        return out

    cur, vers = state(), [state() for _ in range(V)]
    anchors = [(3 * l + 1) % V for l in range(N)]
    sens = torch.linspace(0.1, 2.0, N, device="cuda")
    drift, risk = torch.full((N,), -1.0, device="cuda"), torch.full((N,), -1.0, device="cuda")
    sq = torch.full((V * N,), -1.0, device="cuda")
    ctx = crf.Context(cdims(dims), 1, rank)
    arrays = crf.lora_array(cur, N), [crf.lora_array(v, N) for v in vers]
    for _ in range(6):   # more calls in flight than staging buffers
        crf.layer_drift(ctx, cdims(dims), *arrays, anchors, sens, drift, risk, sq, per_layer_only=per_layer_only)
    torch.cuda.synchronize()
    ref = np.zeros((V, N))
    for v in range(V):
        for l in range(N):
            for t in targets:
                for a, b in zip(cur[l]["targets"][t], vers[v][l]["targets"][t]):
                    ref[v, l] += float(((a.double() - b.double()) ** 2).sum())
    d = np.sqrt(ref[anchors, np.arange(N)] if per_layer_only else ref.sum(1)[anchors])
    tol = 2.0 ** -23   # one fp32 rounding of the output, with a factor of two
    assert np.allclose(sq.cpu().numpy().reshape(V, N), ref, rtol=tol, atol=0)
    assert np.allclose(drift.cpu().numpy(), d, rtol=tol, atol=0)
    assert np.allclose(risk.cpu().numpy(), d * sens.double().cpu().numpy(), rtol=tol, atol=0)
