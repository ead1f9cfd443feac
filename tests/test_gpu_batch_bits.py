"""A batch of several caches against its windows as separate calls and against the
batch run in order, bitwise, at sizes that take the large tiles with their last
rounds in K-parts (two, three, as many as fill the GPU) and attention's long
blocks in two key parts, next to mid-sized and few-row items."""
import pytest

import synthetic as syn
from tests.helpers import bits_equal, cdims
from tests.test_gpu_parity import _batched_cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WINDOWS = [syn.Window(2300, 3, 2), syn.Window(3000, 3, 1), syn.Window(5600, 8, 1), syn.Window(700, 26, 2),
           syn.Window(12, 3, 1)]


def test_batch_equals_separate_calls_and_in_order_run():
    import paper_2609_30884_amd as crf
    base, cases = _batched_cases(WINDOWS)
    cd = cdims(base.dims)
    ctx = crf.Context(cd, max(c.window.n_tokens for c in cases), base.lora_rank)
    w = crf.layer_weights_array(cases[0].weights_dev)
    las = [crf.lora_array(c.lora_dev, base.dims.n_layers) for c in cases]
    kvs = [crf.kv_cache(c.k_pool, c.v_pool, c.block_table_dev, c.window.n_tokens, base.page_size) for c in cases]
    its = [crf.window_item(c.hidden_dev, la, c.window.l0, c.window.h, kv, c.hidden_out)
           for c, la, kv in zip(cases, las, kvs)]

    def results(call):
        for c in cases:
            c.k_pool.zero_()
            c.v_pool.zero_()
            c.hidden_out.zero_()
        call()
        torch.cuda.synchronize()
        return [(c.hidden_out.clone(), c.k_pool.clone(), c.v_pool.clone()) for c in cases]

    def separate():
        for c, la, kv in zip(cases, las, kvs):
            crf.recompute_window(ctx, cd, c.hidden_dev, w, la, c.window.l0, c.window.h, kv, c.hidden_out)

    def in_order():   # timed batches run on one stream
        ctx.set_timing(True)
        crf.recompute_window_batched(ctx, cd, w, its)
        torch.cuda.synchronize()
        ctx.set_timing(False)
        ctx.read_timing()

    print("[case] batch bits", flush=True)
    ref = results(separate)
    for call in (in_order, lambda: crf.recompute_window_batched(ctx, cd, w, its)):
        for c, got, want in zip(cases, results(call), ref):
            assert all(bits_equal(g, r) for g, r in zip(got, want)), c.window
    assert ctx.device_errors() == 0
