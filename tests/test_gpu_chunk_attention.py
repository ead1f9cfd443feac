"""Key-split attention under whole query blocks (17 and more new tokens over a
long prefix) against the oracle: one and two query blocks, a last key range past
the earlier block's last key, head sizes 64 and 128, group sizes 6, 7 and 1,
page sizes 16 and 8, and a prefix whose tiles do not divide by the splits."""
import pytest

from tests.test_gpu_decode import _check_decode

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "m17_hd64": (2031, 17, dict(n_layers=2, d_model=768, n_q_heads=12, n_kv_heads=2, head_dim=64, d_ffn=1024), 16),
    "m129_hd128": (2300, 129, dict(n_layers=2, d_model=512, n_q_heads=7, n_kv_heads=1, head_dim=128, d_ffn=1024), 16),
    # the second block's tokens fill a tile that the first block's rows never see
    "m200_hd64_page8": (2040, 200, dict(n_layers=2, d_model=512, n_q_heads=4, n_kv_heads=4, head_dim=64,
                                        d_ffn=1024), 8),
}


@pytest.mark.parametrize("name", list(CASES))
def test_chunk_over_a_long_prefix(name):
    n, m, shape, page = CASES[name]
    _check_decode(23, n, m, 1, base="qwen7b_16k", shape=shape, page_size=page)
