"""Spans that leave 27 bits of a place behind (they fit the card's memory, so they are accepted): one unit, every key and query
but a few at zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _zeros(shape, need):
    import torch

    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip(f"needs {need / 1e9:.0f} GB of device memory")
    return torch.zeros(shape, dtype=torch.bfloat16, device="cuda:0")


@pytest.mark.parametrize("heads", [1, 16])
def test_window_far_behind_the_first_text_token(heads):
    # a window of 33 tokens behind 2^27 text tokens; 16 heads share one tensor (strides of zero between them), the window's queries
    # in front of those of other tokens at 2^27 places less
    import torch

    import paper_2503_23956_amd as A

    d, n_vis, W = 64, 70, 33
    n_text = 2 ** 27 + 40
    n = n_vis + n_text
    k = _zeros((1, 1, n, d), 100e9)
    q = torch.zeros((1, 1, n_text, d), dtype=torch.bfloat16, device="cuda:0")
    k[0, 0, :n_vis, 0] = torch.arange(n_vis, device="cuda:0") / 8  # logits of the visual keys: 0, 1/8, 2/8, ...
    q[0, 0, -W:, 0] = 8.0
    q[0, 0, :W + 40, 0] = -8.0
    s = [type("Seq", (), dict(seq_len=n, vis_start=0, vis_len=n_vis, win_start=n - W, win_len=W))]
    cfg = A.make_config(n_layers=1, n_q_heads=heads, n_kv_heads=1, head_dim=d, batch=1, max_vis_len=n_vis, max_nonvis_len=n_text, max_window=W,
                        max_decode_steps=1, dtype=A.AIR_BF16, alpha=0.0)
    ac = A.AirCache(cfg, "cuda:0")
    ac.air_score(0, 1, [q.expand(1, heads, n_text, d)], [k], [k], s)
    got = ac.air_get_scores(0)[0, 0]
    ac.close()
    del q, k, ac
    torch.cuda.empty_cache()
    e = np.exp(np.arange(n_vis) / 8)
    np.testing.assert_allclose(got, e / (e.sum() + W), rtol=1e-5)
