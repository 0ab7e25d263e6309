"""Windows of many rows (bf16, no threshold): runs of one, two and four chunks of keys per workgroup, scores that do not depend
on how the layers are cut into calls."""
import numpy as np
import pytest

import synth
from oracle import aircache_oracle as O
from tests import parity_util as P

pytestmark = pytest.mark.gpu


class _Prompt:
    """Random device tensors of one shape: L layers, B sequences, G query heads over each of hkv KV heads."""

    def __init__(self, L, B, hkv, G, d, n_vis, n_text, window, visual=False, spread=1.0, n_sys=9):
        import torch

        dev = torch.device("cuda:0")
        gen = torch.Generator(device=dev)
        gen.manual_seed(11)
        self.L, self.B, self.hkv, self.G, self.d, self.visual = L, B, hkv, G, d, visual
        n = n_sys + n_vis + n_text
        start = n_sys + n_vis - window if visual else n - window
        self.seqs = [synth.configs.Seq(n, n_sys, n_vis, start, window) for _ in range(B)]
        self.n_q = window if visual else n_text
        self.k = [torch.randn((B, hkv, n, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(L)]
        self.q = [(spread * torch.randn((B, hkv * G, self.n_q, d), generator=gen, device=dev)).to(torch.bfloat16) for _ in range(L)]

    def context(self, **tuning):
        import paper_2503_23956_amd as A

        s = self.seqs[0]
        cfg = A.make_config(n_layers=self.L, n_q_heads=self.hkv * self.G, n_kv_heads=self.hkv, head_dim=self.d, batch=self.B,
                            max_vis_len=s.vis_len, max_nonvis_len=s.seq_len - s.vis_len, max_window=s.win_len, max_decode_steps=1,
                            dtype=A.AIR_BF16, alpha=0.0, window_kind=A.AIR_WINDOW_VISUAL if self.visual else A.AIR_WINDOW_TEXT)
        ac = A.AirCache(cfg, "cuda:0")
        if tuning:
            ac.air_set_tuning(**tuning)
        return ac

    def score(self, ac, pieces=None):
        ac.air_reset()
        for l0, l1 in pieces or [(0, self.L)]:
            ac.air_score(l0, l1, self.q[l0:l1], self.k[l0:l1], self.k[l0:l1], self.seqs)
        return [ac.air_get_scores(l) for l in range(self.L)]

    def oracle(self, l, b, h):
        """fp64 importance of one unit."""
        s = self.seqs[b]
        q = self.q[l][b, h * self.G:(h + 1) * self.G].double().cpu().numpy()
        k = self.k[l][b, h:h + 1].double().cpu().numpy()
        seg = P.seg_of(s)
        return (O.layer_importance_visual_window(q, k, seg) if self.visual else O.layer_importance(q, k, seg, 0.0))[0][0]


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("L", [5, 16, 34])  # runs of one, two and four chunks of 256 keys; 34 layers take two launches
def test_scores_are_the_same_bits_however_the_layers_are_cut(L, d, visual):
    p = _Prompt(L, 6, 8, 2, d, 1000, 24, 20, visual)
    ac = p.context()
    want = p.score(ac)
    for (l, b, h) in [(0, 0, 0), (L // 2, 3, 5), (L - 1, 5, 7)]:
        np.testing.assert_allclose(want[l][b, h], p.oracle(l, b, h), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
    for pieces in ([(l, l + 1) for l in range(L)], [(3, L), (0, 3)]):
        assert all(np.array_equal(x, y) for x, y in zip(want, p.score(ac, pieces)))
    ac.close()
    ac = p.context(score_block_mb=2)
    assert all(np.array_equal(x, y) for x, y in zip(want, p.score(ac)))
    ac.close()
