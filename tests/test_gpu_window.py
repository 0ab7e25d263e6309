"""Windows of many rows (bf16, no threshold): runs and parts of 512 to 2048 keys per workgroup, logits that outrun their reference,
scores that do not depend on how the layers are cut into calls, their error against fp64 and the statistics formed from them."""
import math

import numpy as np
import pytest

import synth
from oracle import aircache_oracle as O
from tests import parity_util as P

pytestmark = pytest.mark.gpu


def _part_keys(n_vis, units, most=2048, extra=8):
    """Keys of a workgroup as the launcher chooses them: least rounds of 512 workgroups times what a round costs."""
    groups = -(-n_vis // 64)
    cost = {g: -(-units * -(-groups // g) // 512) * (g + extra) for g in range(8, most // 64 + 1)}
    return 64 * min(cost, key=lambda g: (cost[g], -g))


def _run_keys(n_vis, units, rows):
    """Keys of a run of the first pass, by the units of the context and the rows of a unit."""
    return _part_keys(n_vis, units, 1536, 4) if rows <= 96 else _part_keys(n_vis, units)


def _share_rows(rows, runs):
    """Rows of a workgroup of the first pass: whole blocks of 32, dealt to as many workgroups as leave each a CU."""
    blocks = -(-rows // 32)
    return 32 * -(-blocks // max(1, min(256 // runs, blocks)))


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

    def context(self, alpha=0.0, **tuning):
        import paper_2503_23956_amd as A

        s = self.seqs[0]
        cfg = A.make_config(n_layers=self.L, n_q_heads=self.hkv * self.G, n_kv_heads=self.hkv, head_dim=self.d, batch=self.B,
                            max_vis_len=s.vis_len, max_nonvis_len=s.seq_len - s.vis_len, max_window=s.win_len, max_decode_steps=1,
                            dtype=A.AIR_BF16, alpha=alpha, window_kind=A.AIR_WINDOW_VISUAL if self.visual else A.AIR_WINDOW_TEXT)
        ac = A.AirCache(cfg, "cuda:0")
        if tuning:
            ac.air_set_tuning(**tuning)
        return ac

    def score(self, ac, pieces=None):
        ac.air_reset()
        for l0, l1 in pieces or [(0, self.L)]:
            ac.air_score(l0, l1, self.q[l0:l1], self.k[l0:l1], self.k[l0:l1], self.seqs)
        return [ac.air_get_scores(l) for l in range(self.L)]

    def oracle(self, l, b, h, alpha=0.0):
        """fp64 importance of one unit."""
        s = self.seqs[b]
        q = self.q[l][b, h * self.G:(h + 1) * self.G].double().cpu().numpy()
        k = self.k[l][b, h:h + 1].double().cpu().numpy()
        seg = P.seg_of(s)
        return (O.layer_importance_visual_window(q, k, seg) if self.visual else O.layer_importance(q, k, seg, alpha))[0][0]


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("L", [5, 16, 34])  # runs of 512, 1024 and 1024 keys; 34 layers take two launches
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


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("visual", [False, True])
@pytest.mark.parametrize("shape", ["rising", "falling", "peaks"])
@pytest.mark.parametrize("L", [1, 34])
def test_logits_that_outrun_their_reference(d, visual, shape, L):
    # raw logits that step by 240 (30 or 43 bits) every 64 keys, or stand 1600 above everything at single keys: a step's sums
    # pass their limit, references are raised and sums scaled, in runs of 512 and of 1024 keys.  Small whole numbers, so that
    # every logit is exact in fp32.
    import torch

    p = _Prompt(L, 6 if L > 1 else 1, 8 if L > 1 else 2, 2, d, 1000, 24, 20, visual)
    n0 = p.seqs[0].vis_start
    step = torch.arange(1000, device="cuda:0")
    lead = {"rising": 30 * (step // 64), "falling": 30 * (15 - step // 64), "peaks": torch.where(step % 97 == 90, 200, 0)}[shape]
    for x in (*p.k, *p.q):
        x.copy_(x.clamp(-2, 2).round())
    for l in range(L):
        p.k[l][..., 0] = 0.0
        p.k[l][:, :, n0:n0 + 1000, 0] = lead.to(torch.bfloat16)
        p.q[l][..., 0] = 8.0
    ac = p.context()
    got = p.score(ac)
    for (l, b, h) in [(0, 0, 0), (L - 1, p.B - 1, p.hkv - 1)]:
        np.testing.assert_allclose(got[l][b, h], p.oracle(l, b, h), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
    ac.close()


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("visual", [False, True])
@pytest.mark.parametrize("spread,bound", [(1.0, 1e-7), (5.0, 6e-7), (18.0, 1.5e-6)])
@pytest.mark.parametrize("L,B,run", [(2, 1, 512), (16, 16, 1152)])  # lanes with references of their own, references over the first keys of a run
def test_error_against_fp64(d, visual, spread, bound, L, B, run):
    # Relative 2-norm.  A logit near the maximum is about 4 spreads in size; its fp32 sum is rounded at partial sums of that size,
    # 4 spread 2^-24 = 2.4e-7 spread at the most for one row, and averages over the rows that share a key.  Sums from zero
    # with references near the maximum: 0.6e-7, 4.3e-7 and 8.7e-7 measured (with the logits of this kernel as with those of
    # the one before it); sums that start at minus the reference: 0.7e-7, 9.7e-7 and 4.0e-6.
    assert _run_keys(2304, L * B * 2, 7 * 32) == run
    p = _Prompt(L, B, 2, 7, d, 2304, 64, 32, visual, spread)
    ac = p.context()
    got = p.score(ac)
    ac.close()
    errs = []
    for l in (0, L - 1):
        for h in range(2):
            want = p.oracle(l, l % B, h)
            errs.append(np.linalg.norm(got[l][l % B, h] - want) / np.linalg.norm(want))
    assert math.sqrt(np.mean(np.square(errs))) <= bound, errs


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("n_vis", [63, 512, 545, 1025, 2049, 4160])  # less than a group, whole parts, parts with a remainder
@pytest.mark.parametrize("window,G", [(9, 4), (32, 7), (33, 7), (43, 6), (32, 16)])  # 36 to 512 rows: blocks of 16 and 32, groups of 256
def test_edges_of_parts_and_row_blocks(n_vis, window, G, d, visual):
    p = _Prompt(3, 2, 2, G, d, n_vis, 48, window, visual)
    ac = p.context()
    got = p.score(ac)
    one_by_one = p.score(ac, [(l, l + 1) for l in range(3)])  # (parts of 512 keys in both)
    ac.air_budget()
    s_t, s_k = ac.air_get_stats()
    ac.close()
    assert all(np.array_equal(x, y) for x, y in zip(got, one_by_one))
    for (l, b, h) in [(0, 0, 0), (2, 1, 1)]:
        np.testing.assert_allclose(got[l][b, h], p.oracle(l, b, h), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
    for b in range(2):  # strength and skewness of the scores that the call left
        want = [O.skewness(got[2][b, h].astype(np.float64)) for h in range(2)]
        np.testing.assert_allclose(s_t[b, 2], got[2][b].astype(np.float64).sum(axis=1).mean(), rtol=1e-12)
        np.testing.assert_allclose(s_k[b, 2], np.mean(want), rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("n_vis", [8192, 8193, 12289, 16385, 33000])  # 16, 17, 25, 33 and 65 runs
@pytest.mark.parametrize("window,G", [(9, 4), (33, 8)])
def test_spans_of_many_runs(n_vis, window, G, d, visual):
    # the partial sums of a row past the first sixteen, the unit's statistics from scores that are read in several turns
    p = _Prompt(2, 1, 1, G, d, n_vis, 48, window, visual)
    ac = p.context()
    got = p.score(ac)
    ac.air_budget()
    s_t, s_k = ac.air_get_stats()
    one_by_one = p.score(ac, [(l, l + 1) for l in range(2)])
    ac.close()
    assert all(np.array_equal(x, y) for x, y in zip(got, one_by_one))
    for l in range(2):
        np.testing.assert_allclose(got[l][0, 0], p.oracle(l, 0, 0), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
        np.testing.assert_allclose(s_t[0, l], got[l][0, 0].astype(np.float64).sum(), rtol=1e-12)
        np.testing.assert_allclose(s_k[0, l], O.skewness(got[l][0, 0].astype(np.float64)), rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("window,G", [(9, 4), (33, 8)])  # 36 rows: runs of at most 1536 keys, and 264 rows: two groups of rows
@pytest.mark.parametrize("n_vis,few,run", [(4160, 1088, 1088), (7290, 960, 1856), (8192, 1024, 2048)])
def test_parts_that_are_larger_in_one_call_than_layer_by_layer(n_vis, few, run, window, G, d, visual):
    # 128 units in one launch, four layer by layer: units of several runs and parts that are no power of two, and as large as LDS
    # takes.  Rows of a run in one workgroup, or dealt to several: 264 rows as 160 + 104 in calls of seven layers, 3 x 96 (the last 72) in calls
    # of five, blocks of 32 in calls of one.
    L, B = 32, 4
    assert (_part_keys(n_vis, L * B), _part_keys(n_vis, B)) == (run, 512)
    assert (_run_keys(n_vis, L * B, 36), _run_keys(n_vis, L * B, 96), _run_keys(n_vis, L * B, 97)) == (few, few, run)
    assert [_share_rows(264, n * B * -(-n_vis // run)) for n in (32, 7, 5, 1)] == [288, 160, 96, 32]
    p = _Prompt(L, B, 1, G, d, n_vis, 48, window, visual)
    ac = p.context()
    stats = []
    got = []
    for pieces in (None, [(l, l + 1) for l in range(L)], [(0, 7), (7, 12), (12, 32)]):
        got.append(p.score(ac, pieces))
        ac.air_budget()
        stats.append(ac.air_get_stats())
    ac.close()
    assert all(np.array_equal(x, y) and np.array_equal(x, z) for x, y, z in zip(*got))
    assert all(np.array_equal(x, y) and np.array_equal(x, z) for x, y, z in zip(*stats))
    for (l, b) in [(0, 0), (L // 2, 1), (L - 1, B - 1)]:
        np.testing.assert_allclose(got[0][l][b, 0], p.oracle(l, b, 0), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
        np.testing.assert_allclose(stats[0][1][b, l], O.skewness(got[0][l][b, 0].astype(np.float64)), rtol=1e-9, atol=1e-12)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("G", [2, 7])
@pytest.mark.parametrize("spread", [1.0, 18.0, 100.0, 1e3, 1e4, 1e5])
@pytest.mark.parametrize("L,B,run", [(2, 1, 512), (16, 16, 1152)])
def test_weights_of_a_row_add_up_to_one_whatever_the_logits(spread, G, d, L, B, run):
    # Pass 1 forms its logits with products of 32 x 32, pass 2 with products of 16 x 16: they have to be the same bits, or a weight is
    # off by 2^(difference) where a key stands above all others (raw logits of 4e6 have a spacing of 0.5, that is 4 % of a weight).
    # No text columns: every row's weights add up to 1, to the rounding of fp32 sums of 2304 terms in runs of 512 or 1152.
    assert _run_keys(2304, L * B * 2, G * 32) == run
    p = _Prompt(L, B, 2, G, d, 2304, 16, 32, True, spread)
    ac = p.context()
    got = p.score(ac)
    ac.close()
    for x in got:
        np.testing.assert_allclose(x.astype(np.float64).sum(axis=2), 1.0, rtol=0, atol=1e-6)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("visual", [False, True])
@pytest.mark.parametrize("n_vis", [500, 3000])  # one part, several
def test_skewness_of_rows_with_little_or_no_spread(n_vis, visual, d):
    # visual keys that are equal, equal but for k 2^-21 in one element (below what fp32 scores resolve) and for k 2^-6
    import torch

    p = _Prompt(4, 2, 1, 7, d, n_vis, 48, 32, visual)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    for l, step in enumerate([None, 0.0, 2.0 ** -21, 2.0 ** -6]):
        if step is None:
            continue
        vis = p.k[l][:, :, 9:9 + n_vis]
        vis.copy_(vis[:, :, :1].clone())
        vis[..., 5] = step * torch.randint(0, 4, vis.shape[:3], generator=gen, device="cuda:0").to(torch.bfloat16)
    ac = p.context()
    got = p.score(ac)
    ac.air_budget()
    s_t, s_k = ac.air_get_stats()
    ac.close()
    for l in range(4):
        for b in range(2):
            want = p.oracle(l, b, 0)
            np.testing.assert_allclose(got[l][b, 0], want, rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
            np.testing.assert_allclose(s_k[b, l], O.skewness(got[l][b, 0].astype(np.float64)), rtol=1e-7, atol=1e-7)
            if l in (1, 2) and not visual:  # (rows of a visual window do not see its last keys: their scores are smaller)
                assert s_k[b, l] == 0.0 and O.skewness(want) == 0.0


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("G,window,lost", [(7, 32, (3, 31)), (2, 20, (0,)), (2, 17, (5,)), (8, 40, (17, 18, 39))])  # to 32 rows, none for the second share; more than 256
def test_text_keys_that_are_no_numbers_leave_the_window(d, G, window, lost):
    # Eq.5 with a threshold of 0 takes every candidate whose logit is a number: the rows of the group are then fewer than the window
    # has tokens, and come from the lists.
    import torch

    p = _Prompt(2, 1, 2, G, d, 1300, window + 5, window)
    s = p.seqs[0]
    for j in lost:
        p.k[1][0, 1, s.win_start + j] = float("nan")
    ac = p.context()
    got = p.score(ac)
    cnt, _ = ac.air_get_elite(1)
    ac.close()
    assert cnt[0].tolist() == [window] * G + [window - len(lost)] * G
    rows = [j for j in range(window) if j not in lost]
    k = p.k[1][0, 1].double()
    want = torch.zeros(s.vis_len, dtype=torch.float64, device=k.device)
    for g in range(G):
        q = p.q[1][0, G + g, s.win_start - s.vis_start - s.vis_len:].double()[rows]
        keys = torch.cat([k[s.vis_start:s.vis_start + s.vis_len], k[s.win_start:s.win_start + window][rows]])
        want += torch.softmax(q @ keys.T / math.sqrt(d), dim=1)[:, :s.vis_len].mean(dim=0) / G
    np.testing.assert_allclose(got[1][0, 1], want.cpu().numpy(), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
    for l, h in [(0, 0), (0, 1), (1, 0)]:
        np.testing.assert_allclose(got[l][0, h], p.oracle(l, 0, h), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("G,window", [(5, 7), (7, 33), (3, 43), (7, 43)])  # 35 to 301 rows, none a whole number of blocks of 16
@pytest.mark.parametrize("behind", [1, 11, 700 - 333])  # keys that are no numbers: the first behind the window, the rest of its group of 32, all
@pytest.mark.parametrize("value", ["nan", "inf", "-inf"])
def test_keys_behind_a_visual_window_do_not_count_whatever_they_hold(d, G, window, behind, value):
    # A row of a visual window is normalised over the keys at or before its own: behind the window's end every score is 0.
    end = 333
    p = _Prompt(2, 1, 2, G, d, 700, 16, window, True)
    s = p.seqs[0]
    p.seqs = [synth.configs.Seq(s.seq_len, s.vis_start, s.vis_len, s.vis_start + end - window, window)]
    ac = p.context()
    want = p.score(ac)
    ac.air_budget()
    want_stats = ac.air_get_stats()
    for k in p.k:
        k[:, :, s.vis_start + end:s.vis_start + end + behind] = float(value)
    got = p.score(ac)
    ac.air_budget()
    stats = ac.air_get_stats()
    ac.close()
    for l in range(2):
        assert np.array_equal(got[l], want[l])
        assert not got[l][..., end:].any()
        np.testing.assert_allclose(got[l].astype(np.float64).sum(axis=2), 1.0, rtol=0, atol=1e-6)
    assert all(np.array_equal(x, y) for x, y in zip(stats, want_stats))


@pytest.mark.parametrize("d,alpha", [(128, 0.0), (64, 0.0), (64, 0.9)])
def test_a_unit_without_rows_scores_zero(d, alpha):
    # every text key of one unit is no number: no candidate passes, with a threshold (in a workspace without the stash) and without one
    import ctypes as C

    import torch

    p = _Prompt(2, 1, 2, 7, d, 1300, 40, 32)
    s = p.seqs[0]
    p.k[1][0, 1, s.win_start:] = float("nan")
    ac = p.context(alpha=alpha)
    if alpha:
        stash = 2 * 2 * 6 * 32 * 256 * 4
        least = ac.workspace_bytes - stash - (stash // 256 + 255) // 256 * 256
        ac.lib.air_destroy(ac.handle)
        ac.workspace, ac.handle = torch.empty(least, dtype=torch.uint8, device="cuda:0"), C.c_void_p()
        assert ac.lib.air_create(C.byref(ac.cfg), ac.workspace.data_ptr(), least, C.byref(ac.handle)) == 0
    for _ in range(2):  # (the second time over the first one's scores)
        got = p.score(ac)
        cnt, _ = ac.air_get_elite(1)
        assert not cnt[0, 7:].any() and cnt[0, :7].all()
        assert not got[1][0, 1].any()
        for l, h in [(0, 0), (0, 1), (1, 0)]:
            np.testing.assert_allclose(got[l][0, h], p.oracle(l, 0, h, alpha), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
    ac.air_budget()
    assert ac.air_get_budgets().sum() > 0
    ac.close()


@pytest.mark.parametrize("d,visual", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("value", ["-inf", "nan", "3e9", "-3e9"])
def test_first_references_from_keys_that_are_far_or_no_numbers(value, d, visual):
    # Runs of 1152 keys: a row's first reference is its maximum over the run's first 256 keys.  Here all of those are infinitely low, no
    # numbers, or beyond the bound of the references on either side.
    L = B = 16
    assert _run_keys(2304, L * B * 2, 7 * 32) == 1152
    p = _Prompt(L, B, 2, 7, d, 2304, 40, 32, visual)
    n0 = p.seqs[0].vis_start
    for x, y in zip(p.q, p.k):
        x[..., 1], y[..., 1] = 1.0, 0.0
    ac = p.context()
    want = p.score(ac)
    units = [(0, 0, 0), (9, 3, 1), (L - 1, B - 1, 1)]
    for l, b, h in units:
        for lo in (n0, n0 + 1152) if value != "nan" else (n0,):
            p.k[l][b, h, lo:lo + 256] = 0.0
            p.k[l][b, h, lo:lo + 256, 1] = float(value)
    got = p.score(ac)
    ac.close()
    for l, b, h in units:
        if value == "nan":  # no row has a softmax then; the keys say so
            assert np.isnan(got[l][b, h, :256]).all() and not np.isnan(got[l][b, h, 256:]).any()
        else:
            np.testing.assert_allclose(got[l][b, h], p.oracle(l, b, h), rtol=P.SCORE_RTOL, atol=P.SCORE_ATOL)
        got[l][b, h] = want[l][b, h]
    assert all(np.array_equal(x, y) for x, y in zip(got, want))
