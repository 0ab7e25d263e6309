"""Eq.5 on bf16 tensors far from the usual magnitudes: the fp32 logits of the matrix unit settle what lies outside their own
error, everything else is decided in fp64, so the elite sets are the oracle's at any size of the operands.  And on fp32 tensors
around the length of the span and the number of units where the kernel takes eight waves in place of four."""
import numpy as np
import pytest

import synth
from oracle import aircache_oracle as O
from tests import parity_util as P

pytestmark = pytest.mark.gpu


def _bf16(x):
    from synth.generate import f32_to_bf16_bits

    return f32_to_bf16_bits(x.astype(np.float32))


def _elite_sets(w, q, k, alpha):
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device

    dev = torch.device("cuda:0")
    seqs = w.seqs()
    ac = A.AirCache(config_for(w, 0.1, alpha=alpha, seqs=seqs, max_decode_steps=1), dev)
    qd, kd = to_device(q, dev), to_device(k, dev)
    ac.air_score(0, 1, [qd], [kd], [kd], seqs)
    cnt, idx = ac.air_get_elite(0)
    ac.close()
    return seqs, cnt, idx


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("big", [1.0, 64.0, 2048.0, 2.0 ** 17])
def test_elite_sets_of_large_operands_match_the_oracle(d, big):
    # half of the elements cancel: products of size `big`^2 that fp32 sums with errors far above the spacing of the logits,
    # which the other half spreads around the threshold
    w = synth.get_workload(2).scaled(head_dim=d, n_layers=1, n_vis=40, n_text=300, decode_steps=1)
    rng = np.random.default_rng(17)
    li = synth.layer_inputs(w, 0, w.seqs())
    q, k = (synth.storage_to_f64(x).copy() for x in (li.q_text, li.k))
    h, m = d // 4, d // 2  # elements [0, h) cancel against [m, m + h): in different slices of the contraction
    q[..., :h] = rng.integers(1, 4, q[..., :h].shape) * big
    q[..., m:m + h] = q[..., :h]
    k[..., :h] = rng.integers(-4, 5, k[..., :h].shape) * big
    k[..., m:m + h] = -k[..., :h]
    for lo in (h, m + h):
        q[..., lo:lo + h] = rng.integers(-3, 4, q[..., lo:lo + h].shape) * 0.25
        k[..., lo:lo + h] = rng.integers(-3, 4, k[..., lo:lo + h].shape) * 0.0625
    q, k = (_bf16(x) for x in (q, k))
    alpha = 0.9
    seqs, cnt, idx = _elite_sets(w, q, k, alpha)
    q64, k64 = synth.storage_to_f64(q), synth.storage_to_f64(k)
    s = seqs[0]
    ref, cand = s.win_start + s.win_len - 1, np.arange(s.win_start, s.win_start + s.win_len)
    t0 = s.vis_start + s.vis_len
    want = []
    for hq in range(w.n_q_heads):
        logits = O.last_row_logits(q64[0, hq, ref - t0], k64[0, hq // w.group][cand])  # every partial sum is exact in fp64
        want.append(cand[O.elite_set(logits, alpha)])
    P.check_elite(cnt, idx, [want], f"d={d} big={big}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_text,group", [(1, 7), (63, 9), (64, 4), (65, 9), (128, 16), (129, 1), (600, 7)])
def test_fp32_elite_sets_on_both_sides_of_64_candidates(d, n_text, group):
    # whole numbers: every logit is exact, in any order of its sum, and candidates of equal logit are in or out together
    w = synth.get_workload(2).scaled(dtype="f32", head_dim=d, n_layers=1, n_q_heads=2 * group, n_kv_heads=2, n_vis=300, n_text=n_text,
                                     decode_steps=1)
    rng = np.random.default_rng(5)
    li = synth.layer_inputs(w, 0, w.seqs())
    q, k = (rng.integers(-2, 3, x.shape).astype(np.float32) for x in (li.q_text, li.k))
    alpha = 0.5
    seqs, cnt, idx = _elite_sets(w, q, k, alpha)
    s = seqs[0]
    ref, cand = s.win_start + s.win_len - 1, np.arange(s.win_start, s.win_start + s.win_len)
    t0 = s.vis_start + s.vis_len
    want = []
    for hq in range(w.n_q_heads):
        logits = O.last_row_logits(q[0, hq, ref - t0].astype(np.float64), k[0, hq // group].astype(np.float64)[cand])
        want.append(cand[O.elite_set(logits, alpha)])
    P.check_elite(cnt, idx, [want], f"d={d} n_text={n_text} group={group}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,spans", [(2, (129, 64, 20)), (7, (65, 130, 1)), (3, (64, 64, 64))])
def test_fp32_elite_sets_are_the_same_bits_in_launches_of_many_units_and_of_few(d, group, spans):
    # 32 layers x 3 sequences x 3 KV heads are 288 units, more than there are CUs (four waves); one layer is 9 (eight waves where a
    # span of the call has more than 64 candidates, whatever the context could take)
    import torch

    import paper_2503_23956_amd as A

    L, n_vis, n_sys, n_text, dev = 32, 100, 5, 130, torch.device("cuda:0")
    n = n_sys + n_vis + n_text
    seqs = [synth.configs.Seq(n, n_sys, n_vis, n - w, w) for w in spans]
    gen = torch.Generator(device=dev)
    gen.manual_seed(23)
    k = [torch.randn((3, 3, n, d), generator=gen, device=dev) for _ in range(L)]
    q = [torch.randn((3, 3 * group, n_text, d), generator=gen, device=dev) for _ in range(L)]
    alpha = 0.2
    cfg = A.make_config(n_layers=L, n_q_heads=3 * group, n_kv_heads=3, head_dim=d, batch=3, max_vis_len=n_vis, max_nonvis_len=n - n_vis,
                        max_window=n_text, max_decode_steps=1, dtype=A.AIR_F32, alpha=alpha)
    ac = A.AirCache(cfg, dev)
    got = []
    for pieces in ([(0, L)], [(l, l + 1) for l in range(L)]):
        ac.air_reset()
        for l0, l1 in pieces:
            ac.air_score(l0, l1, q[l0:l1], k[l0:l1], k[l0:l1], seqs)
        got.append([(*ac.air_get_elite(l), ac.air_get_scores(l)) for l in range(L)])
    ac.close()
    for (cnt, idx, scores), (cnt1, idx1, scores1) in zip(*got):
        assert np.array_equal(cnt, cnt1) and np.array_equal(scores, scores1)
        assert all(np.array_equal(idx[b, h, :c], idx1[b, h, :c]) for (b, h), c in np.ndenumerate(cnt))
    for l in (0, L - 1):
        cnt, idx, _ = got[0][l]
        for b, s in enumerate(seqs):
            cand = np.arange(s.win_start, n)
            for h in range(3 * group):
                logits = O.last_row_logits(q[l][b, h, -1].double().cpu().numpy(), k[l][b, h // group].double().cpu().numpy()[cand])
                near = np.exp(logits - logits.max()) / alpha - 1  # (random logits: none on the threshold to fp64 rounding)
                assert np.abs(near).min() > 1e-9 and np.array_equal(idx[b, h, :cnt[b, h]], cand[near >= 0])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("alpha", [0.0, 0.5])
def test_infinite_logits(d, alpha):
    # a candidate with a logit of -inf is in the set exactly if the threshold is 0, one that is no number never is
    w = synth.get_workload(2).scaled(head_dim=d, n_layers=1, n_vis=40, n_text=70, decode_steps=1)
    s = w.seqs()[0]
    t0 = s.vis_start + s.vis_len
    li = synth.layer_inputs(w, 0, w.seqs())
    q, k = (synth.storage_to_f64(x).copy() for x in (li.q_text, li.k))
    q[..., 0] = 1.0
    k[:, :, t0 + 5, 0] = -np.inf
    k[:, :, t0 + 33, 0] = np.nan
    seqs, cnt, idx = _elite_sets(w, _bf16(q), _bf16(k), alpha)
    q64, k64 = synth.storage_to_f64(_bf16(q)), synth.storage_to_f64(_bf16(k))
    for hq in range(w.n_q_heads):
        with np.errstate(invalid="ignore"):
            logits = k64[0, hq // w.group, t0:] @ q64[0, hq, -1] / np.sqrt(d)
            want = t0 + np.nonzero(np.exp(logits - np.nanmax(logits)) >= alpha)[0]
        got = idx[0, hq, : cnt[0, hq]]
        assert np.array_equal(got, want), (hq, got, want)
        assert (t0 + 5 in got) == (alpha == 0.0) and t0 + 33 not in got


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_text", [7, 40, 100])
@pytest.mark.parametrize("above", [False, True])
def test_infinite_logits_beside_logits_that_overflow_fp32(d, n_text, above):
    # With a threshold of 0: a candidate of -inf below finite ones that overflow fp32 to -inf is in the set; one of +inf, which an
    # overflow to -inf in fp32 makes no number, is not, and the finite ones beside it are.
    w = synth.get_workload(2).scaled(head_dim=d, n_layers=1, n_vis=40, n_text=n_text, decode_steps=1)
    li = synth.layer_inputs(w, 0, w.seqs())
    q, k = (synth.storage_to_f64(x).copy() for x in (li.q_text, li.k))
    s = w.seqs()[0]
    t0 = s.vis_start + s.vis_len
    q[..., :2] = (0.0, 1.0)
    q[:, :, -1, 0] = 2.0 ** 100  # of the row that Eq.5 asks
    k[..., :2] = 0.0
    if not above:
        k[:, :, t0:, 0] = -2.0 ** 100
    k[:, :, t0 + 5, :2] = (-2.0 ** 100, np.inf) if above else (0.0, -np.inf)
    seqs, cnt, idx = _elite_sets(w, _bf16(q), _bf16(k), 0.0)
    want = [t for t in range(s.win_start, s.win_start + s.win_len) if not (above and t == t0 + 5)]
    for h in range(w.n_q_heads):
        assert idx[0, h, :cnt[0, h]].tolist() == want


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("low", [-3000.0, -1e5, -3e7, -3e9, -1e20, -7e25, -3e30, -1e36])
@pytest.mark.parametrize("alpha,n_text", [(0.9, 40), (0.0, 4), (0.0, 40)])  # the elite window, 28 rows, 280 rows
def test_visual_keys_masked_by_a_large_negative_logit(d, low, alpha, n_text):
    # whole chunks of visual keys with logits far below all others weigh nothing and leave the rest as it is without them
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device

    dev = torch.device("cuda:0")
    w = synth.get_workload(2).scaled(head_dim=d, n_layers=1, n_vis=1100, n_text=n_text, decode_steps=1)
    seqs = w.seqs()
    li = synth.layer_inputs(w, 0, seqs)
    q, k = (synth.storage_to_f64(x).copy() for x in (li.q_text, li.k))
    v0 = seqs[0].vis_start
    masked = np.zeros(1100, dtype=bool)
    masked[:256] = masked[600:1040] = True
    q[..., 0], k[..., 0] = 1.0, 0.0
    k[:, :, v0:v0 + 1100][:, :, masked, 0] = low
    q, k = _bf16(q), _bf16(k)
    ac = A.AirCache(config_for(w, 0.1, alpha=alpha, seqs=seqs, max_decode_steps=1), dev)
    qd, kd = to_device(q, dev), to_device(k, dev)
    ac.air_score(0, 1, [qd], [kd], [kd], seqs)
    got = ac.air_get_scores(0)
    ac.close()
    want, _ = O.layer_importance(synth.storage_to_f64(q)[0], synth.storage_to_f64(k)[0], P.seg_of(seqs[0]), alpha)
    P.check_scores(got, [want], seqs, f"low={low}")
    assert (got[0][:, masked] < 1e-30).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("high", [3000.0, 1e6, 3e7, 3e9, 1e20, 1e36])
@pytest.mark.parametrize("alpha,n_text,visual", [(0.9, 40, False), (0.0, 4, False), (0.0, 40, False), (0.0, 40, True)])
def test_visual_keys_of_a_large_positive_logit(d, high, alpha, n_text, visual):
    # two equal keys far above all others share the weight of every row that sees both
    import dataclasses

    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device

    dev = torch.device("cuda:0")
    w = synth.get_workload(2).scaled(head_dim=d, n_layers=1, n_vis=1100, n_text=n_text, decode_steps=1)
    seqs = w.seqs()
    if visual:
        seqs = [dataclasses.replace(s, win_start=s.vis_start + 690, win_len=n_text) for s in seqs]  # the second key is inside the window
    li = synth.layer_inputs(w, 0, w.seqs())
    q, k = (synth.storage_to_f64(x).copy() for x in (li.q_text, li.k))
    v0 = seqs[0].vis_start
    q[..., 0], k[..., 0] = 1.0, 0.0
    for key in (300, 700):
        k[:, :, v0 + key] = 0.0
        k[:, :, v0 + key, 0] = high
    q, k = _bf16(q), _bf16(k)
    ac = A.AirCache(config_for(w, 0.1, alpha=alpha, seqs=seqs, max_decode_steps=1, window_kind=int(visual)), dev)
    qd, kd = to_device(q, dev), to_device(k, dev)
    ac.air_score(0, 1, [qd], [kd], [kd], seqs)
    got = ac.air_get_scores(0)
    ac.close()
    q64, k64 = synth.storage_to_f64(q)[0], synth.storage_to_f64(k)[0]
    want = (O.layer_importance_visual_window(q64, k64, P.seg_of(seqs[0])) if visual else O.layer_importance(q64, k64, P.seg_of(seqs[0]), alpha))[0]
    P.check_scores(got, [want], seqs, f"high={high}")
    assert visual or np.allclose(got[0][:, [300, 700]], 0.5)


@pytest.mark.parametrize("n_text,window,alpha", [(48, 20, 0.0), (48, 33, 0.0), (48, 48, 0.02), (90, 90, 0.02)])  # up to 20, 33, 48, 90 rows a head
def test_many_units_of_heads_of_64_elements_are_those_of_small_calls(n_text, window, alpha):
    # A launch of more than 1024 units (512 with a threshold) keeps no tiles of the text columns: sets, columns (through the scores) and statistics are the same
    # bits as those of a call for every layer, which keeps them.
    import torch

    import paper_2503_23956_amd as A

    L, B, hkv, G, d, n_vis, n_sys = 33, 16, 3, 4, 64, 130, 5  # 32 layers a launch: 1536 units
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(64)
    n = n_sys + n_vis + n_text
    seqs = [synth.configs.Seq(n, n_sys, n_vis, n - window, window)] * B
    k = [torch.randn((B, hkv, n, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(L)]
    q = [torch.randn((B, hkv * G, n_text, d), generator=gen, device=dev).to(torch.bfloat16) for _ in range(L)]
    ac = A.AirCache(A.make_config(n_layers=L, n_q_heads=hkv * G, n_kv_heads=hkv, head_dim=d, batch=B, max_vis_len=n_vis, max_nonvis_len=n - n_vis,
                                  max_window=window, max_decode_steps=1, dtype=A.AIR_BF16, alpha=alpha), dev)
    got = []
    for calls in ([(0, L)], [(l, l + 1) for l in range(L)]):
        ac.air_reset()
        for l0, l1 in calls:
            ac.air_score(l0, l1, q[l0:l1], k[l0:l1], k[l0:l1], seqs)
        ac.air_budget()
        sets = []
        for l in range(L):
            cnt, idx = ac.air_get_elite(l)
            sets += [(cnt, [idx[b, h, :cnt[b, h]] for b in range(B) for h in range(hkv * G)])]
        got.append((sets, [ac.air_get_scores(l) for l in range(L)], ac.air_get_stats()))
    ac.close()
    rows = np.concatenate([cnt.ravel() for cnt, _ in got[0][0]])
    assert (rows.max() > 16) and (alpha or (rows == window).all())
    for (c0, i0), (c1, i1) in zip(got[0][0], got[1][0]):
        assert np.array_equal(c0, c1) and all(np.array_equal(x, y) for x, y in zip(i0, i1))
    assert all(np.array_equal(x, y) for x, y in zip(got[0][1], got[1][1]))
    assert all(np.array_equal(x, y) for x, y in zip(got[0][2], got[1][2]))
