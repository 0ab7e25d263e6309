"""The storages beside bf16 with heads of 128 elements (bf16 with heads of 64, fp32 with either): every compiled launch
shape of their decode kernel, caches whose ends fall on every side of a tile, a block and a split, against the oracle."""
import pytest

import synth
from tests.test_gpu_parity import _run_case

pytestmark = pytest.mark.gpu

STORAGES = [("bf16", 64), ("f32", 64), ("f32", 128)]


def _workload(dtype, d, **kw):
    return synth.get_workload(2).scaled(dtype=dtype, head_dim=d, **kw)


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("splits,waves,halves", [(1, 1, 1), (1, 2, 1), (1, 4, 1), (1, 8, 1), (4, 4, 1), (16, 8, 1), (2, 1, 1), (1, 4, 2)])
def test_decode_launch_shapes(dtype, d, splits, waves, halves):
    # 225 + 51 rows: appends cross blocks of 16 and of 32 tokens, splits of which some hold a single block or none
    w = _workload(dtype, d, n_layers=2, n_vis=900, n_text=37, decode_steps=36)
    _run_case(w, 0.25, steps=36, oracle_steps=[0, 1, 12, 13, 28, 29, 35],
              tuning=dict(decode_splits=splits, decode_waves=waves, decode_halves=halves))


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("waves", [1, 4])
def test_decode_longest_cache_first_in_a_ragged_batch(dtype, d, waves):
    w = synth.get_workload(3).scaled(dtype=dtype, head_dim=d, batch=3, n_layers=5, n_vis=700, n_text=40, decode_steps=18)
    _run_case(w, 0.25, steps=18, oracle_steps=[0, 16, 17], token_major=True,
              tuning=dict(decode_order=2, decode_splits=1, decode_waves=waves))


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("n_vis,n_text,n_sys,steps", [(1, 1, 0, 40), (2, 1, 1, 2), (15, 1, 0, 2), (33, 2, 0, 3), (257, 3, 0, 17)])
def test_small_caches(dtype, d, n_vis, n_text, n_sys, steps):
    w = _workload(dtype, d, n_layers=2, n_vis=n_vis, n_text=n_text, n_sys=n_sys, decode_steps=steps)
    _run_case(w, 1.0 if n_vis < 30 else 0.3, steps=steps)


@pytest.mark.parametrize("dtype,d", STORAGES)
def test_one_head_per_group_and_sixteen(dtype, d):
    _run_case(_workload(dtype, d, n_layers=1, n_q_heads=3, n_kv_heads=3, n_vis=300, n_text=20, decode_steps=2), 0.2, steps=2)
    _run_case(_workload(dtype, d, n_layers=1, n_q_heads=16, n_kv_heads=1, n_vis=300, n_text=20, decode_steps=2), 0.2, steps=2)


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("n_vis,n_text,alpha,visual", [
    (255, 9, None, None), (256, 9, None, None), (257, 9, None, None), (1024, 24, None, None), (1025, 24, None, None),
    (1100, 40, 0.02, None),      # an elite window of more rows than a unit's stash holds
    (700, 4, 0.0, None),         # 28 rows: a stash of several rounds
    (1300, 5, 0.0, None),        # 35 rows: one more round than the stash
    (600, 40, 0.0, None),        # 280 rows
    (780, 12, 0.0, (250, 12)),   # visual window across a chunk boundary
    (1100, 3, 0.0, (-3, 3)),
])
def test_scoring_at_the_edges_of_chunks_and_of_the_stash(dtype, d, n_vis, n_text, alpha, visual):
    w = _workload(dtype, d, n_layers=2, n_vis=n_vis, n_text=n_text, decode_steps=1)
    _run_case(w, 0.10, alpha=alpha, steps=1, visual_window=visual)


@pytest.mark.parametrize("dtype,d", STORAGES)
def test_scoring_strided_ragged_batch_layer_by_layer(dtype, d):
    w = synth.get_workload(3).scaled(dtype=dtype, head_dim=d, batch=3, n_layers=3, n_vis=900, n_text=30, decode_steps=1)
    _run_case(w, 0.10, steps=1, layer_chunk=1, token_major=True)
    _run_case(w, 0.10, steps=1, causal_text=True, alpha=0.0)


@pytest.mark.parametrize("dtype,d", [("bf16", 128)] + STORAGES)
@pytest.mark.parametrize("base,batch,n_layers", [(2, 1, 3), (2, 1, 11), (2, 1, 18), (3, 2, 5), (3, 3, 6)])
def test_decode_column_parts_equal_one_workgroup_per_unit(dtype, d, base, batch, n_layers):
    # 12 (eight parts), 40 and 44 (four), 72 (two) units of ~690 keys, one sequence and ragged batches: a workgroup of a part does the same
    # arithmetic per output column, so outputs and appended rows agree bit for bit
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device, to_host

    dev = torch.device("cuda:0")
    steps = 34
    w = synth.get_workload(base).scaled(dtype=dtype, head_dim=d, batch=batch, n_layers=n_layers, n_vis=1800, n_text=221, decode_steps=steps)
    seqs, L = w.seqs(), w.n_layers
    layers = [synth.layer_inputs(w, l, seqs) for l in range(L)]
    q, k, v = ([to_device(getattr(li, name), dev) for li in layers] for name in ("q_text", "k", "v"))
    ins = [[to_device(np.stack(x), dev) for x in zip(*[synth.decode_inputs(w, l, t) for l in range(L)])] for t in range(steps)]
    seen = []
    for halves in (1, 2):
        ac = A.AirCache(config_for(w, 0.25, seqs=seqs, max_decode_steps=steps), dev)
        ac.air_set_tuning(decode_splits=1, decode_waves=4, decode_tiles=4, decode_halves=halves)
        ac.air_score(0, L, q, k, v, seqs)
        ac.air_budget()
        ac.air_select_compact(0, L, k, v)
        out = torch.empty((steps, L, batch, w.n_q_heads, d), dtype=q[0].dtype, device=dev)
        for t in range(steps):
            ac.air_decode_attn(0, L, *ins[t], out[t])
        lens = ac.air_get_lengths()
        seen.append((to_host(out), [ac.air_get_cache(l, b, h, int(lens[b, l])) for l in (0, L - 1) for b in range(batch) for h in (0, w.n_kv_heads - 1)]))
        ac.close()
    assert np.array_equal(seen[0][0], seen[1][0]) and not np.isnan(synth.storage_to_f64(seen[0][0])).any()
    for (k1, v1), (k2, v2) in zip(seen[0][1], seen[1][1]):
        assert np.array_equal(k1, k2) and np.array_equal(v1, v2)


@pytest.mark.parametrize("dtype,d,n_layers", [("bf16", 128, 8), ("bf16", 64, 16), ("f32", 64, 8), ("f32", 128, 4)])
def test_caches_several_times_the_memory_side_cache(dtype, d, n_layers):
    # 660 MB of cache: loads and stores marked as used once, in the gather (retention 1: the compacted rows are the prompt's)
    # and in every decode launch shape that has them, on sampled units
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from oracle import aircache_oracle as O
    from paper_2503_23956_amd.device_inputs import config_for, device_layer_inputs, to_device, to_host
    from tests import parity_util as P

    dev = torch.device("cuda:0")
    shapes = [(1, 1), (1, 2), (2, 1), (4, 1), (4, 2)]  # (waves, order of the units)
    w = synth.get_workload(3).scaled(dtype=dtype, head_dim=d, n_layers=n_layers, n_vis=2450, n_text=60, decode_steps=len(shapes))
    seqs, L, G = w.seqs(), w.n_layers, w.group
    q, k, v = zip(*[device_layer_inputs(w, l, seqs, dev) for l in range(L)])
    ac = A.AirCache(config_for(w, 1.0, seqs=seqs, max_decode_steps=len(shapes)), dev)
    ac.air_score(0, L, q, k, v, seqs)
    ac.air_budget()
    ac.air_select_compact(0, L, k, v)
    units = [(0, 0, 0), (L // 2, 7, 2), (L - 1, w.batch - 1, w.n_kv_heads - 1)]
    rows = {}
    for (l, b, h) in units:
        n = seqs[b].seq_len
        rows[l, b, h] = [to_host(x[l][b, h, :n]) for x in (k, v)]
        kk, vv = ac.air_get_cache(l, b, h, n)
        assert np.array_equal(kk, rows[l, b, h][0]) and np.array_equal(vv, rows[l, b, h][1])
    out = torch.empty((L, w.batch, w.n_q_heads, d), dtype=q[0].dtype, device=dev)
    for t, (waves, order) in enumerate(shapes):
        ac.air_set_tuning(decode_splits=1, decode_waves=waves, decode_tiles=4, decode_order=order)
        qn, kn, vn = (np.stack(x) for x in zip(*[synth.decode_inputs(w, l, t) for l in range(L)]))
        ac.air_decode_attn(0, L, to_device(qn, dev), to_device(kn, dev), to_device(vn, dev), out)
        got = synth.storage_to_f64(to_host(out))
        for (l, b, h) in units:
            rows[l, b, h] = [np.concatenate([r, x[l, b, h][None]]) for r, x in zip(rows[l, b, h], (kn, vn))]
            want = O.decode_attn(synth.storage_to_f64(qn[l, b, h * G:(h + 1) * G]), *(synth.storage_to_f64(r) for r in rows[l, b, h]))
            assert np.abs(got[l, b, h * G:(h + 1) * G] - want).max() <= P.DECODE_ATOL[w.dtype], (t, l, b, h)
    ac.close()


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("splits,waves,halves", [(1, 1, 1), (1, 4, 1), (1, 8, 1), (4, 4, 1), (1, 4, 2)])
def test_infinite_values_and_masked_runs_of_keys(dtype, d, splits, waves, halves):
    # K': the first 70 rows have logits of -inf (whole chunks of every launch shape); V': infinite elements in the first block,
    # in the last one (which the tail of a chunk reads again) and in appended tokens, next to finite columns
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from oracle import aircache_oracle as O
    from paper_2503_23956_amd.device_inputs import config_for, to_device, to_host
    from tests import parity_util as P

    dev = torch.device("cuda:0")
    steps = 3
    w = _workload(dtype, d, n_layers=1, n_sys=80, n_vis=400, n_text=21, decode_steps=steps)
    seqs, G = w.seqs(), w.group
    n0 = seqs[0].vis_start + seqs[0].vis_len
    li = synth.layer_inputs(w, 0, seqs)
    q, k, v = (to_device(x, dev) for x in (li.q_text, li.k, li.v))
    k[:, :, :70, 0] = -np.inf
    v[:, :, 3, 1] = np.inf
    v[:, 1, 75, 2] = -np.inf
    v[:, :, n0 + 20, 5] = -np.inf  # the last text token: the last row of the cache
    v[:, :, 40, 7] = np.inf        # a row of zero weight: its column is infinite or no number
    ac = A.AirCache(config_for(w, 0.25, seqs=seqs, max_decode_steps=steps), dev)
    ac.air_set_tuning(decode_splits=splits, decode_waves=waves, decode_halves=halves)
    ac.air_score(0, 1, [q], [k], [v], seqs)
    ac.air_budget()
    ac.air_select_compact(0, 1, [k], [v])
    out = torch.empty((1, 1, w.n_q_heads, d), dtype=q.dtype, device=dev)
    for t in range(steps):
        qn, kn, vn = (to_device(x, dev)[None] for x in synth.decode_inputs(w, 0, t))
        qn[..., 0] = 1.0
        vn[..., 9 + t] = np.inf
        ac.air_decode_attn(0, 1, qn, kn, vn, out)
        got = synth.storage_to_f64(to_host(out))[0, 0]
        q64 = synth.storage_to_f64(to_host(qn))[0, 0]
        n = int(ac.air_get_lengths()[0, 0])
        for h in range(w.n_kv_heads):
            kk, vv = (synth.storage_to_f64(x) for x in ac.air_get_cache(0, 0, h, n))
            assert np.isneginf(kk[:70, 0]).all() and np.isfinite(kk[70:]).all()
            kk, vv, zero = kk[70:], vv[70:], vv[:70]
            want = O.decode_attn(q64[h * G:(h + 1) * G], kk, np.where(np.isfinite(vv), vv, 0.0))
            for col in range(d):
                x = got[h * G:(h + 1) * G, col]
                inf = vv[~np.isfinite(vv[:, col]), col]
                if len(inf):
                    assert (x == inf[0]).all(), (t, h, col, x)
                elif np.isfinite(zero[:, col]).all():
                    assert np.abs(x - want[:, col]).max() <= P.DECODE_ATOL[w.dtype], (t, h, col)
                else:
                    assert not np.isfinite(x).any()
    ac.close()


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("q0,k0", [(8.0, 37.0), (8.0, -37.0), (64.0, 47.0), (-256.0, 83.0), (1024.0, 997.0), (1024.0, -771.0)])
def test_appended_token_weighs_what_a_cached_key_of_the_same_logit_does(dtype, d, q0, k0):
    # every key the same: the weights are equal however large the logit (up to 1e6 before the scale), so that with values of 0
    # and 1 the output is the appended token's share of the cache
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device, to_host

    dev = torch.device("cuda:0")
    w = _workload(dtype, d, n_layers=1, n_sys=5, n_vis=90, n_text=11, decode_steps=1)
    seqs = w.seqs()
    q, k, v = (torch.zeros_like(to_device(x, dev)) for x in (lambda li: (li.q_text, li.k, li.v))(synth.layer_inputs(w, 0, seqs)))
    k[..., 0] = k0
    qn, kn, vn = (torch.zeros_like(to_device(x, dev)[None]) for x in synth.decode_inputs(w, 0, 0))
    qn[..., 0], kn[..., 0], vn[:] = q0, k0, 1.0
    for splits, waves, halves in [(1, 1, 1), (1, 4, 1), (4, 4, 1), (1, 4, 2)]:
        ac = A.AirCache(config_for(w, 1.0, seqs=seqs, max_decode_steps=1), dev)
        ac.air_set_tuning(decode_splits=splits, decode_waves=waves, decode_halves=halves)
        ac.air_score(0, 1, [q], [k], [v], seqs)
        ac.air_budget()
        ac.air_select_compact(0, 1, [k], [v])
        out = torch.empty((1, 1, w.n_q_heads, d), dtype=q.dtype, device=dev)
        ac.air_decode_attn(0, 1, qn, kn, vn, out)
        share = synth.storage_to_f64(to_host(out)) * (seqs[0].seq_len + 1)
        # fp32: 107 equal addends, each partial sum rounded; bf16: the output's rounding
        assert np.abs(share - 1.0).max() <= (2e-6 if dtype == "f32" else 2.0 ** -8), (splits, waves, halves, share.min(), share.max())
        ac.close()


@pytest.mark.parametrize("dtype,d", STORAGES)
@pytest.mark.parametrize("alpha,n_text,visual", [(0.9, 24, None), (0.3, 24, None), (0.0, 3, None), (0.0, 3, (-3, 3)), (0.0, 24, None)])
def test_scoring_in_a_workspace_without_the_stash(dtype, d, alpha, n_text, visual):
    # such a workspace is accepted to the byte and reads the visual keys twice: fp32 scores bit for bit the same
    import ctypes as C
    import dataclasses

    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device

    dev = torch.device("cuda:0")
    w = _workload(dtype, d, n_layers=2, n_vis=1300, n_text=n_text, decode_steps=1)
    seqs, L = w.seqs(), w.n_layers
    if visual:
        seqs = [dataclasses.replace(s, win_start=s.vis_start + s.vis_len + visual[0], win_len=visual[1]) for s in seqs]
    layers = [synth.layer_inputs(w, l, w.seqs()) for l in range(L)]
    q, k, v = ([to_device(getattr(li, name), dev) for li in layers] for name in ("q_text", "k", "v"))
    cfg = config_for(w, 0.1, alpha=alpha, seqs=seqs, max_decode_steps=1, window_kind=int(visual is not None))
    full = A.AirCache(cfg, dev)
    many = alpha == 0.0 and w.group * seqs[0].win_len > 32
    stash = 0 if many else L * w.n_kv_heads * 6 * 32 * 256 * 4
    least = full.workspace_bytes - stash - ((stash // 256 + 255) // 256 * 256 if dtype == "bf16" else 0)
    lib, h = full.lib, C.c_void_p()
    workspace = torch.empty(least, dtype=torch.uint8, device=dev)
    assert lib.air_create(C.byref(cfg), workspace.data_ptr(), least - 1, C.byref(h)) == A.binding.AIR_ERR_WORKSPACE
    small = A.AirCache(cfg, dev)
    lib.air_destroy(small.handle)
    assert lib.air_create(C.byref(cfg), workspace.data_ptr(), least, C.byref(h)) == 0
    small.handle, small.workspace = h, workspace
    seen = []
    for ac in (full, small):
        ac.air_score(0, L, q, k, v, seqs)
        ac.air_budget()
        seen.append(([ac.air_get_scores(l) for l in range(L)], ac.air_get_budgets()))
        ac.close()
    for x, y in zip(seen[0][0], seen[1][0]):
        if dtype == "f32":
            assert np.array_equal(x, y)
        else:
            np.testing.assert_allclose(x, y, rtol=1e-5, atol=1e-30)
    assert np.abs(seen[0][1] - seen[1][1]).max() <= (0 if dtype == "f32" else 1)


@pytest.mark.parametrize("dtype,d,rows", [("f32", 64, 570), ("bf16", 64, 1140), ("f32", 128, 283)])
def test_decode_keeps_its_launch_shape_while_the_cache_grows(dtype, d, rows):
    # 285 KB a unit by the prompt, 288 KB passed after a few steps: the shape goes by the prompt, so every step has the bits of
    # the first step's shape (one workgroup of four waves, or its column parts)
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device

    dev = torch.device("cuda:0")
    steps = 24
    w = _workload(dtype, d, n_layers=1, n_sys=4, n_vis=rows - 24, n_text=20, decode_steps=steps)
    seqs = w.seqs()
    li = synth.layer_inputs(w, 0, seqs)
    q, k, v = ([to_device(x, dev)] for x in (li.q_text, li.k, li.v))
    outs = []
    for tuning in ({}, dict(decode_splits=1, decode_waves=4)):
        ac = A.AirCache(config_for(w, 1.0, seqs=seqs, max_decode_steps=steps), dev)
        ac.air_set_tuning(**tuning)
        ac.air_score(0, 1, q, k, v, seqs)
        ac.air_budget()
        ac.air_select_compact(0, 1, k, v)
        out = torch.empty((steps, 1, 1, w.n_q_heads, d), dtype=q[0].dtype, device=dev)
        for t in range(steps):
            ac.air_decode_attn(0, 1, *(to_device(x[None], dev) for x in synth.decode_inputs(w, 0, t)), out[t])
        outs.append(out)
        ac.close()
    for t in range(steps):
        assert torch.equal(outs[0][t], outs[1][t]), t


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("tuning", [{}, dict(score_rows_kernel=1)])
def test_a_low_threshold_that_leaves_more_rows_than_one_staging_round(dtype, d, tuning):
    # several hundred rows a unit with a threshold: the finish kernel's own passes over K_v, 512 rows staged at a time
    w = _workload(dtype, d, n_layers=1, n_q_heads=14, n_kv_heads=2, n_vis=560, n_text=160, decode_steps=1)
    import numpy as np
    import torch

    import paper_2503_23956_amd as A
    from paper_2503_23956_amd.device_inputs import config_for, to_device
    from tests import parity_util as P

    dev = torch.device("cuda:0")
    seqs = w.seqs()
    li = synth.layer_inputs(w, 0, seqs)
    alpha = 1e-6
    scores, elites, _, _ = P.oracle_score_layer(w, li, seqs, alpha)
    assert sum(len(e) for e in elites[0][:7]) > 512
    ac = A.AirCache(config_for(w, 0.1, alpha=alpha, seqs=seqs, max_decode_steps=1), dev)
    ac.air_set_tuning(**tuning)
    ac.air_score(0, 1, [to_device(li.q_text, dev)], [to_device(li.k, dev)], [to_device(li.v, dev)], seqs)
    cnt, idx = ac.air_get_elite(0)
    P.check_elite(cnt, idx, elites)
    P.check_scores(ac.air_get_scores(0), scores, seqs)
    ac.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_vis", [1, 15, 17, 33, 256, 257, 300])
@pytest.mark.parametrize("G,window", [(1, 1), (3, 1), (2, 3), (7, 1), (3, 5), (16, 1), (4, 8), (3, 11), (16, 5)])  # 1 to 80 rows
def test_fp32_scores_at_the_edges_of_tiles_and_row_blocks(d, n_vis, G, window):
    import numpy as np
    import torch

    import paper_2503_23956_amd as A

    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    n = 2 + n_vis + window
    seq = synth.configs.Seq(n, 2, n_vis, n - window, window)
    k = torch.randn((1, 2, n, d), generator=gen, device=dev)
    q = torch.randn((1, 2 * G, window, d), generator=gen, device=dev)
    cfg = A.make_config(n_layers=1, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, batch=1, max_vis_len=n_vis, max_nonvis_len=n - n_vis,
                        max_window=window, max_decode_steps=1, dtype=A.AIR_F32, alpha=0.0)
    ac = A.AirCache(cfg, dev)
    ac.air_score(0, 1, [q], [k], [k], [seq])
    got = ac.air_get_scores(0)[0]
    ac.close()
    want = torch.softmax(q[0].double().view(2, G, window, d) @ k[0, :, 2:].double().transpose(1, 2).unsqueeze(1) / d ** 0.5, dim=3)
    want = want[..., :n_vis].mean(dim=(1, 2)).cpu().numpy()
    # logits of a few units in fp32: sums of d products, each rounding 2^-24 of a partial sum, and as much again in the exponential
    np.testing.assert_allclose(got, want, rtol=1e-5)


@pytest.mark.parametrize("d,bound", [(128, 1e-6), (64, 1e-6)])
def test_error_of_fp32_scores_against_fp64(d, bound):
    # Relative 2-norm of the scores of an elite window (threshold 0.1), raw logits of a spread of 5 sqrt(d).  The largest are about 4 spreads, 20 units
    # scaled, and the sum of their products is rounded at partial sums of half that size, 10 2^-25 units each time: 3e-7, for d / 4 matrix
    # products about 1.3e-6 in one sum over all of them and half as much in two.  7.0e-7 measured; one chain of multiply-adds 1.30e-6 and
    # 1.39e-6, one sum of matrix products 1.52e-6 and 1.26e-6.
    import numpy as np
    import torch

    import paper_2503_23956_amd as A

    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    errs = []
    for seed, n_vis, G in ((1, 7290, 7), (2, 1300, 4), (3, 577, 2), (4, 16384, 8)):
        gen.manual_seed(seed)
        n = 9 + n_vis + 69
        seq = synth.configs.Seq(n, 9, n_vis, n - 60, 60)
        k = torch.randn((1, 2, n, d), generator=gen, device=dev)
        q = 5.0 * torch.randn((1, 2 * G, 69, d), generator=gen, device=dev)
        cfg = A.make_config(n_layers=1, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, batch=1, max_vis_len=n_vis, max_nonvis_len=78, max_window=60,
                            max_decode_steps=1, dtype=A.AIR_F32, alpha=0.1)
        ac = A.AirCache(cfg, dev)
        ac.air_score(0, 1, [q], [k], [k], [seq])
        got = ac.air_get_scores(0)[0].astype(np.float64)
        cnt, idx = ac.air_get_elite(0)
        ac.close()
        want = torch.zeros((2, n_vis), dtype=torch.float64, device=dev)
        for h in range(2 * G):
            rows = torch.tensor(idx[0, h, :cnt[0, h]].astype(np.int64), device=dev)
            keys = torch.cat([k[0, h // G, 9:9 + n_vis], k[0, h // G][rows]]).double()
            want[h // G] += torch.softmax(q[0, h][rows - 9 - n_vis].double() @ keys.T / d ** 0.5, dim=1).mean(dim=0)[:n_vis] / G
        errs.append(np.linalg.norm(got - want.cpu().numpy()) / np.linalg.norm(want.cpu().numpy()))
    assert np.mean(errs) <= bound, errs


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5])  # rows of a unit: products of four rows, of sixteen from the fifth on
@pytest.mark.parametrize("spread", [1.0, 300.0])
def test_fp32_scores_of_few_rows_are_the_same_bits_without_the_stash(d, G, spread):
    # Both passes form the logits there: raw ones in the thousands, of which a last bit would change a weight by a per cent.
    import ctypes as C

    import numpy as np
    import torch

    import paper_2503_23956_amd as A

    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(8)
    n_vis, n = 777, 3 + 777 + 1
    seq = synth.configs.Seq(n, 3, n_vis, n - 1, 1)
    k = [torch.randn((1, 2, n, d), generator=gen, device=dev) for _ in range(2)]
    q = [spread * torch.randn((1, 2 * G, 1, d), generator=gen, device=dev) for _ in range(2)]
    cfg = A.make_config(n_layers=2, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, batch=1, max_vis_len=n_vis, max_nonvis_len=n - n_vis, max_window=1,
                        max_decode_steps=1, dtype=A.AIR_F32, alpha=0.9)
    full, small = A.AirCache(cfg, dev), A.AirCache(cfg, dev)
    least = full.workspace_bytes - 2 * 2 * 4 * 32 * 256 * 4
    small.lib.air_destroy(small.handle)
    small.workspace, small.handle = torch.empty(least, dtype=torch.uint8, device=dev), C.c_void_p()
    assert small.lib.air_create(C.byref(cfg), small.workspace.data_ptr(), least, C.byref(small.handle)) == 0
    got = []
    for ac in (full, small):
        ac.air_score(0, 2, q, k, k, [seq])
        got.append([ac.air_get_scores(l)[0] for l in range(2)])
        ac.close()
    for l in range(2):
        assert np.array_equal(got[0][l], got[1][l])
        want = torch.softmax(q[l][0].double().view(2, G, d) @ k[l][0, :, 3:].double().transpose(1, 2) / d ** 0.5, dim=2)
        want = want[..., :n_vis].mean(dim=1).cpu().numpy()
        # sums of d products in eight parts, each rounded at d / 8 partial sums of up to `spread` 4 sqrt(d) / 2 raw units, scaled by 1 / sqrt(d)
        bound = 2.0 ** -24 * (d / 8 + 3) * 2 * spread * 4 + 1e-6
        assert np.linalg.norm(got[0][l] - want) <= bound * np.linalg.norm(want)
