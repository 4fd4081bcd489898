"""The matrix-core path's kernels at the edges of their ranges."""
import dataclasses

import numpy as np
import pytest

import workloads
from gpu_util import make_engine, oracle_model, scaled_weights, teacher_forced_compare
from oracle import transformer as T

pytestmark = pytest.mark.gpu

TOL = 2e-2  # bf16 weights, as in test_gpu_parity


@pytest.mark.parametrize("n_experts,top_k,n_samples", [(256, 9, 3), (16, 16, 1), (80, 1, 9), (64, 33, 2)])
def test_moe_routing_edges(n_experts, top_k, n_samples):
    """Experts up to four per lane and not a multiple of 64, all of them picked, one pick, picks beyond a batch of
    eight rows in the weighted sum.  Experts come in pairs with one router row, so their logits are equal
    bit for bit: the lower index must win every tie."""
    shape = dataclasses.replace(workloads.SMALL_MOE_BF16, n_experts=n_experts, top_k=top_k, expert_ffn_dim=64)
    w = scaled_weights(shape, seed=1, scale=1.5)
    for name in w:
        if name.endswith("router"):
            w[name][1::2] = w[name][::2]
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, flags=2)
    toks, offs = workloads.make_prompts(3, 5, 70, shape.vocab, seed=2)
    steps = 3
    forced = np.random.default_rng(4).integers(0, shape.vocab, (3 * n_samples, steps)).astype(np.int32)
    worst, worst_lp = teacher_forced_compare(eng, model, toks, offs, n_samples, forced, steps)
    below, outside = (max(g[i] for g in model.routing_regret) for i in (0, 1))
    print(f"max |dlogits| = {worst:.3e}, max |dlogp| = {worst_lp:.3e}, routing gaps {below:.3e} {outside:.3e}")
    assert worst <= TOL and worst_lp <= TOL and below <= TOL and outside <= TOL
    picks = eng.rollout_debug_routing(3 * n_samples).reshape(-1, top_k)
    for row in picks:
        chosen = set(row.tolist())
        assert len(chosen) == top_k
        assert all(e - 1 in chosen for e in chosen if e % 2), row
    eng.close()


@pytest.mark.parametrize("rows", [56, 57, 80, 81, 264, 600])
def test_moe_block_rows_lines(rows):
    """Packed passes on either side of the line between the experts' block sizes (32 and 64 rows: 14 picks per
    expert, 16 experts, 4 picks a row) and beyond it, two sequences, against the oracle with the GPU's expert sets."""
    shape = workloads.SMALL_MOE_BF16
    w = scaled_weights(shape, seed=1, scale=1.5)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_context=700, max_batch_tokens=1024, flags=2)
    cu = [0, rows - 21, rows]
    toks = np.random.default_rng(rows).integers(0, shape.vocab, rows).astype(np.int32)
    got = eng.rollout_logprobs(toks, cu, temperature=1.0)
    picks = eng.rollout_debug_routing(rows)
    assert picks.shape == (shape.n_layers, rows, shape.top_k)
    want = []
    for a, b in zip(cu[:-1], cu[1:]):
        model.routing_override = {l: picks[l][a:b] for l in range(shape.n_layers)}
        want.append(T.packed_log_probs(model, toks[a:b], [0, b - a]))
    err = float(np.max(np.abs(got - np.concatenate(want))))
    below, outside = (max(g[i] for g in model.routing_regret) for i in (0, 1))
    print(f"{rows} rows: max |dlogp| = {err:.3e}, routing gaps {below:.3e} {outside:.3e}")
    assert err <= TOL and below <= TOL and outside <= TOL
    eng.close()


@pytest.mark.parametrize("rows", [12, 13, 28, 29, 56, 57, 80, 81])
def test_moe_tile_shape_lines(rows):
    """On either side of the lines between the experts' tile shapes (3, 7, 14 and 20 picks per expert: 16 experts, 4 picks a
    row), with column counts that leave remainders in tiles of 128, 192 and 256 columns (gate/up 2 x 160, hidden 544; only the
    latter in tiles of 64, which divide every gate/up projection)."""
    shape = dataclasses.replace(workloads.SMALL_MOE_BF16, hidden=544, expert_ffn_dim=160)
    w = scaled_weights(shape, seed=1, scale=1.5)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, flags=2)
    toks = np.random.default_rng(rows).integers(0, shape.vocab, rows).astype(np.int32)
    got = eng.rollout_logprobs(toks, [0, rows], temperature=1.0)
    picks = eng.rollout_debug_routing(rows)
    model.routing_override = {l: picks[l] for l in range(shape.n_layers)}
    err = float(np.max(np.abs(got - T.packed_log_probs(model, toks, [0, rows]))))
    below, outside = (max(g[i] for g in model.routing_regret) for i in (0, 1))
    print(f"{rows} rows: max |dlogp| = {err:.3e}, routing gaps {below:.3e} {outside:.3e}")
    assert err <= TOL and below <= TOL and outside <= TOL
    eng.close()


@pytest.mark.parametrize("rows,hidden,ffn", [(1, 512, 544), (17, 544, 1056), (40, 2080, 4000), (65, 544, 9000 // 32 * 32), (97, 1056, 2016),
                                             (129, 2080, 1056), (193, 544, 5024), (300, 1056, 544), (700, 2080, 2016), (1985, 544, 1056)])
def test_tile_plans_remainders(rows, hidden, ffn):
    """Whole packed passes whose rows, columns and k-tiles leave remainders in the tile shapes and numbers of splits that the
    planner picks for them (17 and 33 k-tiles among them: odd, and no more than a few per split).  These are tiles of up to 96 rows;
    test_gpu_tile_shapes launches every shape by itself."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1, hidden=hidden, ffn_dim=ffn)
    w = scaled_weights(shape, seed=1, scale=0.7 if hidden > 1024 else 1.0)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_context=600, max_batch_tokens=2048)
    lens = [rows % 500] * bool(rows % 500) + [500] * (rows // 500)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = np.random.default_rng(rows).integers(0, shape.vocab, rows).astype(np.int32)
    got = eng.rollout_logprobs(toks, cu, temperature=1.0)
    err = float(np.max(np.abs(got - T.packed_log_probs(model, toks, cu))))
    print(f"{rows} rows, hidden {hidden}, ffn {ffn}: max |dlogp| = {err:.3e}")
    assert err <= TOL
    eng.close()


@pytest.mark.parametrize("rows", [15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("hidden", [512, 2080])
def test_streamed_rows_lines(rows, hidden):
    """Decode steps around the lines of the streamed path: a full 16-row fragment, a second one of a single row, 32 rows
    and the first step of the tile path (17 for hidden sizes above 2048).  The samples end one by one, so the rows
    cross the lines on the way down: both operand layouts in the same buffers, one after the other."""
    shape = dataclasses.replace(workloads.SMALL_BF16, hidden=hidden, ffn_dim=544)
    w = scaled_weights(shape, seed=1, scale=1.0 if hidden == 512 else 0.7)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_live_samples=40)
    toks, offs = workloads.make_prompts(1, 70, 70, shape.vocab, seed=4)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 6)).astype(np.int32)
    lens = np.full(rows, 6, np.int32)
    lens[::7] = 2                                     # 17 -> 14, 33 -> 28 rows after the first step
    lens[1::9] = 4
    fwd = T.KVForward(model)
    prefix = fwd.new_cache()
    fwd.extend([prefix], [toks])
    caches = [prefix.fork() for _ in range(rows)]
    ids, *_ = eng.rollout_prefill(toks, offs, rows, lens, forced_first=forced[:, 0])
    worst = 0.0
    for t in range(1, 6):
        live = np.flatnonzero(lens > t)
        got_ids, _, _, _ = eng.rollout_decode_step(forced_tokens=forced[live, t])
        assert np.array_equal(got_ids, ids[live])
        gpu = eng.rollout_debug_logits()
        ref = fwd.extend([caches[i] for i in live], [[int(forced[i, t - 1])] for i in live])
        worst = max(worst, max(float(np.max(np.abs(gpu[k] - ref[k][0]))) for k in range(len(live))))
    print(f"{rows} rows, hidden {hidden}: max |dlogits| = {worst:.3e}")
    assert worst <= TOL
    assert eng.rollout_get_stats()["live_samples"] == 0
    eng.close()


def other_work():
    """A few ms of other kernels, on a stream of their own."""
    import torch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        a = torch.ones(1536, 1536, device="cuda")
        for _ in range(40):
            a = (a @ a).clamp_(0.0, 1.0)
    return stream


@pytest.mark.parametrize("rows,hidden,ffn", [(1, 512, 8960), (9, 544, 9024), (16, 1056, 4992), (17, 544, 9024), (32, 1056, 6016),
                                             (8, 3072, 5024), (16, 3104, 8032)])
def test_streamed_splits_join(rows, hidden, ffn):
    """Down projections deep enough for K splits that join inside their launch (or nearly so): one and two row tiles, splits with
    remainders.  Several steps and layers, so that every ticket is drawn again; the same job gives the same bits again, alone
    and beside other work on the GPU.  (Which split comes last is the hardware's to say; other work changes it.)"""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=2, hidden=hidden, ffn_dim=ffn)
    w = scaled_weights(shape, seed=1, scale=0.7 if hidden > 1024 else 1.0)
    model = oracle_model(shape, w)
    toks, offs = workloads.make_prompts(1, 20, 20, shape.vocab, seed=4)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 4)).astype(np.int32)
    runs = []
    for load in (False, False, True):
        eng = make_engine(shape, w, max_live_samples=40)
        eng.rollout_prefill(toks, offs, rows, np.full(rows, 4, np.int32), forced_first=forced[:, 0])
        got = []
        for t in range(1, 4):
            if load:
                other_work()
            eng.rollout_decode_step(forced_tokens=forced[:, t])
            got.append(eng.rollout_debug_logits())
        runs.append(got)
        eng.close()
    fwd = T.KVForward(model)
    prefix = fwd.new_cache()
    fwd.extend([prefix], [toks])
    caches = [prefix.fork() for _ in range(rows)]
    worst = 0.0
    for t in range(1, 4):
        ref = fwd.extend(caches, [[int(forced[i, t - 1])] for i in range(rows)])
        worst = max(worst, max(float(np.max(np.abs(runs[0][t - 1][k] - ref[k][0]))) for k in range(rows)))
    print(f"{rows} rows, hidden {hidden}, ffn {ffn}: max |dlogits| = {worst:.3e}")
    assert worst <= TOL
    assert all(np.array_equal(a, b) and np.array_equal(a, c) for a, b, c in zip(*runs))


def stream_kernels(eng):
    """template arguments of the streamed projections' kernels that ran"""
    return {k["name"][len("gemm_stream_kernel<"):-1] for k in eng.rollout_kernel_stats() if k["name"].startswith("gemm_stream_kernel<")}


@pytest.mark.parametrize("rows,hidden,ffn,kernel", [(1, 5152, 4896, "1,4,2,8,false,2"), (9, 5152, 4896, "1,4,2,8,false,2"),
                                                    (16, 5120, 5024, "1,4,2,8,false,2"), (16, 3104, 8032, "1,2,3,8,false,2"),
                                                    (4, 4096, 4096, "1,1,3,16,false,2"), (32, 1056, 6016, "2,2,2,8,false,2")])
def test_streamed_residual_shapes(rows, hidden, ffn, kernel):
    """O and down projections on either side of the lines between one piece, splits with two column tiles and splits with four, the
    last of 322 column tiles not a whole block, 153 k-tiles in three splits."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=2, hidden=hidden, ffn_dim=ffn)
    w = scaled_weights(shape, seed=1, scale=0.5 if hidden > 4000 else 0.7)
    model = oracle_model(shape, w)
    toks, offs = workloads.make_prompts(1, 20, 20, shape.vocab, seed=4)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 3)).astype(np.int32)
    eng = make_engine(shape, w, max_live_samples=40, flags=4)
    worst, worst_lp = teacher_forced_compare(eng, model, toks, offs, rows, forced, 3)
    ran = stream_kernels(eng)
    eng.close()
    print(f"{rows} rows, hidden {hidden}, ffn {ffn}: max |dlogits| = {worst:.3e}, {sorted(ran)}")
    assert worst <= TOL and worst_lp <= TOL
    assert kernel in ran


@pytest.mark.parametrize("rows,hidden,vocab,kernel", [
    (8, 512, 16 * 1025, "1,2,2,8,false,0"), (9, 512, 16 * 1025, "1,4,1,8,false,0"), (16, 512, 16 * 1027, "1,4,1,8,false,0"),
    (16, 2048, 16 * 1025, "1,2,2,8,false,0"), (17, 512, 16 * 1025, "2,4,1,4,false,0"), (31, 512, 16 * 1026, "2,4,1,4,false,0"),
    (32, 512, 16 * 1027, "2,4,1,4,false,0"), (8, 512, 16 * 501, "1,2,2,8,false,0"), (16, 512, 16 * 1023, "1,2,2,8,false,0"),
    (17, 512, 16 * 501, "2,2,2,4,false,0"), (32, 512, 16 * 1023, "2,2,2,4,false,0"), (8, 1536, 16 * 191, "1,1,3,16,false,0"),
    (17, 512, 16 * 65, "1,1,3,16,true,0")])
def test_streamed_logits(rows, hidden, vocab, kernel):
    """The logits of decode steps in every shape they are planned with, vocabularies that leave one, two or three of a workgroup's
    column tiles over: all logits against the oracle."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1, hidden=hidden, ffn_dim=544, vocab=vocab)
    w = scaled_weights(shape, seed=1, scale=0.7 if hidden > 1024 else 1.0)
    model = oracle_model(shape, w)
    toks, offs = workloads.make_prompts(1, 20, 20, shape.vocab, seed=4)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 3)).astype(np.int32)
    eng = make_engine(shape, w, max_live_samples=40, flags=4)
    worst, worst_lp = teacher_forced_compare(eng, model, toks, offs, rows, forced, 3)
    ran = stream_kernels(eng)
    eng.close()
    print(f"{rows} rows, hidden {hidden}, vocab {vocab}: max |dlogits| = {worst:.3e}, {sorted(ran)}")
    assert worst <= TOL and worst_lp <= TOL
    assert kernel in ran


def test_timing_records_count_the_planes_that_attention_reads():
    """A streamed step of 3 rows whose QKV projection (1536 x 1024) leaves four planes: the attention's record counts them, as it does
    on the tile path."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1, hidden=1024, ffn_dim=544)
    eng = make_engine(shape, scaled_weights(shape, seed=1), flags=4)
    toks, offs = workloads.make_prompts(1, 20, 20, shape.vocab, seed=4)
    eng.rollout_prefill(toks, offs, 3, np.full(3, 4, np.int32), forced_first=np.array([1, 2, 3], np.int32))
    eng.rollout_decode_step(forced_tokens=np.array([4, 5, 6], np.int32))
    (attn,) = [k for k in eng.rollout_kernel_stats() if k["name"].startswith("attn_decode_fused_kernel")]
    ran = stream_kernels(eng)
    eng.close()
    assert "1,2,3,8,false,0" in ran
    cached = 3 * (20 + 1)                             # 20 prompt positions fill no page of 32: nothing is shared
    q, qkv = 8 * 128, (8 + 2 * 2) * 128
    assert attn["launches"] == 1
    assert attn["bytes"] == cached * 2 * 128 * 2 * 2 + 3 * (4.0 * 4 * qkv + 4.0 * q)


@pytest.mark.parametrize("rows", [7, 20, 43, 127, 129])
def test_attention_splits_fill_the_chip_once(rows):
    """Row counts that do not divide the 256 CUs, with contexts long enough to be cut: 16, 6, 2 and 1 splits per
    (row, KV head), and one row past the workgroups of eight wavefronts."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1)
    w = scaled_weights(shape, seed=1)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_live_samples=136, max_context=1600, max_batch_tokens=2048)
    toks, offs = workloads.make_prompts(1, 1500, 1500, shape.vocab, seed=8)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 3)).astype(np.int32)
    worst, worst_lp = teacher_forced_compare(eng, model, toks, offs, rows, forced, 3)
    print(f"{rows} rows: max |dlogits| = {worst:.3e}, max |dlogp| = {worst_lp:.3e}")
    assert worst <= TOL and worst_lp <= TOL
    eng.close()


EDGE_LENS = [1, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65, 95, 96, 97, 127, 129]


@pytest.mark.parametrize("rows,context", [(1, 4100), (3, 1100), (20, 1000), (33, 1500)])
def test_attention_splits_join(rows, context):
    """Contexts cut over several workgroups, whose last one to finish joins the results: the oracle's logits, and the same
    bits in a second context and beside other work on the GPU (up to 16 splits; eight and four wavefronts; rows of the tile
    path).  Which split comes last is the hardware's to say; other work changes it."""
    shape = dataclasses.replace(workloads.SMALL_BF16, hidden=512, ffn_dim=544)
    w = scaled_weights(shape, seed=1)
    model = oracle_model(shape, w)
    toks, offs = workloads.make_prompts(1, context, context, shape.vocab, seed=4)
    forced = np.random.default_rng(6).integers(0, shape.vocab, (rows, 4)).astype(np.int32)
    runs = []
    for load in (False, False, True):
        eng = make_engine(shape, w, max_live_samples=40, max_context=4200, max_batch_tokens=4200)
        eng.rollout_prefill(toks, offs, rows, np.full(rows, 4, np.int32), forced_first=forced[:, 0])
        got = []
        for t in range(1, 4):
            if load:
                other_work()
            eng.rollout_decode_step(forced_tokens=forced[:, t])
            got.append(eng.rollout_debug_logits())
        runs.append(got)
        eng.close()
    fwd = T.KVForward(model)
    prefix = fwd.new_cache()
    fwd.extend([prefix], [toks])
    caches = [prefix.fork() for _ in range(min(rows, 2))]
    worst = 0.0
    for t in range(1, 4):
        ref = fwd.extend(caches, [[int(forced[i, t - 1])] for i in range(len(caches))])
        worst = max(worst, max(float(np.max(np.abs(runs[0][t - 1][k] - ref[k][0]))) for k in range(len(caches))))
    print(f"{rows} rows at {context}: max |dlogits| = {worst:.3e}")
    assert worst <= TOL
    assert all(np.array_equal(a, b) and np.array_equal(a, c) for a, b, c in zip(*runs))


@pytest.mark.parametrize("copies", [1, 4])
def test_packed_attention_tiles(copies):
    """Sequences around the edges of 16- and 32-position tiles and 32-position key groups: 16 of them take one
    tile to a wavefront, 64 of them (5 blocks of 32 x 8 heads x 64) two."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1)
    w = scaled_weights(shape, seed=1)
    model = oracle_model(shape, w)
    lens = EDGE_LENS * copies
    eng = make_engine(shape, w, max_live_samples=80, max_batch_tokens=8192)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = np.random.default_rng(copies).integers(0, shape.vocab, int(cu[-1])).astype(np.int32)
    got = eng.rollout_logprobs(toks, cu, temperature=1.0)
    err = float(np.max(np.abs(got - T.packed_log_probs(model, toks, cu))))
    print(f"{len(lens)} sequences: max |dlogp| = {err:.3e}")
    assert err <= TOL
    eng.close()


def test_appended_rows_attention_tiles():
    """The same edges as appended tokens behind a cached context that is no multiple of 32, enough of them for two
    tiles to a wavefront: the logits after the last appended token against the oracle."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1)
    w = scaled_weights(shape, seed=1)
    model = oracle_model(shape, w)
    n = 64
    lens = np.array([max(1, x - 1) for x in EDGE_LENS * 4])  # a sequence is the last response token and these
    eng = make_engine(shape, w, max_live_samples=80, max_batch_tokens=8192)
    toks, offs = workloads.make_prompts(1, 45, 45, shape.vocab, seed=4)
    rng = np.random.default_rng(5)
    first = rng.integers(0, shape.vocab, n).astype(np.int32)
    ids, *_ = eng.rollout_prefill(toks, offs, n, np.full(n, 4, np.int32), forced_first=first)
    aoffs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    app = rng.integers(0, shape.vocab, int(aoffs[-1])).astype(np.int32)
    eng.rollout_extend(ids, app, aoffs, forced_next=rng.integers(0, shape.vocab, n).astype(np.int32))
    gpu = eng.rollout_debug_logits()
    fwd = T.KVForward(model)
    prefix = fwd.new_cache()
    fwd.extend([prefix], [toks])
    caches = [prefix.fork() for _ in range(n)]
    ref = fwd.extend(caches, [[int(first[i])] + [int(t) for t in app[aoffs[i]:aoffs[i + 1]]] for i in range(n)])
    worst = max(float(np.max(np.abs(gpu[i] - ref[i][-1]))) for i in range(n))
    print(f"max |dlogits| = {worst:.3e}")
    assert worst <= TOL
    eng.close()


@pytest.mark.parametrize("hidden,rows", [(96, 1), (1024, 40), (1056, 1985), (1056, 1986), (2048, 40), (2080, 1008), (2080, 1009), (4128, 40)])
def test_norm_threads_lines(hidden, rows):
    """Norm launches around the lines of their workgroups: a row of one chunk per thread and one more, and as many rows as
    the chip holds at once with a thread per chunk (hidden 1056 and 2080: 1985 and 1008) and one more."""
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1, hidden=hidden, ffn_dim=544)
    w = scaled_weights(shape, seed=1, scale=0.7 if hidden > 1024 else 1.0)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_live_samples=40, max_context=600, max_batch_tokens=2048)
    lens = [rows % 500] * bool(rows % 500) + [500] * (rows // 500)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    toks = np.random.default_rng(rows).integers(0, shape.vocab, rows).astype(np.int32)
    got = eng.rollout_logprobs(toks, cu, temperature=1.0)
    err = float(np.max(np.abs(got - T.packed_log_probs(model, toks, cu))))
    print(f"hidden {hidden}, {rows} rows: max |dlogp| = {err:.3e}")
    assert err <= TOL
    eng.close()
