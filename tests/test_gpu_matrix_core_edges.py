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


@pytest.mark.parametrize("rows", [112, 113, 184, 185, 264, 265, 640, 641])
def test_moe_block_rows_lines(rows):
    """One packed pass on either side of every line between the experts' block sizes (28, 46, 66 and 160 picks per
    expert: 16 experts, 4 picks a row), two sequences, against the oracle with the GPU's expert sets."""
    shape = workloads.SMALL_MOE_BF16
    w = scaled_weights(shape, seed=1, scale=1.5)
    model = oracle_model(shape, w)
    eng = make_engine(shape, w, max_context=700, max_batch_tokens=1024, flags=2)
    cu = [0, rows - 61, rows]
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
