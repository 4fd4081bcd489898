"""The plain path's kernels where they can go wrong: operand widths that are no multiple of the four values a
lane takes, row counts around the tile of eight, head sizes between the powers of two, contexts around the
256-position chunk of the attention."""
import dataclasses

import numpy as np
import pytest

import workloads
from gpu_util import make_engine, oracle_model, scaled_weights, teacher_forced_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,ffn,heads,kv_heads,head_dim,lens,n", [
    (66, 101, 2, 1, 32, [1, 9], 4),             # odd widths, scalar loads; 8 decode rows
    (252, 260, 3, 1, 96, [254], 9),             # widths not a multiple of a wavefront's 256; contexts reach 256, 257
    (512, 300, 4, 2, 256, [255, 511, 2], 1),    # one thread per dimension; contexts reach 512
    (130, 6, 6, 3, 64, [17], 1),                # one row
], ids=["odd", "chunk-edge", "wide-head", "one-row"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_plain_path_edges(hidden, ffn, heads, kv_heads, head_dim, lens, n, dtype):
    """Prefill and decode steps, teacher-forced, against the oracle.  fp32: 1e-4, a few hundred fp32 roundings of
    values of order one; bf16 weights with an fp16 cache: 2e-2."""
    shape = dataclasses.replace(workloads.C1_TINY, hidden=hidden, ffn_dim=ffn, n_q_heads=heads, n_kv_heads=kv_heads,
                                head_dim=head_dim, vocab=257, dtype=dtype)
    w = scaled_weights(shape, seed=7)
    model = oracle_model(shape, w)
    rng = np.random.default_rng(hidden)
    toks = rng.integers(0, shape.vocab, sum(lens)).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    steps = 5
    forced = rng.integers(0, shape.vocab, (len(lens) * n, steps)).astype(np.int32)
    eng = make_engine(shape, w, flags=1, max_context=640)
    worst, worst_lp = teacher_forced_compare(eng, model, toks, offs, n, forced, steps)
    print(f"max |dlogits| = {worst:.3e}, max |dlogp| = {worst_lp:.3e}")
    tol = {"fp32": 1e-4, "bf16": 2e-2}[dtype]
    assert worst <= tol and worst_lp <= tol
    assert eng.rollout_get_stats()["matrix_core_path"] == 0
    eng.close()
