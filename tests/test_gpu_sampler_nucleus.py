"""GPU parity of the nucleus selection (top_p < 1): the histogram search for the smallest weight of the
nucleus, on one workgroup per row (up to 28672 ids) and on several, against the oracle's explicit
ordering.  Token ids and weight sums are integers: exact."""
import numpy as np
import pytest

import workloads
from oracle import sampler

pytestmark = pytest.mark.gpu


def hard_rows(vocab, seed):
    """Rows that end the nucleus in every kind of place."""
    rng = np.random.default_rng(seed)
    z = workloads.random_logits(9, vocab, seed=seed, scale=2.5)
    z[1, :] = 0.25                                            # every id at tau: ties decide everything
    z[2, :] = np.where(rng.random(vocab) < 0.5, 1.0, -1.0)    # two weights, many ties at either
    z[3, :] = -1e30
    z[3, vocab // 2] = 3.0                                    # one id holds everything
    z[4, :] = np.round(z[4] * 4) / 4                          # a few dozen distinct weights
    z[5, :] *= 1e-6                                           # weights that differ in their last mantissa bits
    z[6, :] *= 12.0                                           # weights down to the cut-off
    z[7, : vocab // 3] = -np.inf
    z[8, vocab - 1] = z[8].max() + 2.0                        # the largest weight is the last id
    return z.astype(np.float32)


@pytest.mark.parametrize("vocab", [1, 255, 4097, 28672, 28673, 65536 + 3, 262144])
@pytest.mark.parametrize("top_p", [0.0, 1e-7, 0.5, 0.9, 0.999999])
def test_nucleus_matches_oracle(vocab, top_p):
    import torch
    import paper_2506_06122_amd as R
    z = hard_rows(vocab, seed=vocab) if vocab > 2 else np.zeros((9, vocab), np.float32)
    z = np.concatenate([z, z])                                # the same rows with other words
    x = workloads.uniform_words(len(z), seed=7)
    x[:9] = 2 ** 32 - 1                                       # the last id of the nucleus
    toks, _, sums = R.rollout_sample(torch.from_numpy(z).cuda(), 0.8, top_p, x)
    inv_t = sampler.inv_temperature(0.8)
    for r in range(len(z)):
        w = sampler.fixexp_weights(z[r], inv_t)
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"row {r}"
        assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, top_p), int(x[r])), f"row {r}"


def test_more_rows_than_the_nucleus_scratch_holds():
    import torch
    import paper_2506_06122_amd as R
    rows, vocab = 521, 28700                                  # batches of 512 and 9
    z = workloads.random_logits(rows, vocab, seed=3, scale=2.0)
    x = workloads.uniform_words(rows, seed=4)
    toks, _, _ = R.rollout_sample(torch.from_numpy(z).cuda(), 1.0, 0.9, x)
    for r in (0, 1, 255, 511, 512, 513, 520):
        assert int(toks[r]) == sampler.sample(z[r], np.float32(1.0), 0.9, int(x[r]))[0], f"row {r}"


@pytest.mark.parametrize("vocab", [256, 257, 1024, 4352, 4353])
@pytest.mark.parametrize("top_p", [0.9, 1.0])
def test_wavefronts_without_ids(vocab, top_p):
    """One workgroup per row skips the wavefronts whose 256 ids lie past the end: none, one id or all of the last ones."""
    import torch
    import paper_2506_06122_amd as R
    z = hard_rows(vocab, seed=vocab)
    x = workloads.uniform_words(len(z), seed=5)
    x[::2] = 2 ** 32 - 1
    toks, _, sums = R.rollout_sample(torch.from_numpy(z).cuda(), 0.8, top_p, x)
    inv_t = sampler.inv_temperature(0.8)
    for r in range(len(z)):
        w = sampler.fixexp_weights(z[r], inv_t)
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"row {r}"
        assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, top_p), int(x[r])), f"row {r}"


@pytest.mark.parametrize("rows,vocab", [(1, 151936), (40, 65536 + 3), (300, 28676)])
def test_rows_from_flat_to_spread(rows, vocab):
    """The bin that ends the nucleus holds from all ids down to a few: on either side of what a workgroup can list,
    with 16, 6 and 2 workgroups to a row (the scratch of a call holds 512 rows, so 300 are one batch)."""
    import torch
    import paper_2506_06122_amd as R
    for scale in np.geomspace(0.01, 4.0, 9):
        z = workloads.random_logits(rows, vocab, seed=11, scale=float(scale))
        x = workloads.uniform_words(rows, seed=12)
        toks, _, sums = R.rollout_sample(torch.from_numpy(z).cuda(), 1.0, 0.9, x)
        for r in {0, rows - 1}:
            w = sampler.fixexp_weights(z[r], sampler.inv_temperature(1.0))
            assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"scale {scale} row {r}"
            assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, 0.9), int(x[r])), f"scale {scale} row {r}"


@pytest.mark.parametrize("rows,vocab", [(64, 151936), (64, 32001), (256, 32001), (30, 262144)])
@pytest.mark.parametrize("top_p", [0.5, 0.9, 0.99])
def test_flat_rows_lines(rows, vocab, top_p):
    """Rows on either side of the line between the list and full sweeps (8 workgroups to a row with five tiles each, 4 with two, 2 with
    four, 16 with four), flat and spread ones in one call; 2, 4, 8 or one of the last workgroup's wavefronts take a part's list."""
    import torch
    import paper_2506_06122_amd as R
    scales = np.array([0.03, 0.1, 0.2, 0.35, 0.5, 0.6, 0.7, 0.8, 1.0, 1.5], np.float32)
    z = workloads.random_logits(rows, vocab, seed=21, scale=1.0) * scales[np.arange(rows) % 10, None]
    x = workloads.uniform_words(rows, seed=22)
    toks, _, sums = R.rollout_sample(torch.from_numpy(z).cuda(), 1.0, top_p, x)
    for r in range(20, 30):
        w = sampler.fixexp_weights(z[r], sampler.inv_temperature(1.0))
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"scale {scales[r % 10]}"
        assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, top_p), int(x[r])), f"scale {scales[r % 10]}"


@pytest.mark.parametrize("vocab", [1, 255, 4097, 28672, 28673, 65536 + 3, 262144])
def test_whole_vocabulary_matches_oracle(vocab):
    """top_p = 1 on the same rows: every weight counts, from 2^40 (equal maxima: the largest sums of a segment) down
    to the cut-off."""
    import torch
    import paper_2506_06122_amd as R
    z = hard_rows(vocab, seed=vocab) if vocab > 2 else np.zeros((9, vocab), np.float32)
    x = workloads.uniform_words(len(z), seed=7)
    toks, _, sums = R.rollout_sample(torch.from_numpy(z).cuda(), 0.8, 1.0, x)
    inv_t = sampler.inv_temperature(0.8)
    for r in range(len(z)):
        w = sampler.fixexp_weights(z[r], inv_t)
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"row {r}"
        assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, 1.0), int(x[r])), f"row {r}"


@pytest.mark.parametrize("rows,vocab", [(9, 16384), (9, 16385), (42, 28676), (128, 28676), (129, 28676), (171, 28676), (51, 147457),
                                        (64, 20 * 4096), (64, 20 * 4096 + 1), (64, 28 * 4096), (64, 28 * 4096 + 1), (4, 262144)])
@pytest.mark.parametrize("top_p", [0.9, 1.0])
def test_lines_between_the_ways_to_draw(rows, vocab, top_p):
    """64 and 65 segments (one wavefront draws, or the workgroup); 2 to 16 parts to a row, and 63 without a nucleus; the longest shares
    with one workgroup to a CU and the shortest with two (of 64 rows 20 tiles without a nucleus, 28 with one: 4 parts, then 8)."""
    import torch
    import paper_2506_06122_amd as R
    hard = hard_rows(vocab, seed=vocab)
    z = torch.from_numpy(hard).cuda()[torch.arange(rows, device="cuda") % len(hard)].contiguous()
    x = workloads.uniform_words(rows, seed=6)
    x[::5] = 2 ** 32 - 1
    toks, _, sums = R.rollout_sample(z, 0.8, top_p, x)
    inv_t = sampler.inv_temperature(0.8)
    weights = [sampler.fixexp_weights(h, inv_t) for h in hard]
    members = [sampler.nucleus(w, top_p) for w in weights]
    for r in range(rows):
        w = weights[r % len(hard)]
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"row {r}"
        assert int(toks[r]) == sampler.draw(w, members[r % len(hard)], int(x[r])), f"row {r}"


@pytest.mark.parametrize("vocab", [28673, 32001, 65536 + 3, 151936, 262144])
@pytest.mark.parametrize("top_p", [0.5, 0.9, 1.0])
def test_shares_left_to_the_last(vocab, top_p):
    """Parts of a row that do not wait for each other leave their shares to the one that finishes last: every phase, with lists
    and with full sweeps, by one workgroup or by some; and the calls that wait give the same bits, again and again."""
    import torch
    import paper_2506_06122_amd as R
    from paper_2506_06122_amd import binding
    z = hard_rows(vocab, seed=vocab)
    z = torch.from_numpy(np.concatenate([z, z[:3]])).cuda()
    x = workloads.uniform_words(len(z), seed=7)
    toks, lps, sums = R.rollout_sample(z, 0.8, top_p, x)
    inv_t = sampler.inv_temperature(0.8)
    for r in range(len(z)):
        w = sampler.fixexp_weights(z[r].cpu().numpy(), inv_t)
        assert int(sums[r]) == int(np.sum(w, dtype=np.uint64)), f"row {r}"
        assert int(toks[r]) == sampler.draw(w, sampler.nucleus(w, top_p), int(x[r])), f"row {r}"
    for again in range(4):
        for call in (binding.rollout_debug_sample_impatient, R.rollout_sample):
            got = call(z, 0.8, top_p, x)
            assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(got, (toks, lps, sums)))


@pytest.mark.parametrize("vocab,top_p,kernels", [(4096, 0.9, {"sample_kernel"}), (32768, 1.0, {"sample_max_kernel", "sample_rest_kernel<false>"}),
                                                 (32768, 0.9, {"sample_max_kernel", "sample_rest_kernel<true>"})])
def test_launches_are_timed_under_their_names(vocab, top_p, kernels):
    """A decode step's sampler in the timing records: one bracket to a launch, each with its logits."""
    import dataclasses
    from gpu_util import make_engine, scaled_weights
    shape = dataclasses.replace(workloads.SMALL_BF16, n_layers=1, ffn_dim=544, vocab=vocab)
    eng = make_engine(shape, scaled_weights(shape, seed=1), flags=4)
    toks, offs = workloads.make_prompts(1, 20, 20, shape.vocab, seed=4)
    eng.rollout_prefill(toks, offs, 3, np.full(3, 6, np.int32), top_p=top_p)
    for _ in range(4):
        eng.rollout_decode_step()
    got = {k["name"]: k for k in eng.rollout_kernel_stats() if k["name"].startswith("sample_")}
    eng.close()
    assert set(got) == kernels
    assert all(k["launches"] == 4 and k["bytes"] == 4 * 4.0 * 3 * vocab and k["ms"] > 0 for k in got.values())
