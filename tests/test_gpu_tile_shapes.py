"""Every tile shape of the projection kernel with every epilogue it is launched with, at the edges of its tiles and of its
ring of stages, whatever shape the planner would take there: against the same products in 64 bits."""
import numpy as np
import pytest

import paper_2506_06122_amd as R
from paper_2506_06122_amd import binding as B

SHAPES = B.rollout_debug_tile_shapes()   # (rows, columns, K groups, stages, grouped)
F32, SWIGLU, LSE = 0, 1, 3


def hi_lo(v):
    """fp32 [rows][k] -> bf16 [rows][k / 32][2][32], and the values that the two parts carry, in 64 bits"""
    import torch
    hi = v.bfloat16()
    lo = (v - hi.float()).bfloat16()
    rows, k = v.shape
    both = torch.stack([hi.view(rows, k // 32, 32), lo.view(rows, k // 32, 32)], 2).contiguous()
    return both, hi.double() + lo.double()


def fragments(w):
    """bf16 [n][k] -> [n / 16][k / 32][k % 32 / 8][n % 16][8]"""
    n, k = w.shape
    return w.view(n // 16, 16, k // 32, 4, 8).permute(0, 2, 3, 1, 4).contiguous()


def interleaved(gate, up):
    """rows of gate and up weights -> tiles of 8 gates and their 8 ups"""
    import torch
    f, k = gate.shape
    return torch.stack([gate.view(f // 8, 8, k), up.view(f // 8, 8, k)], 1).reshape(2 * f, k)


def guarded_buffer(n, dtype):
    """n elements and a margin behind them, all NaN"""
    import torch
    return torch.full((n + 4096,), float("nan"), dtype=dtype, device="cuda")


def lengths(kg, stages):
    """k-tiles of a split: 1 stage, 2, and around the ring's length; with two K groups also an odd last k-tile"""
    out = []
    for st in sorted({1, 2, stages - 1, stages, stages + 1}):
        out += [st * kg] + ([st * kg - 1] if kg > 1 else [])
    return [x for x in out if x > 0]


def random_operands(gen, m, n, k):
    import torch
    a = torch.randn(m, k, device="cuda", generator=gen)
    w = torch.randn(n, k, device="cuda", generator=gen).bfloat16()
    return a, w


def check(got, want, bound, what):
    import torch
    bad = ~((got - want).abs() <= bound)   # NaN: not written
    assert not bool(bad.any()), f"{what}: {int(bad.sum())} of {bad.numel()} values, first at {torch.nonzero(bad)[0].tolist()}"


def exact(values, w):
    """the product in 64 bits, and what 2 k fp32 additions (and one join per plane) can be off it: 2^-24 of the sum of magnitudes each"""
    want, size = values @ w.double().T, values.abs() @ w.double().abs().T
    return want, size * (2 * w.shape[1] + 16) * 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("shape", range(len(SHAPES)), ids=lambda i: "%dx%d" % SHAPES[i][:2])
def test_fp32_planes(shape):
    import torch
    bm, bn, kg, stages, _ = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(shape)
    rows, tiles, turn = [1, bm - 1, bm + 1, 2 * bm + 19], [1, max(1, bn // 16 - 1), bn // 16 + 1, 2 * (bn // 16) + 1], 0
    for per in lengths(kg, stages):
        for splits in (1, 2, 3):
            for k_tiles in {per * splits, max(splits, per * splits - 1)}:
                for i, m in enumerate(rows):
                    n = 16 * tiles[(i + turn) % 4]
                    a, w = random_operands(gen, m, n, 32 * k_tiles)
                    both, values = hi_lo(a)
                    out = guarded_buffer(splits * m * n, torch.float32)
                    planes = B.rollout_debug_tile_product(shape=shape, epilogue=F32, splits=splits, m=m, n=n, k=32 * k_tiles, a=both,
                                                          w=fragments(w), out=out)
                    what = f"{m} x {n} x {k_tiles} k-tiles in {splits} splits"
                    assert planes == -(-k_tiles // -(-k_tiles // splits)), what
                    assert bool(out[planes * m * n:].isnan().all()), what
                    want, bound = exact(values, w)
                    check(out[:planes * m * n].view(planes, m, n).double().sum(0), want, bound, what)
                turn += 1


def swiglu_reference(values, gate, up):
    import torch
    g, g_off = exact(values, gate)
    u, u_off = exact(values, up)
    s = g * torch.sigmoid(g)
    # |silu'| < 1.1; e^-g carries some 2^-21; two bf16 parts carry 2^-17
    return s * u, 1.1 * g_off * (u.abs() + u_off) + s.abs() * u_off + (s * u).abs() * 2.0 ** -16 + 1e-30


@pytest.mark.gpu
@pytest.mark.parametrize("shape", range(len(SHAPES)), ids=lambda i: "%dx%d" % SHAPES[i][:2])
def test_swiglu(shape):
    import torch
    bm, bn, kg, stages, _ = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(100 + shape)
    up4 = -(-bn // 64) * 64
    rows, cols, turn = [1, bm - 1, bm + 1, 2 * bm + 19], [64, up4, up4 + 64, 2 * up4 + 64], 0
    for k_tiles in lengths(kg, stages):
        for i, m in enumerate(rows):
            n = cols[(i + turn) % 4]
            a, w = random_operands(gen, m, n, 32 * k_tiles)
            both, values = hi_lo(a * 0.3)
            gate, up = w[:n // 2], w[n // 2:]
            out = guarded_buffer(m * n, torch.bfloat16)
            B.rollout_debug_tile_product(shape=shape, epilogue=SWIGLU, splits=1, m=m, n=n, k=32 * k_tiles, a=both,
                                         w=fragments(interleaved(gate, up)), out=out)
            what = f"{m} x {n} x {k_tiles} k-tiles"
            assert bool(out[m * n:].isnan().all()), what
            got = out[:m * n].view(m, n // 64, 2, 32).double().sum(2).reshape(m, n // 2)
            check(got, *swiglu_reference(values, gate, up), what)
        turn += 1


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [i for i, s in enumerate(SHAPES) if s[1] >= 128], ids=lambda i: "%dx%d" % SHAPES[i][:2])
def test_log_sum_exp_parts(shape):
    import torch
    bm, bn, kg, stages, _ = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(200 + shape)
    rows, tiles, turn = [1, bm - 1, bm + 1, 2 * bm + 19], [1, bn // 16 - 1, bn // 16 + 1, 2 * (bn // 16) + 1], 0
    for k_tiles in lengths(kg, stages):
        for i, m in enumerate(rows):
            n = 16 * tiles[(i + turn) % 4]
            a, w = random_operands(gen, m, n, 32 * k_tiles)
            both, values = hi_lo(a * 0.2)
            parts = -(-n // bn)
            target = torch.randint(-1, n, (m,), device="cuda", generator=gen, dtype=torch.int32)
            top, total, value = (guarded_buffer(c, torch.float32) for c in (parts * m, parts * m, m))
            B.rollout_debug_tile_product(shape=shape, epilogue=LSE, splits=1, m=m, n=n, k=32 * k_tiles, a=both, w=fragments(w),
                                         target=target, scale=0.5, part_max=top, part_sum=total, target_value=value)
            what = f"{m} x {n} x {k_tiles} k-tiles"
            assert bool(top[parts * m:].isnan().all() and total[parts * m:].isnan().all() and value[m:].isnan().all()), what
            want, bound = exact(values, w)
            want, bound = 0.5 * want, 0.5 * bound
            got = torch.logsumexp(top[:parts * m].view(parts, m).double() + total[:parts * m].view(parts, m).double().log(), 0)
            # a sum's n exponentials and additions: 2^-22 each, relative
            check(got, torch.logsumexp(want, 1), bound.max(1).values + (n + 16) * 2.0 ** -22, what)
            has = target >= 0
            at = target.clamp_min(0).long()[:, None]
            check(value[:m].double()[has], want.gather(1, at)[has, 0], bound.gather(1, at)[has, 0] + 1e-6 * want.abs().max(), what)
            assert bool(value[:m][~has].isnan().all()), what
        turn += 1


@pytest.mark.gpu
@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("shape", [i for i, s in enumerate(SHAPES) if s[4]], ids=lambda i: "%dx%d" % SHAPES[i][:2])
def test_row_blocks_of_groups(shape, gather):
    """The experts' launches: blocks of one row, a few, all but one and all rows of the tile, one unused."""
    import torch
    bm, bn, kg, stages, _ = SHAPES[shape]
    gen = torch.Generator(device="cuda").manual_seed(300 + shape)
    sizes, groups = [bm, 1, bm - 1, 5, bm], [2, 2, 0, 1, 1]
    ends = np.cumsum(sizes)
    m = int(ends[-1])
    index = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    blocks = dict(group_of_block=index(groups + [0]), block_begin=index([0] + ends.tolist()[:-1] + [0]),
                  block_end=index(ends.tolist() + [0]), n_blocks=6)
    up4 = -(-bn // 64) * 64
    for k_tiles in lengths(kg, stages):
        for n in (64, up4, up4 + 64, 2 * up4 + 64) if gather else (16, bn - 16, bn + 16, 2 * bn + 16):
            ws = [random_operands(gen, 1, n, 32 * k_tiles)[1] for _ in range(3)]
            a = random_operands(gen, 40 if gather else m, 16, 32 * k_tiles)[0] * 0.3
            both, values = hi_lo(a)
            what = f"{n} columns, {k_tiles} k-tiles"
            if gather:
                row_map = torch.randint(0, 40, (m,), device="cuda", generator=gen, dtype=torch.int32)
                packed = torch.stack([fragments(interleaved(w[:n // 2], w[n // 2:])) for w in ws])
                out = guarded_buffer(m * n, torch.bfloat16)
                B.rollout_debug_tile_product(shape=shape, epilogue=SWIGLU, splits=1, m=m, n=n, k=32 * k_tiles, a=both, w=packed, out=out,
                                             row_map=row_map, **blocks)
                got = out[:m * n].view(m, n // 64, 2, 32).double().sum(2).reshape(m, n // 2)
                values = values[row_map.long()]
            else:
                out = guarded_buffer(m * n, torch.float32)
                B.rollout_debug_tile_product(shape=shape, epilogue=F32, splits=1, m=m, n=n, k=32 * k_tiles, a=both,
                                             w=torch.stack([fragments(w) for w in ws]), out=out, **blocks)
                got = out[:m * n].view(m, n).double()
            assert bool(out[m * n:].isnan().all()), what
            for b, e, g in zip([0] + ends.tolist()[:-1], ends.tolist(), groups):
                ref = swiglu_reference(values[b:e], ws[g][:n // 2], ws[g][n // 2:]) if gather else exact(values[b:e], ws[g])
                check(got[b:e], *ref, f"{what}, rows {b} to {e}")


def test_launches_that_do_not_exist_are_refused():
    """No launch is made: the arguments are refused first (without a GPU as well)."""
    ok = dict(shape=0, epilogue=F32, splits=1, m=4, n=64, k=64, a=4096, w=4096, out=4096)
    lse = dict(out=None, target=4096, part_max=4096, part_sum=4096, target_value=4096, epilogue=LSE)
    blocks = dict(group_of_block=4096, block_begin=4096, block_end=4096, n_blocks=1)
    narrow = next(i for i, s in enumerate(SHAPES) if s[1] < 128)
    plain = next(i for i, s in enumerate(SHAPES) if not s[4])
    for bad in (dict(shape=-1), dict(shape=len(SHAPES)), dict(m=0), dict(n=40), dict(k=40), dict(k=0), dict(splits=0), dict(splits=3),
                dict(a=None), dict(w=None), dict(out=None), dict(epilogue=2), dict(epilogue=4), dict(epilogue=SWIGLU, splits=2),
                dict(epilogue=SWIGLU, n=32), dict(lse, shape=narrow), dict(lse, shape=5, target=None), dict(row_map=4096),
                dict(blocks, splits=2), dict(blocks, n_blocks=0), dict(blocks, block_end=None), dict(blocks, row_map=4096),
                dict(blocks, shape=plain, epilogue=SWIGLU, row_map=4096), dict(lse, shape=5, **blocks)):
        with pytest.raises(R.RolloutError) as e:
            B.rollout_debug_tile_product(**{**ok, **bad})
        assert e.value.code == B.E_INVAL, bad
