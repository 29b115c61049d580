"""Kernels that are picked by a rule on sizes, at the sizes where their tiles end: against the CPU oracle, every element."""
import os

import numpy as np
import pytest

import oracle as ora
from helpers import reduction_check

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1901_03771_amd import lazy as gr
    ctx = gr.Context()
    ctx.set_option("interp", 0)       # always the generated kernels
    ctx.set_option("plan_cache", 2)   # remembered plans and kernels against fresh ones
    ora.set_threads(min(16, os.cpu_count() or 1))
    yield gr, ctx, torch
    ctx.sync()
    ctx.close()


def both(env, program, **arrays):
    gr, ctx, torch = env
    keep = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in arrays.items()}
    got = program(gr, **{k: ctx.array(t) for k, t in keep.items()}).numpy()
    ref = program(ora, **{k: ora.array(v) for k, v in arrays.items()}).numpy()
    assert got.shape == ref.shape and got.dtype == ref.dtype
    return got, ref


def planned(env, program, **arrays):
    gr, ctx, torch = env
    code = {np.dtype(f32): gr.GR_F32, np.dtype(np.int32): gr.GR_I32}
    return program(gr, **{k: ctx.spec(v.shape, code[v.dtype]) for k, v in arrays.items()}).plan()


def positive(shape, seed):
    return (np.random.default_rng(seed).random(shape) + 0.25).astype(f32)


# outputs: below and at a group of four, ragged groups, one block, several blocks, blocks of the whole workgroup;
# reduced lengths: none, one, one batch of loads and its neighbours, one launch and two
@pytest.mark.parametrize("shape,axis", [
    ((1, 5), 0), ((2, 4), 0), ((7, 3), 0), ((8, 1027), 0), ((9, 65), 0), ((257, 257), 0), ((1025, 514), 0), ((5000, 24), 0),
    ((2, 1 << 20), 0), ((33, 40001), 0), ((1200, 33000), 0), ((20011, 90), 0), ((100000, 3), 0), ((6, 70, 9), 1), ((3, 2000, 130), 1),
    ((40, 6, 50, 7), (0, 2)), ((50, 30, 6), (0, 1)), ((0, 300), 0)])
def test_column_reductions(env, shape, axis):
    a = positive(shape, 7)
    assert " lanes=" in planned(env, lambda xp, a: xp.sum(a * a, axis=axis), a=a)
    if 0 not in shape:
        a.reshape(-1)[:: max(1, a.size // 5)] = -3.5
        for op in ("max", "min"):
            got, ref = both(env, lambda xp, a: getattr(xp, op)(a, axis=axis), a=a)
            assert np.array_equal(got, ref), op
        a = np.abs(a)
    got, ref = both(env, lambda xp, a: xp.sum(a * a, axis=axis), a=a)   # positive terms: 1e-5 of every element
    assert reduction_check(got, ref)[0].all()
    i = np.random.default_rng(8).integers(-2**31, 2**31 - 1, shape, dtype=np.int64).astype(np.int32)
    got, ref = both(env, lambda xp, i: xp.sum(i, axis=axis), i=i)
    assert np.array_equal(got, ref)


def test_column_reductions_keep_infinities_and_nan(env):
    a = positive((3000, 70), 9)
    a[5, 0], a[2999, 69], a[17, 33], a[18, 33] = np.inf, np.nan, np.inf, -np.inf
    for op in ("sum", "max", "min"):
        got, ref = both(env, lambda xp, a: getattr(xp, op)(a, axis=0), a=a)
        assert reduction_check(got, ref)[0].all(), op


# outputs that fill the chip by themselves: short ranges in one batch, whole batches of four and what is left of them, blocks of 64 elements
# and beside them, ragged rows; operands of one and two arrays, strided groups of outputs
@pytest.mark.parametrize("shape,axis", [((3, 1 << 18), 0), ((16, 1 << 17), 0), ((17, 131077), 0), ((65, 65536), 0), ((270, 32768), 0), ((515, 65536), 0), ((600, 16500), 0), ((530, 70001), 0),
                                        ((70, 64, 1024), 1), ((40, 130, 1030), 1), ((3, 300, 30000), 1)])
def test_wide_column_reductions(env, shape, axis):
    a, b = positive(shape, 23), positive(shape, 24)
    b.reshape(-1)[::7] *= -1.0
    got, ref = both(env, lambda xp, a: xp.sum(a, axis=axis), a=a)   # positive terms: 1e-5 of every element
    assert reduction_check(got, ref)[0].all()
    for op in ("max", "min"):
        got, ref = both(env, lambda xp, a, b: getattr(xp, op)(a * b, axis=axis), a=a, b=b)
        assert np.array_equal(got, ref), op
    i = np.random.default_rng(25).integers(-2**31, 2**31 - 1, shape, dtype=np.int64).astype(np.int32)
    got, ref = both(env, lambda xp, i: xp.sum(i, axis=axis), i=i)
    assert np.array_equal(got, ref)


# Signed values summed in chains of c additions leave a relative error of u sqrt(c / 6), u = 2^-24 (an addition's error is uniform
# in u times the partial sum).  c: blocks of 64 where the outputs fill the chip (chains of 256 to 4096 before), at most 256 elsewhere.
@pytest.mark.parametrize("shape,c", [((2048, 65536), 64), ((1600, 100000), 64), ((700, 70001), 64), ((4096, 30000), 256), ((30000, 4000), 256), ((16384, 2048), 256), ((200000, 300), 256)])
def test_column_sums_do_not_chain_additions(env, shape, c):
    gr, ctx, torch = env
    x = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(26))
    assert (" wide" in gr.sum(ctx.array(x), axis=0).plan()) == (c == 64)
    got = gr.sum(ctx.array(x), axis=0).torch().double()
    want = sum(part.double().sum(0) for part in x.chunk(16, 0))
    assert float((got - want).norm() / want.norm()) < 2.0**-24 * (c / 6) ** 0.5


# columns: ragged and whole groups of four, narrow arrays, one tile and a little more; rows: below, at and beside a patch.
# `kinds`, of a long program, a short one and a stencil: L lanes numbered over groups of columns, o tiles whose last groups overlap, - others
@pytest.mark.parametrize("shape,kinds", [((2, 5), "Lo"), ((2, 3), "--"), ((3, 4), "--"), ((5, 6), "Lo-"), ((17, 9), "Loo"), ((4, 257), "Lo"), ((63, 63), "ooo"), ((66, 1027), "LLL"), ((1031, 1028), "LLL"),
                                         ((70, 1501), "LLo"), ((4100, 1537), "LLo"), ((3000, 3000), "--o"), ((2001, 340), "L-o"), ((3, 65, 7), "oo"), ((5, 130, 1030), "LL"), ((2, 3, 4, 5), "Lo"), ((70001, 33), "Loo")])
def test_maps_of_ragged_rows(env, shape, kinds):
    a, b = positive(shape, 10), positive(shape[-1:], 11)
    long, short = (lambda xp, a, b: xp.sqrt(a * b + 1.0) / (a + b)), (lambda xp, a, b: a * b + 1.0)
    stencil = lambda xp, a: a[2:, 2:] - a[:-2, :-2] * a[1:-1, 1:-1]
    runs = [(long, dict(a=a, b=b)), (short, dict(a=a, b=b))] + ([(stencil, dict(a=a))] if len(shape) == 2 and min(shape) > 4 else [])
    routes = ""
    for prog, arrays in runs:   # operations that round once: the same bits
        plan = planned(env, prog, **arrays)
        routes += "L" if "lanes over groups" in plan else "o" if "overlapping" in plan else "-"
        got, ref = both(env, prog, **arrays)
        assert np.array_equal(got, ref)
    assert routes == kinds


@pytest.mark.parametrize("shape", [(40, 9), (66, 1027), (1031, 1030)])
def test_in_place_maps_of_ragged_rows(env, shape):
    # a value that reads the elements it overwrites is computed once per element
    gr, ctx, torch = env
    a = positive(shape, 12)
    t = torch.from_numpy(a.copy()).cuda()
    A, B = ctx.array(t), ora.array(a.copy())
    for X in (A, B):
        X[:] = X * X + 0.5
        X[1:-1, 1:] = X[1:-1, 1:] * 3.0
    assert np.array_equal(A.numpy(), B.numpy()) and np.array_equal(t.cpu().numpy(), B.numpy())


# pairs of rows: a lane per row of the longer operand; row lengths around the groups of four and the lane groups of the
# general kernel (whose order of additions is kept), few and many rows of the other operand, either operand the longer one,
# workgroups along the longer one that are fewer than the chiplets, a multiple of their number, beside one, and many.  `kernels`: of squared
# distances with and without a matrix added to them, of a maximum of minima and of an i32 sum: P the pairs' kernel, - the general one
@pytest.mark.parametrize("n,c,d,kernels", [
    (256, 4, 2, "----"), (257, 5, 4, "----"), (300, 7, 5, "----"), (1000, 19, 16, "----"), (1001, 33, 17, "----"), (4099, 6, 31, "----"), (511, 64, 33, "----"), (2049, 9, 63, "----"),
    (700, 3, 64, "----"), (5, 1030, 12, "----"), (260, 260, 54, "PP--"), (260, 260, 64, "----"),
    (32768, 4, 2, "-P--"), (32768, 5, 4, "-P--"), (28001, 5, 7, "-P--"), (65536, 4, 16, "PPPP"), (20001, 14, 9, "PPPP"), (4099, 65, 24, "PPPP"), (363, 362, 64, "PP--"), (300, 1030, 17, "PPPP"),
    (1030, 300, 17, "PPPP"), (1100, 1030, 25, "PP-P"), (1030, 1100, 33, "PP-P"), (40001, 33, 63, "PP-P"), (65536, 18, 65, "----"), (400000, 3, 16, "----"), (5, 70000, 31, "PP--")])
def test_rows_over_pairs(env, n, c, d, kernels):
    gr, ctx, torch = env
    a, b, w = positive((n, d), 13), positive((c, d), 14), positive((n, c), 15)

    def squares(xp, a, b):
        diff = a - b
        return xp.sum(diff * diff, axis=2)

    def distances(xp, a, b, w):
        return xp.sqrt(squares(xp, a, b)) + w

    def route(program, **arrays):
        return "P" if "pairs:" in planned(env, program, **arrays) else "-"

    largest = lambda xp, a, b: xp.max(xp.minimum(a, b), axis=2)
    products = lambda xp, i, j: xp.sum(i * j, axis=2)
    i, j = (np.random.default_rng(16 + k).integers(-2**31, 2**31 - 1, s, dtype=np.int64).astype(np.int32) for k, s in enumerate(((n, 1, d), (1, c, d))))
    arrays = dict(a=a[:, None, :], b=b[None, :, :], w=w)
    two = dict(a=a[:, None, :], b=b[None, :, :])
    assert route(distances, **arrays) + route(squares, **two) + route(largest, **two) + route(products, i=i, j=j) == kernels
    got, ref = both(env, distances, **arrays)
    assert reduction_check(got, ref)[0].all()
    other = gr.Context()
    other.set_option("interp", 2)      # the byte-code interpreter: the same bits
    keep = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in arrays.items()}
    assert np.array_equal(distances(gr, **{k: other.array(t) for k, t in keep.items()}).numpy(), got)
    other.sync()
    other.close()
    got, ref = both(env, squares, **two)
    assert reduction_check(got, ref)[0].all()
    got, ref = both(env, largest, **two)
    assert np.array_equal(got, ref)
    got, ref = both(env, products, i=i, j=j)
    assert np.array_equal(got, ref)


# sums of squares over rows: every count of lanes, rows that do not fill them, short of one position and over several
@pytest.mark.parametrize("shape", [(700, 1), (500, 3), (300, 7), (1000, 30), (65, 64), (33, 250), (40, 1027), (9, 5000), (5, 16384)])
def test_row_sums_of_squares(env, shape):
    gr, ctx, torch = env
    a = positive(shape, 21)
    a[0, -1], a[1, 0], a[2, 0], a[3, 0], a[4, 0] = np.inf, np.nan, 2e19, -1e-30, -np.inf   # (a square that overflows, one that underflows)
    other = gr.Context()
    other.set_option("interp", 2)
    t = torch.from_numpy(a).cuda()
    for program in (lambda xp, a: xp.sum(a * a, axis=1), lambda xp, a: xp.sum(xp.square(a), axis=1) + 0.5, lambda xp, a: a * a / xp.sum(a * a, axis=1, keepdims=True),
                    lambda xp, a: xp.sum((a - 0.25) ** 2, axis=1) / (xp.sum(a, axis=1) + 1.0)):
        got, ref = both(env, program, a=a)
        assert reduction_check(got, ref)[0].all()
        assert np.array_equal(program(gr, other.array(t)).numpy(), got, equal_nan=True)    # the interpreter: the same bits
    other.sync()
    other.close()


# partial results of 1024 outputs and more: splits just below the several lanes per output and at them, one round of them and more, a last
# workgroup of one output
@pytest.mark.parametrize("shape,splits", [((3840, 1024), 15), ((4096, 1024), 16), ((40000, 1024), 64), ((30000, 1025), 103), ((5000, 2049), 39)])
def test_partial_results_of_many_columns(env, shape, splits):
    a = positive(shape, 22)
    assert f"splits={splits} " in planned(env, lambda xp, a: xp.sum(a, axis=0), a=a).replace("\n", " ") + " "
    got, ref = both(env, lambda xp, a: xp.sum(a, axis=0), a=a)
    assert reduction_check(got, ref)[0].all()
    a[7::11, 3::5] *= -1
    got, ref = both(env, lambda xp, a: xp.min(a, axis=0), a=a)
    assert np.array_equal(got, ref)
    i = np.random.default_rng(23).integers(-2**31, 2**31 - 1, shape, dtype=np.int64).astype(np.int32)
    got, ref = both(env, lambda xp, i: xp.sum(i, axis=0), i=i)
    assert np.array_equal(got, ref)
    gr, ctx, torch = env
    got = gr.var(ctx.array(torch.from_numpy(a).cuda()), 0).numpy()
    want = a.astype(np.float64).var(0)
    assert (np.abs(got - want) <= 60 * 2.0 ** -24 * want).all()   # (the bound of test_columns_with_their_squared_deviations)
    a[5, 0], a[shape[0] - 1, shape[1] - 1], a[17, 33], a[18, 33] = np.inf, np.nan, np.inf, -np.inf
    got, ref = both(env, lambda xp, a: xp.sum(a, axis=0), a=a)
    assert reduction_check(got, ref)[0].all()
    got = gr.var(ctx.array(torch.from_numpy(a).cuda()), 0).numpy()
    assert np.isnan(got[[0, 33, shape[1] - 1]]).all() and np.isfinite(got[1:33]).all()


# lines of a few lane groups: positions that stick out of the line by every count, one to four positions, both widths of
# group; lines that do not fill the last workgroup
@pytest.mark.parametrize("shape", [(3, 4), (17, 5), (40, 63), (33, 64), (37, 65), (50, 66), (21, 67), (16, 144), (7, 255), (5, 256), (9, 257), (100, 511), (6, 513),
                                   (1001, 703), (4, 1021), (3, 1024), (2, 9, 130), (40, 3), (5, 1025)])
def test_scans_of_short_lines(env, shape):
    a = positive(shape, 17)
    assert ("lines-in-lane-groups" in planned(env, lambda xp, a: xp.cumsum(a * 0.5 + 1.0, -1), a=a)) == (4 <= shape[-1] <= 1024)
    got, ref = both(env, lambda xp, a: xp.cumsum(a * 0.5 + 1.0, -1), a=a)   # positive terms: 1e-5 of every prefix
    assert reduction_check(got, ref)[0].all()
    for op in ("cummax", "cummin"):
        got, ref = both(env, lambda xp, a: getattr(xp, op)(a - 0.75, -1), a=a)
        assert np.array_equal(got, ref)
    b = a.copy()
    b.reshape(-1)[:: 97] = np.inf
    got, ref = both(env, lambda xp, a: xp.cumsum(a, -1), a=b)
    assert reduction_check(got, ref)[0].all()
    i = np.random.default_rng(18).integers(-2**31, 2**31 - 1, shape, dtype=np.int64).astype(np.int32)
    got, ref = both(env, lambda xp, i: xp.cumsum(i, -1), i=i)
    assert got.dtype == np.int64 and np.array_equal(got, ref)


# rows kept by 1024 lanes: one element more than 256 lanes keep, ragged, every count of positions, the first length
# beyond; one row and many.  `kept`: whether a softmax, a program that normalises one array and a program over two arrays stay in one kernel
@pytest.mark.parametrize("shape,kept", [((16, 16385), "RRR"), ((19, 20000), "RRR"), ((15, 20000), "RRR"), ((1, 20479), "RRR"), ((40, 25000), "RRR"), ((16, 33001), "RRR"), ((40, 36864), "RRR"),
                                        ((64, 40001), "RRR"), ((70, 45056), "R-R"), ((64, 49153), "R-R"), ((33, 53000), "R-R"), ((64, 57344), "R-R"), ((65, 61437), "R-R"), ((17, 65535), "R--"),
                                        ((16, 65536), "R--"), ((64, 65536), "R-R"), ((300, 65533), "R-R"), ((16, 65537), "---"), ((2, 8, 17000), "RRR")])
def test_programs_over_long_rows(env, shape, kept):
    gr, ctx, torch = env
    a, b = positive(shape, 19) * f32(3.0), positive(shape, 20)

    def softmax(xp, a):
        e = xp.exp(a - xp.max(a, axis=-1, keepdims=True))
        return e / xp.sum(e, axis=-1, keepdims=True)

    def normal(xp, a):       # positive terms only
        s = xp.sqrt(a) + a
        return s / xp.sqrt(xp.sum(s * s, axis=-1, keepdims=True)) + a * xp.max(s, axis=-1, keepdims=True)

    def product(xp, a, b):
        s = a * b + a
        return s / xp.sum(s * s, axis=-1, keepdims=True)

    other = gr.Context()
    other.set_option("interp", 2)      # the byte-code interpreter: the same bits
    routes = ""
    for prog in (softmax, normal, product, lambda xp, a: xp.log(xp.sum(xp.exp(a), axis=-1) + 1.0)):
        arrays = dict(a=a, b=b) if prog is product else dict(a=a)
        got, ref = both(env, prog, **arrays)
        assert reduction_check(got, ref)[0].all()
        routes += "R" if "row_threads=1024" in planned(env, prog, **arrays) else "-"
        if routes[-1] == "R":
            keep = {k: torch.from_numpy(v).cuda() for k, v in arrays.items()}
            assert np.array_equal(prog(gr, **{k: other.array(t) for k, t in keep.items()}).numpy(), got)
    assert routes[:3] == kept
    i = np.random.default_rng(20).integers(-2**31, 2**31 - 1, shape, dtype=np.int64).astype(np.int32)
    got, ref = both(env, lambda xp, i: i - xp.max(i, axis=-1, keepdims=True) + xp.min(i, axis=-1, keepdims=True), i=i)
    assert np.array_equal(got, ref)
    other.sync()
    other.close()


# (see test_column_sums_do_not_chain_additions: a lane adds up 16 positions of four elements, pairs first: an error below that of chains
# of 32; one chain of 64 elements was above it)
@pytest.mark.parametrize("shape", [(512, 65536), (512, 40001), (600, 33000)])
def test_long_row_sums_do_not_chain_additions(env, shape):
    gr, ctx, torch = env
    err = 0.0
    for seed in range(4):
        x = torch.randn(shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed))
        got, want = (gr.sum(ctx.array(x), axis=1) * 0.5).torch().double(), x.double().sum(1) * 0.5
        err += float((got - want).norm() / want.norm()) / 4
    assert err < 2.0**-24 * (32 / 6) ** 0.5


# small integers: every sum is exact in any order.  Extents below, at and beside the tiles of 64 x 64, 128 x 32 and 32 x 128, groups
# of four that stick out, sums of one step, of whole steps, of steps in flight and around them, sums split over workgroups
@pytest.mark.parametrize("m,k,n", [(4, 17, 4), (5, 19, 6), (724, 9, 740), (801, 12, 702), (33, 31, 35), (63, 32, 61), (64, 33, 64), (65, 64, 67), (70, 95, 130), (129, 96, 66), (100, 97, 31), (300, 128, 19),
                                   (131, 160, 32), (29, 129, 200), (32, 161, 129), (30, 1000, 300), (37, 4100, 41), (66, 2051, 200), (257, 515, 255), (8, 300, 5)])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_products_with_clamped_tiles(env, m, k, n, layout):
    gr, ctx, torch = env
    rng = np.random.default_rng(21)
    a = rng.integers(-4, 5, (m, k) if layout[0] == "n" else (k, m)).astype(f32)
    b = rng.integers(-4, 5, (k, n) if layout[1] == "n" else (n, k)).astype(f32)
    c, d = rng.integers(-9, 9, n).astype(f32), rng.integers(-9, 9, (m, n)).astype(f32)

    def prog(xp, a, b, c, d):
        return (a if layout[0] == "n" else xp.transpose(a)) @ (b if layout[1] == "n" else xp.transpose(b)) * 2.0 + c - d

    specs = [ctx.spec(v.shape) for v in (a, b, c, d)]
    assert "clamped" in prog(gr, *specs).plan()
    got, ref = both(env, prog, a=a, b=b, c=c, d=d)
    assert np.array_equal(got, ref)
    # the result in the middle of a guarded buffer; infinities stay in their rows and columns
    a[a.shape[0] // 2, a.shape[1] // 2] = np.inf
    ta, tb, tc, td = (torch.from_numpy(v).cuda() for v in (a, b, c, d))
    guard = torch.full((m * n + 128,), 7.0, device="cuda")
    out = guard[64:64 + m * n].view(m, n)
    prog(gr, *(ctx.array(t) for t in (ta, tb, tc, td))).materialize_into(out)
    assert (guard[:64] == 7.0).all() and (guard[64 + m * n:] == 7.0).all()
    ref = prog(ora, *(ora.array(v) for v in (a, b, c, d))).numpy()
    assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)


# blocks of 32 x 32 from registers: k over the waves of a workgroup (w, also split over workgroups) and waves side by side (r), on both sides of every rule; sums that
# leave waves without a share, end within a group of eight, a step and two steps; small integers: exact in any order
@pytest.mark.parametrize("m,k,n,way", [
    (33, 9, 65, "w"), (64, 15, 31, "w"), (1, 16, 40, "w"), (40, 17, 1, "w"), (100, 65, 97, "w"), (512, 384, 1024, "w"), (511, 129, 1000, "w"), (512, 385, 1024, "-"), (545, 64, 1024, "-"),
    (545, 31, 1022, "r"), (545, 33, 1022, "-"), (3130, 9, 3190, "r"), (3163, 9, 3163, "-"), (65, 30, 12000, "r"), (9000, 31, 70, "r"), (17000, 31, 32, "-"), (192, 2000, 320, "w"), (33, 9000, 30, "w"), (256, 400, 256, "-")])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_products_of_blocks_from_registers(env, m, k, n, way, layout):
    gr, ctx, torch = env
    rng = np.random.default_rng(24)
    a = rng.integers(-4, 5, (m, k) if layout[0] == "n" else (k, m)).astype(f32)
    b = rng.integers(-4, 5, (k, n) if layout[1] == "n" else (n, k)).astype(f32)
    c = rng.integers(-9, 9, n).astype(f32)

    def prog(xp, a, b, c):
        return (a if layout[0] == "n" else xp.transpose(a)) @ (b if layout[1] == "n" else xp.transpose(b)) * 2.0 + c

    if layout == "nn" or min(m, n) >= 4:    # (an operand of fewer than four rows that lie along its other dimension takes the general kernel)
        plan = prog(gr, *(ctx.spec(v.shape) for v in (a, b, c))).plan()
        assert ("w" if "k over waves" in plan else "r" if "from registers" in plan else "-") == way
    got, ref = both(env, prog, a=a, b=b, c=c)
    assert np.array_equal(got, ref)
    a[a.shape[0] // 2, a.shape[1] // 2] = np.inf      # stays in its row
    ta, tb, tc = (torch.from_numpy(v).cuda() for v in (a, b, c))
    guard = torch.full((m * n + 128,), 7.0, device="cuda")
    out = guard[64:64 + m * n].view(m, n)
    prog(gr, *(ctx.array(t) for t in (ta, tb, tc))).materialize_into(out)
    assert (guard[:64] == 7.0).all() and (guard[64 + m * n:] == 7.0).all()
    ref = prog(ora, *(ora.array(v) for v in (a, b, c))).numpy()
    assert np.array_equal(out.cpu().numpy(), ref, equal_nan=True)


def test_short_products_under_a_long_function_take_blocks(env):
    gr, ctx, torch = env
    for m, k, n, way in ((2100, 128, 700, True), (2100, 129, 700, False), (4096, 128, 4096, True)):
        rng = np.random.default_rng(25)
        a, b, c = rng.standard_normal((m, k)).astype(f32), rng.standard_normal((k, n)).astype(f32) * f32(0.1), rng.standard_normal(n).astype(f32)
        prog = lambda xp, a, b, c: xp.tanh(a @ b + c)
        assert ("from registers" in prog(gr, *(ctx.spec(v.shape) for v in (a, b, c))).plan()) == way
        t = [torch.from_numpy(v).cuda() for v in (a, b, c)]
        got = prog(gr, *(ctx.array(v) for v in t)).torch()
        exact = torch.tanh(t[0].double() @ t[1].double() + t[2].double())
        # (a sum of k products in two chains: k / 2 + 2 roundings of what |a| |b| + |c| adds up to, and two ulp of the result)
        bound = (k / 2 + 2) * 2.0 ** -24 * (t[0].double().abs() @ t[1].double().abs() + t[2].double().abs()) + 2.0 ** -22
        assert ((got.double() - exact).abs() <= bound).all()


def test_static_entry_near_the_scratch_limit_takes_fewer_partial_sums(env):
    # column sums whose partial results do not fit beside the stored prefix sums (16680000 of 16777216 bytes): still served
    gr, ctx, torch = env
    rows, cols = 13900, 300
    a = np.random.default_rng(22).integers(-3, 4, (rows, cols)).astype(f32)
    t = torch.from_numpy(a).cuda()
    prog = lambda: gr.sum(gr.cumsum(ctx.array(t), 1), axis=0)
    want = prog().torch()
    lazy = prog()
    lazy.compile()
    got = torch.empty(cols, device="cuda")
    assert gr.lib().gr_materialize_into_static(ctx._p, lazy.h, got.data_ptr(), cols * 4) == 0, ctx.last_error()
    assert torch.equal(got, want) and np.array_equal(got.cpu().numpy(), np.cumsum(a.astype(np.float64), 1).sum(0).astype(f32))


@pytest.mark.parametrize("rows,cols", [(13900, 300), (13900, 299), (4080, 1024), (64, 300)])
def test_column_sums_have_the_same_bits_from_every_entry_point(env, rows, cols):
    # near the limit of the static scratch array, where there is room for fewer partial results, as elsewhere
    gr, ctx, torch = env
    t = torch.randn(rows, cols, device="cuda", generator=torch.Generator(device="cuda").manual_seed(27))
    prog = lambda leaf: gr.sum(gr.cumsum(leaf, 1), axis=0)
    want = prog(ctx.array(t)).torch()
    lazy = prog(ctx.array(t))
    lazy.compile()
    got = torch.empty(cols, device="cuda")
    assert gr.lib().gr_materialize_into_static(ctx._p, lazy.h, got.data_ptr(), cols * 4) == 0, ctx.last_error()
    assert torch.equal(got, want)
    into = torch.empty(cols, device="cuda")
    prog(ctx.array(t)).materialize_into(into)
    assert torch.equal(into, want)
    leaf = ctx.array(t)
    replayed = torch.empty(cols, device="cuda")
    ctx.program(prog(leaf), [leaf]).run([t], replayed)
    assert torch.equal(replayed, want)


IN_PLACE = {   # destination and value of a slice assignment that reads its own destination elsewhere
    "five points": lambda u: (np.s_[1:-1, 1:-1], 3 * (u[1:-1, 1:-1] + u[:-2, 1:-1] + u[1:-1, 2:] + u[1:-1, :-2] + u[2:, 1:-1])),
    "corners": lambda u: (np.s_[1:-1, 1:-1], u[:-2, :-2] + u[2:, 2:] - u[:-2, 2:] + u[2:, :-2]),
    "from below": lambda u: (np.s_[:-1, :], u[1:, :] + u[:-1, :]),
    "from the left": lambda u: (np.s_[:, 3:], u[:, :-3] - u[:, 3:]),
    "from the right": lambda u: (np.s_[:, :-4], u[:, 4:] * 1),
    "far corner": lambda u: (np.s_[4:, 4:], u[:-4, :-4] * 2),
    "two corners": lambda u: (np.s_[2:-3, 3:-1], u[:-5, 4:] - u[5:, :-4]),
    "twice": lambda u: (np.s_[1:-1, 1:-1], 2 * u[:-2, 1:-1] - abs(u[2:, 2:])),
}


def in_place_launches(ctx):
    """Launches that saved the cells around tiles, and assignments of one launch (whose kernel's name starts like theirs)."""
    once = ctx.profile_read("gr_map_save_store")[0]
    return ctx.profile_read("gr_map_save")[0] - once, once


# one tile, tiles that end at, before and behind the box, rows shorter than a tile (several tile rows of lanes), one column of the last tile; both ways
@pytest.mark.parametrize("rows,cols", [(8, 20), (17, 66), (33, 257), (34, 258), (35, 259), (64, 263), (66, 514), (131, 300), (1030, 1282), (2500, 600), (4000, 24)])
@pytest.mark.parametrize("dtype", [f32, np.int32])
@pytest.mark.parametrize("launches", [1, 2])
def test_assignments_evaluated_in_place(env, rows, cols, dtype, launches):
    gr, ctx, torch = env
    ctx.set_option("assign_in_place", launches)
    ctx.set_option("profile", 1)
    try:
        for name, program in IN_PLACE.items():
            for window in (0, 1):   # the whole array, or a window that starts off a 16-byte boundary, whose surroundings stay
                a = np.random.default_rng(31).integers(-50, 50, (rows + 5 * window, cols + 6 * window)).astype(dtype)
                t = torch.from_numpy(a).cuda()
                cut = np.s_[2 * window:2 * window + rows, 3 * window:3 * window + cols]
                u, ref = ctx.array(t[cut]), a[cut]
                ctx.profile_reset()
                for _ in range(2):
                    box, value = program(u)
                    u[box] = value
                    box, value = program(ref)
                    ref[box] = value.copy()
                ctx.sync()
                # (along the rows only, in one column of tiles: nothing around a tile to save)
                nothing = name.startswith("from the") and cols < 260
                assert in_place_launches(ctx) in ([(0, 2)] if launches == 1 else [(2, 0), (0, 0)] if nothing else [(2, 0)]), (name, window)
                assert np.array_equal(t.cpu().numpy(), a), (name, window)
    finally:
        ctx.set_option("profile", 0)
        ctx.set_option("assign_in_place", 1)


# few tiles, in one launch: tiles that wait for the ones around them, that look once and save (nearly all of them then, and read what others
# saved), sweep after sweep; the most tiles of that way (512 for all of these values), and a row of tiles more
@pytest.mark.parametrize("rows,cols,once", [(70, 1030, True), (1000, 1000, True), (2040, 1900, True), (2054, 1900, False), (16380, 200, True), (16390, 200, False)])
@pytest.mark.parametrize("polls", [0, 1, 16, 1 << 20])
def test_assignments_in_place_whether_tiles_wait_or_save(env, rows, cols, once, polls):
    gr, ctx, torch = env
    ctx.set_option("assign_polls", polls)
    ctx.set_option("profile", 1)
    try:
        for name, program in IN_PLACE.items():
            a = torch.randint(-50, 50, (rows, cols), device="cuda", dtype=torch.int32)
            want, u = a.clone(), ctx.array(a)
            ctx.profile_reset()
            for sweep in range(4):
                box, value = program(u)
                u[box] = value
                box, value = program(want)
                want[box] = value.clone()
            assert torch.equal(a, want), name
            nothing = name.startswith("from the") and cols < 260
            assert in_place_launches(ctx) in ([(0, 4)] if once else [(4, 0), (0, 0)] if nothing else [(4, 0)]), name
    finally:
        ctx.set_option("profile", 0)
        ctx.set_option("assign_polls", 16)


def test_assignments_not_evaluated_in_place(env):
    # values that read another array as well, other strides, a destination read further away: copied back as before
    gr, ctx, torch = env
    a = np.random.default_rng(32).integers(-50, 50, (70, 300)).astype(f32)
    b = np.random.default_rng(33).integers(-50, 50, (70, 300)).astype(f32)

    def other(u, w):
        u[1:-1, 1:-1] = u[2:, 1:-1] + w[1:-1, 1:-1]

    def wide(u, w):
        u[:, 5:] = u[:, :-5] * 2

    def stepped(u, w):
        u[2:, ::2] = u[:-2, ::2] + 1

    def twice_turned(u, w):
        u[1:, 1:] = u[:-1, :-1].T.T * 3

    def overwritten_scalar(u, w):
        u[:, :] = u[3:4, 4:5] + u * 1

    ctx.set_option("profile", 1)
    for f in (other, wide, stepped, overwritten_scalar, twice_turned):
        x, y = a.copy(), a.copy()
        t, w = torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()
        ctx.profile_reset()
        f(ctx.array(t), ctx.array(w))
        ctx.sync()
        saved = ctx.profile_read("gr_map_save")[0]
        class Copy(np.ndarray):
            def __setitem__(self, key, value):
                np.ndarray.__setitem__(self, key, np.array(value))
        f(y.view(Copy), b)
        assert np.array_equal(t.cpu().numpy(), y), f.__name__
        assert saved == (1 if f is twice_turned else 0), f.__name__   # (transposed twice is not turned)
    ctx.set_option("profile", 0)


@pytest.mark.parametrize("n", [20, 64, 300])
def test_assignments_of_turned_values_and_to_turned_arrays(env, n):
    # the destination read across: copied back; a transposed view written from positions beside: the value is written
    # with the view's strides, its elements are not contiguous along its rows
    gr, ctx, torch = env
    programs = {
        "turned": lambda u, xp: (u, np.s_[1:, 1:], (u.T if xp is np else gr.transpose(u))[:-1, :-1] * 3),
        "turned onto itself": lambda u, xp: (u, np.s_[:, :], (u.T if xp is np else gr.transpose(u)) - u),
        "to a transposed view": lambda u, xp: ((u.T if xp is np else gr.transpose(u)), np.s_[1:, :], (u.T if xp is np else gr.transpose(u))[:-1, :] * 2),
    }
    ctx.set_option("profile", 1)
    for name, program in programs.items():
        a = np.random.default_rng(34).integers(-50, 50, (n, n)).astype(f32)
        t = torch.from_numpy(a.copy()).cuda()
        ctx.profile_reset()
        to, box, value = program(ctx.array(t), gr)
        to[box] = value
        ctx.sync()
        to, box, value = program(a, np)
        to[box] = value.copy()
        assert np.array_equal(t.cpu().numpy(), a), name
        assert ctx.profile_read("gr_map_save")[0] == 0, name
    ctx.set_option("profile", 0)


# sums of a column and of its squared deviations from one pass: rows below, at and beside a batch of eight per lane, lanes that meet in
# one step and in groups, several launches' worth of splits, one output per lane (fewer than four columns), several reduced dimensions.
# Bound: a lane joins at most 32 batches, each a tree of three levels, groups and splits of at most 64 each in eight chains:
# 32 + 3 + 2 * (8 + 3) roundings, and three in a term itself, 60 of 2^-24.
@pytest.mark.parametrize("shape,axis", [((2, 5), 0), ((3, 3), 0), ((8, 4), 0), ((9, 30), 0), ((33, 1027), 0), ((100, 17), 0), ((257, 2), 0), ((515, 64), 0), ((4099, 257), 0),
                                        ((70001, 90), 0), ((200003, 5), 0), ((40, 70, 33), 1), ((30, 20, 50), (0, 1))])
def test_columns_with_their_squared_deviations(env, shape, axis):
    gr, ctx, torch = env
    rng = np.random.default_rng(41)
    far = rng.standard_normal(shape).astype(f32) + f32(300)          # a mean far from zero
    out = rng.standard_normal(shape).astype(f32)
    out[(0,) * len(shape)] = 5000                                    # an outlier
    assert "fused-with" in planned(env, lambda xp, a: gr.var(a, axis), a=out)
    for a in (rng.random(shape).astype(f32), far, out, np.full(shape, 2.7, f32)):
        t = torch.from_numpy(a).cuda()
        got = gr.var(ctx.array(t), axis).numpy()
        want = a.astype(np.float64).var(axis)
        assert got.shape == want.shape and (np.abs(got - want) <= 60 * 2.0 ** -24 * want + 1e-12).all()
        # the sums keep their bits, and every entry point gives the same ones
        x = ctx.array(t)
        both_used = (x - gr.mean(x, axis, True)) / gr.sqrt(gr.var(x, axis, True) + 1e-5)
        ctx.set_option("moments", 0)
        apart = gr.sum(x, axis).numpy()
        ctx.set_option("moments", 1)
        m = gr.sum(x, axis)
        v = gr.var(x, axis)
        v.materialize()
        assert np.array_equal(m.numpy(), apart)
        lazy = gr.var(ctx.array(t), axis)
        lazy.compile()
        into = torch.empty(want.shape, device="cuda")
        assert gr.lib().gr_materialize_into_static(ctx._p, lazy.h, into.data_ptr(), into.numel() * 4) == 0, ctx.last_error()
        assert np.array_equal(into.cpu().numpy(), got)
        ctx.program(gr.var(x, axis), [x]).run([t], into)
        assert np.array_equal(into.cpu().numpy(), got)
        full = a.astype(np.float64)
        scale = np.sqrt(full.var(axis, keepdims=True) + 1e-5)
        want = (full - full.mean(axis, keepdims=True)) / scale
        # (the mean is a sum of the same depth: its rounding, over the deviation)
        assert (np.abs(both_used.numpy() - want) <= 60 * 2.0 ** -24 * (np.abs(full).max() / scale + np.abs(want))).all()


@pytest.mark.parametrize("arrays", [9, 12])
def test_columns_of_many_loads_with_their_squared_deviations(env, arrays):
    # one row at a time: against two passes
    gr, ctx, torch = env
    rng = np.random.default_rng(42)
    x = [ctx.array(torch.from_numpy(rng.random((1001, 130)).astype(f32)).cuda()) for _ in range(arrays)]

    def squares():
        def value():
            v = x[0] * 1
            for t in x[1:]:
                v = v + t * 0.5
            return v
        return gr.sum(gr.square(value() - gr.sum(value(), 0, True) / 1001), 0)

    one = squares()
    assert "fused-with" in one.plan()
    one = one.numpy()
    ctx.set_option("moments", 0)
    two = squares()
    assert "fused-with" not in two.plan()
    two = two.numpy()
    ctx.set_option("moments", 1)
    # (each within 60 roundings of the sum, as in test_columns_with_their_squared_deviations)
    assert (np.abs(one - two) <= 2 * 60 * 2.0 ** -24 * np.abs(two)).all()


def test_squared_deviations_of_values_that_are_not_finite_or_overflow(env):
    gr, ctx, torch = env
    for rows, cols in ((3, 9), (4, 13), (5, 2), (64, 13), (1000, 13), (1001, 3), (70001, 13), (300, 2050)):
        a = np.ones((rows, max(cols, 13)), f32)
        a[1, 0], a[2, 1], a[0, 2] = np.inf, np.nan, -np.inf
        a[:, 3] = 1e38                                # the sum overflows, the values are equal
        a[::2, 4], a[1::2, 4] = 3e38, -3e38           # differences overflow
        a[0, 5] = 0.0
        a[1:, 5] = 1e25                               # squares overflow
        a[:, 6], a[rows - 1, 6] = 3e38, -3e38         # the sum overflows, and differences do
        a[:, 7], a[1, 7] = -3e38, 3e38
        a[:, 8], a[rows // 2:, 8] = 3e38, -3e38       # parts of the sum are infinite, of either sign
        a[:, 9], a[1, 9], a[2, 9] = 3e38, -3e38, np.inf
        a[:, 10], a[0, 10], a[1, 10] = 2e38, -np.inf, -2e38
        a[:, 11], a[rows - 1, 11] = 1e37, -1e37
        a[:, 12], a[0, 12], a[rows - 1, 12], a[rows // 2, 12] = 3e38, np.inf, np.inf, np.inf
        if cols < 13:
            a = np.ascontiguousarray(np.roll(a, -6, 1)[:, :cols])
        else:
            a = np.tile(a, (1, cols // 13 + 1))[:, :cols].copy()
        t = torch.from_numpy(a).cuda()
        x = ctx.array(t)
        got = gr.var(x, 0).numpy()
        ctx.set_option("moments", 0)
        want = gr.var(x, 0).numpy()
        ctx.set_option("moments", 1)
        assert np.array_equal(got, want, equal_nan=True), (rows, cols, got[:13], want[:13])


# operands in three pieces: the smallest contraction, odd and even numbers of steps for the two groups of waves, edge tiles, several
# workgroups per tile; and what the pieces cannot hold.  The bound: K roundings at most per sum, over the sum of magnitudes.
@pytest.mark.parametrize("m,n,k", [(128, 128, 32), (128, 252, 48), (260, 128, 64), (300, 380, 80), (132, 248, 1040), (2100, 2300, 32), (2100, 2300, 48), (4096, 3584, 48)])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_products_loaded_straight_into_lds(env, m, n, k, layout):
    gr, ctx, torch = env
    rng = np.random.default_rng(51)
    a, b = rng.standard_normal((m, k)).astype(f32), rng.standard_normal((k, n)).astype(f32)
    ctx.set_option("gemm_clamped", 0)
    try:
        for kind in ("ordinary", "infinities", "small", "denormal", "largest"):
            x, y = a.copy(), b.copy()
            if kind == "infinities":
                x[m // 2, k // 2], y[k // 3, n // 3], y[0, n - 1] = np.inf, -np.inf, np.nan
            elif kind == "small":
                x *= f32(2.0 ** -118)          # products stay ordinary, last pieces do not
                y *= f32(2.0 ** 110)
            elif kind == "denormal":
                x *= f32(2.0 ** -130)
                x[::3] = 0
                y *= f32(2.0 ** 120)
            elif kind == "largest":
                x[1, 2], y[2, 1] = np.finfo(f32).max, 0.0
            ta, tb = (torch.from_numpy(np.ascontiguousarray(v.T if t == "t" else v)).cuda() for v, t in ((x, layout[0]), (y, layout[1])))
            A, B = ctx.array(ta), ctx.array(tb)
            out = (gr.transpose(A) if layout[0] == "t" else A) @ (gr.transpose(B) if layout[1] == "t" else B)
            assert "direct" in out.plan()
            got = out.numpy()
            with np.errstate(all="ignore"):
                want = x.astype(np.float64) @ y.astype(np.float64)
                bound = (np.abs(x).astype(np.float64) @ np.abs(y).astype(np.float64)) * (k * 2.0 ** -24) + 2.0 ** -149 * k
            fits = np.isfinite(want) & (np.abs(want) < 3e38)
            assert (np.abs(got - want)[fits] <= bound[fits]).all(), kind
            odd = ~np.isfinite(want)
            assert np.array_equal(got[odd], want[odd].astype(f32), equal_nan=True), kind
    finally:
        ctx.set_option("gemm_clamped", 1)


# a wave that meets a value the pieces cannot hold changes to float32 instructions: in the first step, in the last rows of blocks of the
# last but one step, in the last step of either group; sums that overflow keep their signs
@pytest.mark.parametrize("m,n,k", [(300, 380, 64), (300, 380, 400), (300, 380, 416), (2100, 2300, 176), (4096, 3584, 112)])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_products_change_to_float32_instructions_at_any_step(env, m, n, k, layout):
    gr, ctx, torch = env
    rng = np.random.default_rng(52)
    x, y = rng.standard_normal((m, k)).astype(f32), rng.standard_normal((k, n)).astype(f32)
    x[127::128], y[:, 127::128] = 0, 0
    x[127::128, k - 20] = f32(1.2345678e-35)
    y[k - 5, 127::128] = f32(1.7654321e30)
    x[5, 3], x[6, 3], y[3, 9] = 1e30, -1e30, 1e30
    ta, tb = (torch.from_numpy(np.ascontiguousarray(v.T if t == "t" else v)).cuda() for v, t in ((x, layout[0]), (y, layout[1])))
    A, B = ctx.array(ta), ctx.array(tb)
    ctx.set_option("gemm_clamped", 0)
    out = (gr.transpose(A) if layout[0] == "t" else A) @ (gr.transpose(B) if layout[1] == "t" else B)
    assert "direct" in out.plan()
    got = out.numpy()
    ctx.set_option("gemm_clamped", 1)
    X, Y = (torch.from_numpy(v).cuda().double() for v in (x, y))
    want, bound = (X @ Y).cpu().numpy(), (X.abs() @ Y.abs()).cpu().numpy() * (k * 2.0 ** -24)
    assert got[5, 9] == np.inf and got[6, 9] == -np.inf
    got[5:7, 9] = 0
    want[5:7, 9] = 0
    assert (np.abs(got - want) <= bound).all()
    # one product per sum: within a rounding of it
    assert (np.abs(got - want)[127::128] <= 2.0 ** -23 * np.abs(want[127::128])).all()


@pytest.mark.parametrize("m,k,n", [(2048, 2048, 2048), (3000, 1024, 2048), (4096, 1024, 4096)])
def test_products_with_a_few_values_the_pieces_cannot_hold_take_no_more_than_twice_the_time(env, m, k, n):
    import time
    gr, ctx, torch = env
    a, b, out = torch.randn(m, k, device="cuda"), torch.randn(k, n, device="cuda"), torch.empty(m, n, device="cuda")
    A, B = ctx.array(a), ctx.array(b)
    assert "direct" in (A @ B).plan()
    program = ctx.program(A @ B, [A, B])

    def best():
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            start = time.perf_counter()
            for _ in range(10):
                program.run([a, b], out)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - start)
        return min(times)

    ordinary = best()
    for value in (1e-35, float("inf"), 1e30):
        a[::37, ::41] = value
        assert best() <= 2 * ordinary, value


# one nonzero product per sum leaves nothing for errors to hide in: within one rounding of it, also where last pieces are denormal
# bfloat16 values, at the ends of what the pieces hold, and beyond; denormal products within three units of the last place (the small products
# of pieces are rounded to it one by one)
@pytest.mark.parametrize("m,n,k", [(300, 380, 64), (300, 380, 416), (2100, 2300, 176), (4096, 3584, 112)])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_products_of_one_term_are_rounded_once(env, m, n, k, layout):
    gr, ctx, torch = env
    rng = np.random.default_rng(53)

    def full(shape, low, high):   # all 24 bits, magnitudes from 2^low to 2^(high + 1)
        return (rng.choice([-1.0, 1.0], shape) * np.ldexp(1 + rng.integers(0, 1 << 23, shape) / 2.0 ** 23, rng.integers(low, high + 1, shape))).astype(f32)

    ctx.set_option("gemm_clamped", 0)
    for kind, a, b in (("ordinary", (-3, 3), (-3, 3)), ("denormal last pieces", (-110, -103), (100, 105)), ("just too small", (-112, -111), (100, 105)), ("small", (-51, -49), (-60, -50)),
                       ("almost denormal", (-64, -62), (-62, -60)), ("denormal products", (-66, -64), (-68, -64)), ("large", (46, 47), (46, 47)), ("just too large", (48, 49), (48, 49))):
        x, y = full((m, k), *a), np.zeros((k, n), f32)
        y[np.arange(n) * 7 % k, np.arange(n)] = full(n, *b)
        ta, tb = (torch.from_numpy(np.ascontiguousarray(v.T if t == "t" else v)).cuda() for v, t in ((x, layout[0]), (y, layout[1])))
        A, B = ctx.array(ta), ctx.array(tb)
        out = (gr.transpose(A) if layout[0] == "t" else A) @ (gr.transpose(B) if layout[1] == "t" else B)
        assert "direct" in out.plan()
        got = out.numpy()
        want = x[:, np.arange(n) * 7 % k].astype(np.float64) * y.sum(0, dtype=np.float64)
        assert (np.abs(got - want) <= 2.0 ** -24 * (1 + 2.0 ** -6) * np.abs(want) + (3 * 2.0 ** -149 if a[0] + b[0] < -120 else 0)).all(), kind
    ctx.set_option("gemm_clamped", 1)


@pytest.mark.parametrize("m,n,k", [(512, 640, 4096), (2100, 2300, 2048), (4096, 4096, 4096)])
def test_products_of_positive_operands_do_not_lean_to_one_side(env, m, n, k):
    # K / 2 roundings of a sum that grows evenly: 2^-24 / sqrt(3) times the root of K / 2 / 3, half as much again allowed
    gr, ctx, torch = env
    torch.manual_seed(54)
    a, b = torch.rand(m, k, device="cuda"), torch.rand(k, n, device="cuda")
    ctx.set_option("gemm_clamped", 0)
    out = ctx.array(a) @ ctx.array(b)
    assert "direct" in out.plan()
    got = torch.from_numpy(out.numpy()).cuda().double()
    ctx.set_option("gemm_clamped", 1)
    want = a.double() @ b.double()
    assert float((got - want).norm() / want.norm()) <= 1.5 * 2.0 ** -24 / 3 * (k / 2) ** 0.5


# products of any extents through the kernels that load their tiles straight into LDS: what is left of k after whole steps (also in the last
# part of a divided k, and with infinities there), last tiles that start before their place, next to nothing left of a tile
@pytest.mark.parametrize("m,n,k,split", [(129, 130, 33, 0), (255, 381, 47, 0), (385, 255, 63, 0), (513, 642, 207, 0), (301, 203, 1031, 0), (642, 257, 335, 2), (1157, 1283, 97, 3), (2050, 2047, 45, 0),
                                         (3999, 3997, 81, 0), (4093, 3842, 95, 0)])
@pytest.mark.parametrize("layout", ["nn", "tn", "nt", "tt"])
def test_direct_products_of_ragged_extents(env, m, n, k, split, layout):
    gr, ctx, torch = env
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    whole = lambda *shape: torch.randint(-4, 5, shape, generator=g, device="cuda").float()
    a, b, bias = whole(m, k), whole(k, n), whole(n)
    ta, tb = (v.t().contiguous() if t == "t" else v for v, t in ((a, layout[0]), (b, layout[1])))
    buf = torch.full((m * n + 8192,), -77.0, device="cuda")
    inner = buf[4096:4096 + m * n].view(m, n)
    ctx.set_option("gemm_clamped", 0)
    ctx.set_option("gemm_split", split)
    try:
        for odd in (False, True):
            if odd:
                ta[(k - 1, 5) if layout[0] == "t" else (5, k - 1)] = float("inf")
            A, B = ctx.array(ta), ctx.array(tb)
            out = (gr.transpose(A) if layout[0] == "t" else A) @ (gr.transpose(B) if layout[1] == "t" else B) + ctx.array(bias)
            if n % 128 == 0 or n % 128 > 64:   # (32-wide tiles where the last 128 columns are mostly empty)
                assert "tile=128x128 direct" in out.plan(), out.plan()
            out.materialize_into(inner)
            ctx.sync()
            A64, B64 = (ta.t() if layout[0] == "t" else ta).double(), b.double()
            want = (A64.contiguous() @ B64 + bias.double()).float()   # (whole numbers below 2^24: exact in any order)
            assert torch.equal(torch.nan_to_num(inner, nan=123.0), torch.nan_to_num(want, nan=123.0))
            assert bool((buf[:4096] == -77.0).all()) and bool((buf[4096 + m * n:] == -77.0).all())
    finally:
        ctx.set_option("gemm_clamped", 1)
        ctx.set_option("gemm_split", 0)


# a value that pieces cannot hold, in a row or column that only the last tile has: what that tile shares with the one before keeps the bits that it has
# without such a value, also where the last tile (the 257th and on of a chip that runs 256) ends long after the others
@pytest.mark.parametrize("m,n,layout", [(2049, 2176, "tn"), (2175, 2176, "tt"), (128, 32833, "nn"), (131, 250, "tn"), (390, 507, "tn"), (258, 255, "nn"), (190, 253, "tn")])
@pytest.mark.parametrize("value", [1e-35, 2.0 ** 50])
def test_what_ragged_tiles_share_is_stored_once(env, m, n, layout, value):
    gr, ctx, torch = env
    g = torch.Generator(device="cuda").manual_seed(m + n)
    k, m1, n1 = 331, (m - 1) // 128 * 128, (n - 1) // 128 * 128    # (the last tile's own first row and column: other rows and columns of their wave are shared)
    a, b = torch.randn(m, k, generator=g, device="cuda"), torch.randn(k, n, generator=g, device="cuda")

    def product():
        A, B = (ctx.array(v.t().contiguous() if t == "t" else v) for v, t in ((a, layout[0]), (b, layout[1])))
        out = (gr.transpose(A) if layout[0] == "t" else A) @ (gr.transpose(B) if layout[1] == "t" else B)
        assert "tile=128x128 direct" in out.plan(), out.plan()
        return out.torch()

    ctx.set_option("gemm_clamped", 0)
    try:
        want = product()
        if layout[0] == "t":
            a[m1, 5] = a[m1, 17] = value     # (in steps of both groups of waves)
        if layout[1] == "n":
            b[5, n1] = b[17, n1] = value
        for _ in range(20):
            got = product()
            assert torch.equal(got[:m1, :n1], want[:m1, :n1])
    finally:
        ctx.set_option("gemm_clamped", 1)
    exact = a.double() @ b.double()
    # (331 products in sums of at most 331 parts, the pieces' own error within one of them)
    assert ((got.double() - exact).abs() <= 332 * 2.0 ** -24 * (a.double().abs() @ b.double().abs())).all()


# down the columns of a few hundred to a few thousand rows: two chunks to just over as many as a lane takes, in its first and last column, at and around a workgroup's lanes
@pytest.mark.parametrize("rows,cols", [(300, 16381), (700, 9001), (1352, 15783), (2200, 7001), (2500, 7425), (5000, 3001), (40000, 257), (2600, 255)])
def test_chunk_totals_of_many_lines(env, rows, cols):
    gr, ctx, torch = env
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    whole = torch.randint(-6, 7, (rows, cols), generator=g, device="cuda")
    for dtype in (torch.float32, torch.int32):
        x = whole.to(dtype)
        out = gr.cumsum(ctx.array(x), 0)
        got = torch.from_numpy(out.numpy()).cuda()
        want = torch.cumsum(whole, 0)     # (whole numbers below 2^24: exact in any order)
        assert torch.equal(got.to(torch.int64), want), (dtype, out.plan() if not out.is_materialized else "")
