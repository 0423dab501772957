"""GPU parity at the sizes where a kernel's split of the work has edges: remainders of its blocks, chunks and batches, the
first and last size of a dispatch rule, slices cut by chunk and tile boundaries.  Against the oracle, within the tolerance of
the other parity tests (1e-5 / 1e-12 times the sum of |partial products|)."""
import re

import numpy as np
import pytest
import torch

from paper_2311_09549_amd import binding as sc
from paper_2311_09549_amd import synth
from paper_2311_09549_amd.driver import Contraction

from helpers import assert_parity

pytestmark = pytest.mark.gpu


def _problem(kind, dims, lengths, ranks, dtype="f32", seed=0):
    """lengths: stored entries per slice; the other coordinates are drawn without repetition inside a slice."""
    rng = np.random.default_rng(seed)
    space = int(np.prod(dims[1:]))
    rows, keys = [], []
    for i, n in lengths:
        rows.append(np.full(n, i))
        keys.append(np.sort(rng.choice(space, size=n, replace=False)))
    key, cols = np.concatenate(keys), []
    for n in reversed(dims[1:]):
        cols.append(key % n)
        key = key // n
    coords = [np.concatenate(rows)] + cols[::-1]
    coords = [np.ascontiguousarray(c, dtype=np.int32) for c in coords]
    dt = np.float64 if dtype == "f64" else np.float32
    cfg = dict(kind=kind, dims=tuple(dims), nnz=coords[0].size, ranks=tuple(ranks), dtype=dtype, expr=synth.KINDS[kind][0])
    factors = [rng.standard_normal(s).astype(dt) for s in synth.factor_shapes(cfg)]
    return cfg, dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(dt), factors=factors)


def _run(cfg, data, which, deterministic=False):
    print(f"{cfg['kind']} {which} {cfg['dtype']} dims={cfg['dims']} ranks={cfg['ranks']} nnz={cfg['nnz']}", flush=True)
    con = Contraction(cfg["expr"], data["coords"], data["vals"], cfg["dims"], data["factors"],
                      sc.schedule(which, deterministic=deterministic), synth.output_shape(cfg))
    for n, f in enumerate(con.factors):   # rows start at multiples of 16 bytes: ranks that do not give that get a longer row
        step = 16 // f.element_size()
        if f.shape[1] % step:
            con.factors[n] = torch.nn.functional.pad(f, (0, -f.shape[1] % step), value=float("nan"))[:, : f.shape[1]]
    con.run()
    return con


def _check(oracle, cfg, data, which, deterministic=False):
    con = _run(cfg, data, which, deterministic)
    assert_parity(oracle, cfg, data, con.result())
    return con


# one slice over several tiles, slices that end at a chunk's or a tile's last entry, unit slices
LENGTHS = [(0, 1), (1, 63), (2, 64), (3, 65), (5, 831), (6, 2300), (7, 1), (8, 1), (9, 700)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind,ranks", [("ttmc3", (4, 4)), ("ttmc3", (12, 20)), ("ttmc3", (36, 32)), ("ttmc3", (5, 8)), ("mttkrp3", (4,)),
                                        ("mttkrp3", (12,)), ("mttkrp3", (260,)), ("ttmc4", (3, 4, 4)), ("ttmc4", (12, 12, 4)), ("ttmc4", (2, 6, 4))])
def test_unfactored_nest_blocks(oracle, kind, ranks, dtype):
    """Rows of one block, of a partly filled lane group, of more than a wavefront's blocks; ranks that are no multiple of 4."""
    dims = (11, 41, 97) if kind != "ttmc4" else (11, 13, 17, 19)
    cfg, data = _problem(kind, dims, LENGTHS, ranks, dtype)
    _check(oracle, cfg, data, "linear")


# rows of S over several tiles (first, inner and last ones), rows that end with a tile, rows of one entry between and after them
ROWS = [(0, 3), (1, 1), (2, 2048), (3, 5300), (4, 1), (5, 1024), (6, 2500), (8, 700)] + [(i, 1) for i in range(9, 60)] + [(60, 4097)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("width", [16, 32, 64, 128])
def test_sampled_product_tile_order(oracle, width, dtype):
    """Tiles inside one row (taken by column) and tiles over several rows, in numbers that the XCDs do not divide."""
    cfg, data = _problem("sddmm_spmm", (64, 6007), ROWS, (width, width), dtype)
    for which in ("fused", "fissioned"):
        _check(oracle, cfg, data, which)
        _check(oracle, cfg, data, which, deterministic=True)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("width", [16, 32, 64, 128])
def test_sampled_product_one_row(oracle, width, dtype):
    """A tile inside one row: fewer entries than lane groups, partly filled batches, a full tile, one entry in the next tile."""
    for n in (1, 7, 65, 513, 1023, 1024, 1025):
        cfg, data = _problem("sddmm_spmm", (5, 3001), [(3, n)], (width, width), dtype)
        for which in ("fused", "fissioned"):
            _check(oracle, cfg, data, which)


# slices of 1 .. 9 and 15 .. 18 fibers (distinct j, so that a slice has as many fibers as entries), dealt out to up to four sets of threads
FIBERS = [(i, n) for i, n in enumerate([1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 18, 1, 1, 1, 2, 3, 700, 9, 8])]


@pytest.mark.parametrize("dtype,ranks", [("f64", (8, 8)), ("f64", (16, 8)), ("f64", (8, 64)), ("f64", (32, 16)), ("f32", (8, 8)), ("f32", (8, 32))])
def test_order3_consumer_batches(oracle, dtype, ranks):
    """Whole and partial batches of fibers per slice in the general order-3 consumer, one set of threads and several."""
    cfg, data = _problem("ttmc3", (23, 1009, 1), FIBERS, ranks, dtype)
    data["coords"][2] = np.random.default_rng(1).integers(0, 53, cfg["nnz"]).astype(np.int32)
    cfg["dims"] = (23, 1009, 53)
    data["factors"][1] = np.random.default_rng(2).standard_normal((53, ranks[1])).astype(data["vals"].dtype)
    for which in ("fused", "fissioned"):
        _check(oracle, cfg, data, which)
        _check(oracle, cfg, data, which, deterministic=True)


# tiles of 1024: slices that take a few chunks of a tile, a whole wavefront's, several wavefronts' and a whole tile
HEAVY = [(0, 5), (1, 1000), (2, 19), (3, 256), (4, 70), (5, 300), (6, 398), (7, 3), (8, 3000), (9, 69), (10, 1024)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind,ranks", [("ttmc3", (4, 4)), ("ttmc3", (8, 4)), ("ttmc3", (16, 16)), ("ttmc3", (16, 32)), ("mttkrp3", (4,)), ("mttkrp3", (8,)),
                                        ("mttkrp3", (20,)), ("ttmc4", (1, 4, 4)), ("ttmc4", (4, 4, 8))])
def test_unfactored_nest_heavy_slices(oracle, kind, ranks, dtype):
    """Sums of slices over many chunks, from one lane per chunk (64 chunks in a wavefront) to a wavefront per chunk."""
    dims = (11, 41, 97) if kind != "ttmc4" else (11, 13, 17, 19)
    cfg, data = _problem(kind, dims, HEAVY, ranks, dtype)
    _check(oracle, cfg, data, "linear")


@pytest.mark.parametrize("dtype,ranks,kernel", [
    ("f32", (64, 80), "mfma"), ("f32", (32, 112), "mfma"), ("f32", (16, 96), "mfma"), ("f32", (128, 64), "mfma"),   # partial last block of 64 columns
    ("f32", (8, 12), "tiled"), ("f32", (128, 128), "tiled"), ("f64", (64, 128), "tiled"), ("f64", (8, 4), "tiled"),  # up to 64 KB of E in LDS
    ("f32", (64, 6), "valu"), ("f64", (16, 10), "valu"), ("f64", (128, 128), "valu")])                               # M no multiple of 4, E beyond it
def test_trailing_product_kernels(oracle, dtype, ranks, kernel):
    """Each kernel of the trailing product at one row, odd numbers of rows and remainders of its row blocks."""
    for rows in (1, 17, 64, 333):
        lengths = [(i, 1 + i % 5) for i in range(0, rows, 2)]
        cfg, data = _problem("mttkrp_gemm", (rows, 41, 97), lengths, ranks, dtype)
        con = _check(oracle, cfg, data, "fused")
        sc.plan_set_profiling(con.plan, True)
        con.run()
        torch.cuda.synchronize()
        assert sc.plan_kernel_times(con.plan)[-1][0] == f"trailing_gemm_{kernel}"


@pytest.mark.parametrize("dtype,L,MN,rows", [
    ("f32", 16, (8, 8), (1, 63, 64, 65)), ("f32", 32, (8, 16), (3, 130)), ("f32", 64, (16, 16), (61, 200)), ("f32", 128, (16, 16), (15, 67, 193)),  # 16 columns per wavefront
    ("f32", 16, (64, 64), (577, 700)), ("f32", 32, (128, 128), (193,)), ("f32", 64, (64, 64), (583,)), ("f32", 128, (128, 128), (201,)),           # 64
    ("f32", 16, (16, 16), (8300,)), ("f64", 16, (8, 8), (4099,)), ("f64", 8, (16, 8), (5001,))])                                                   # many chunks, small output
def test_core_tensor_reduction(oracle, dtype, L, MN, rows):
    """The reduction over the first mode: chunks that end inside a batch of slices, one wavefront's worth of columns and many, and
    the sum of the chunks with 16 and with 64 elements per workgroup."""
    for n in rows:
        cfg, data = _problem("ttmc_all", (n, 41, 97), [(i, 1 + i % 3) for i in range(0, n, 1 + n // 300)], (L,) + MN, dtype)
        _check(oracle, cfg, data, "fused")


@pytest.mark.parametrize("ranks,rows", [((64, 64, 64), (7633, 7680)), ((64, 32, 32), (30_529,)), ((128, 64, 64), (3815, 4001)), ((128, 128, 128), (993, 9633)), ((128, 16, 32), (30_530,))])
def test_core_tensor_reduction_in_parts(oracle, ranks, rows):
    """Products of 16 bits: slices that do not fill the last step, both forms of the sum, longer and shorter chunks; and an infinity in C, which
    reaches the outputs of its l and no others."""
    for n in rows:
        stored = range(0, n, 1 + n // 150) if ranks[0] == 64 else range(1, n - n // 9)   # (at 128 five sixths of the slices at least)
        cfg, data = _problem("ttmc_all", (n, 41, 97), [(i, 1 + i % 3 // 2) for i in stored], ranks, "f32")
        con = _check(oracle, cfg, data, "fused")
        sc.plan_set_profiling(con.plan, True)
        con.run()
        torch.cuda.synchronize()
        assert any(name == "ttmc_all_mode0_reduce_split" for name, _ in sc.plan_kernel_times(con.plan))
        con.factors[0][int(data["coords"][0][-1]), 5] = float("inf")
        con.run()
        bad = np.zeros(ranks[0], dtype=bool)
        bad[5] = True
        np.testing.assert_array_equal(~np.isfinite(con.result()).all(axis=(1, 2)), bad)


@pytest.mark.parametrize("what", ["positive", "constant", "infinite", "not a number", "largest", "small slices", "small C"])
@pytest.mark.parametrize("ranks,n", [((64, 64, 64), 7650), ((128, 128, 128), 995)])
def test_core_tensor_reduction_range(oracle, ranks, n, what):
    """Products of 16 bits where the error could add up to one side, and where their parts cannot hold the values: infinities, values that the largest bf16 does not
    reach, and values whose last bits are below the smallest (all alike, so that a lost bit is lost the same way in every slice)."""
    cfg, data = _problem("ttmc_all", (n, 41, 97), [(i, 1 + i % 3 // 2) for i in range(1, n - n // 9)], ranks, "f32")
    rng = np.random.default_rng(1)
    C, D, E = (rng.uniform(0.5, 1.5, f.shape).astype(np.float32) for f in data["factors"])
    if what not in ("positive", "infinite", "not a number", "largest"):
        C[:], D[:], E[:] = 1.2345, 1.3456, 1.4567
    vals = np.full(data["vals"].shape, 0.7, np.float32) if what != "positive" else rng.uniform(0.5, 1, data["vals"].shape).astype(np.float32)
    i, j = int(data["coords"][0][-1]), int(data["coords"][1][0])
    if what in ("infinite", "not a number"):
        C[i, 5] = np.inf if what == "infinite" else np.nan
        D[j, 3] = np.inf
    elif what == "largest":
        C[i - 40 : i, :] = np.float32(3.4e38)
        D *= np.float32(2.0**-60)
    elif what == "small slices":
        D *= np.float32(2.0**-61)
        E *= np.float32(2.0**-61)
    elif what == "small C":
        C *= np.float32(2.0**-121)
    data = dict(data, vals=vals, factors=[C, D, E])
    con = _run(cfg, data, "fused")
    sc.plan_set_profiling(con.plan, True)
    con.run()
    got = con.result().astype(np.float64)
    assert any(name == "ttmc_all_mode0_reduce_split" for name, _ in sc.plan_kernel_times(con.plan))
    with np.errstate(invalid="ignore"):
        ref = oracle.contract(cfg["kind"], data["coords"], vals, cfg["dims"], data["factors"])
    fine = np.isfinite(ref)
    np.testing.assert_array_equal(got[~fine], ref[~fine])
    # one sign: |sum| is the sum of the absolute products.  2-norm: four roundings; alike in every slice, roundings add up over the steps of a chunk
    err = np.linalg.norm(got[fine] - ref[fine]) / np.linalg.norm(ref[fine])
    assert err <= (4 * 2.0**-24 if what not in ("constant", "small slices", "small C") else 4e-6), err


# ---- slice products: steps, chunks (of 16 steps at these sizes, of 32 and 64 below), runs, sums over the runs of a workgroup ----
def _fibers(shape, seed=0):
    """shape: per slice a list of fiber lengths; every fiber's entries start at a drawn place of the last mode."""
    rng = np.random.default_rng(seed)
    J, K = max(len(f) for f in shape) + 3, max(max(f) for f in shape if f) + 5
    i, j, k = [], [], []
    for s, lens in enumerate(shape):
        for f, n in zip(np.sort(rng.choice(J, size=len(lens), replace=False)), lens):
            i.append(np.full(n, s)), j.append(np.full(n, f)), k.append(np.arange(n) + rng.integers(0, K - n + 1))
    coords = [np.concatenate(x).astype(np.int32) for x in (i, j, k)]
    return (len(shape) + 1, J, K), coords, rng


SHAPES = {
    "whole_chunks": [[16] * 64, [16] * 16, [16] * 15, [1] * 256, [4] * 64],   # every place of a chunk taken
    "short": [[1]] * 70 + [[1, 1]] * 5 + [[], [3, 1, 1, 2, 1]] + [[1] * 5] * 9,
    "long_fibers": [[700, 1, 33, 17], [15, 16, 17], [2048]],
    "heavy": [[2, 1], [1, 2, 3, 1] * 1500, [1]],   # one slice through many runs and workgroups
}


@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("ranks,classes", [((16, 16), "ful"), ((8, 8), "fu"), ((64, 32), "fu"), ((16, 128), "fu"), ((128, 16), "u"), ((64, 64), "fu"), ((128, 64), "u"),
                                           ((128, 128), "fu"), ((4, 4), "l"), ((20, 36), "l"), ((72, 12), "l"), ((3, 100), "l"), ((100, 124), "l")])
def test_slice_products(oracle, shape, ranks, classes):
    dims, coords, rng = _fibers(SHAPES[shape])
    cfg = dict(kind="ttmc3", dims=dims, nnz=coords[0].size, ranks=ranks, dtype="f32", expr=synth.KINDS["ttmc3"][0])
    factors = [rng.standard_normal(s).astype(np.float32) for s in synth.factor_shapes(cfg)]
    data = dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(np.float32), factors=factors)
    for which in ("fused", "fissioned", "linear"):
        if {"fused": "f", "fissioned": "u", "linear": "l"}[which] not in classes:
            continue
        for leaves in (0, 32):   # the built-in runs, and runs of eight steps
            sc.tuning_set("tile_leaves", leaves)
            try:
                _check(oracle, cfg, data, which)
            finally:
                sc.tuning_set("tile_leaves", 0)


def _poisoned(oracle, cfg, data, which):
    """Every output element of the reference that is finite is finite here, and right; the others are not finite here, nor (in one kernel) another value."""
    got = _run(cfg, data, which).result()
    clean = [np.nan_to_num(f, nan=0.0, posinf=0.0, neginf=0.0) for f in data["factors"]]   # a zero in the place adds nothing to the bound of the others
    with np.errstate(invalid="ignore"):
        ref = oracle.contract(cfg["kind"], data["coords"], data["vals"], cfg["dims"], data["factors"])
    bound = oracle.abs_bound(cfg["kind"], data["coords"], data["vals"], cfg["dims"], clean)
    fine = np.isfinite(ref)
    assert fine.any() and not fine.all()
    np.testing.assert_array_equal(np.isfinite(got), fine)
    assert np.all(np.abs(got[fine].astype(np.float64) - ref[fine]) <= 1e-5 * bound[fine])
    if which != "fissioned":   # (its first kernel, the leaf traversal, multiplies by masked zeros)
        np.testing.assert_array_equal(got[~fine], ref[~fine].astype(np.float32))


@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("ranks,classes", [((16, 16), "ful"), ((8, 8), "ful"), ((32, 16), "fu"), ((16, 32), "fu"), ((64, 32), "fu"), ((16, 128), "fu"), ((64, 64), "fu"),
                                           ((128, 16), "f"), ((128, 128), "fu"), ((3, 20), "l"), ((72, 12), "l"), ((100, 124), "l")])
def test_slice_products_with_infinities(oracle, ranks, classes, at):
    """An infinity or a NaN in every row of C or of D, a column of its own in each: only the outputs that refer to it are not finite.  Chunks end
    off the batch and runs inside a slice, so places that no child takes stand beside every kind of row."""
    for name in ("short", "heavy", "whole_chunks"):
        dims, coords, rng = _fibers(SHAPES[name])
        cfg = dict(kind="ttmc3", dims=dims, nnz=coords[0].size, ranks=ranks, dtype="f32", expr=synth.KINDS["ttmc3"][0])
        factors = [rng.uniform(0.5, 1.5, s).astype(np.float32) for s in synth.factor_shapes(cfg)]   # one sign: infinities stay infinities in any order
        if name == "short" or factors[at].shape[0] > 64:   # every row but, where that would leave no finite element, a few
            rows = np.arange(factors[at].shape[0]) if name == "short" else rng.choice(factors[at].shape[0], 3, replace=False)
        else:
            rows = np.arange(3)
        for n in rows:
            factors[at][n, n % factors[at].shape[1]] = [np.inf, np.inf, np.nan][n % 3]
        data = dict(coords=coords, vals=rng.uniform(0.5, 1, coords[0].size).astype(np.float32), factors=factors)
        for which in ("fused", "fissioned", "linear"):
            if {"fused": "f", "fissioned": "u", "linear": "l"}[which] in classes:
                _poisoned(oracle, cfg, data, which)


def test_slice_products_with_infinities_at_a_thread_s_end(oracle):
    """From rows of T only the last chunk of a planner thread's share is short: two shares, and a row of C that only the last child of the first one has."""
    counts = np.array(([1] * 7 + [2] * 5 + [5] * 9 + [2] * 3) * 4350 + [4] * 73950)   # 295,800 children in each half, not the same work: no run ends between them
    starts = np.concatenate([[0], np.cumsum(counts)])
    s = int(np.searchsorted(starts, starts[-1] // 2))
    rng = np.random.default_rng(0)
    i = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    j = (np.arange(starts[-1]) - starts[i]).astype(np.int32)
    j[starts[s] - 1] = 6
    coords = [i, j, rng.integers(0, 9, i.size).astype(np.int32)]
    cfg = dict(kind="ttmc3", dims=(len(counts), 7, 9), nnz=i.size, ranks=(8, 8), dtype="f32", expr=synth.KINDS["ttmc3"][0])
    factors = [rng.uniform(0.5, 1.5, x).astype(np.float32) for x in synth.factor_shapes(cfg)]
    factors[0][6, :] = np.inf
    data = dict(coords=coords, vals=rng.uniform(0.5, 1, i.size).astype(np.float32), factors=factors)
    assert ((counts[:s] + 3) // 4).sum() % 4 != 0   # the share's last batch of steps is not full
    _poisoned(oracle, cfg, data, "fissioned")


@pytest.mark.parametrize("least,cap", [(300_000, 32), (560_000, 64)])
@pytest.mark.parametrize("ranks,which", [((16, 16), "fused"), ((32, 32), "fused"), ((8, 8), "fissioned"), ((16, 16), "linear")])
def test_slice_products_longer_chunks(oracle, ranks, which, least, cap):
    """Chunks of 32 and 64 steps (with as many slices, and with 256 leaves in 64 steps), which take so many entries; above 512,000 the steps
    are listed by several threads, each from a first chunk of its own."""
    wide = ranks[0] * ranks[1] > 256
    for name, shape in SHAPES.items():
        once = sum(len(f) if which == "fissioned" else sum(f) for f in shape)
        if wide and name == "short" or which == "fissioned" and once * 4 < sum(map(sum, shape)):
            continue   # (400,000 slices of 4 KB; few fibers of many entries)
        dims, coords, rng = _fibers(shape * -(-least // once))
        cfg = dict(kind="ttmc3", dims=dims, nnz=coords[0].size, ranks=ranks, dtype="f32", expr=synth.KINDS["ttmc3"][0])
        factors = [rng.standard_normal(s).astype(np.float32) for s in synth.factor_shapes(cfg)]
        con = _check(oracle, cfg, dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(np.float32), factors=factors), which)
        slots = (least if which == "fissioned" else coords[0].size) / 4
        chunks = int(re.search(r"runs of (\d+) chunks", sc.plan_describe(con.plan)).group(1))
        if name == "whole_chunks" and which != "fissioned" or which == "linear" and name == "heavy":   # nearly every place is taken
            assert slots / cap <= chunks <= 1.25 * slots / cap + 8
        assert chunks >= slots / cap / 2


MTTKRPS = {   # 32,768 entries and more, most of them in slices of 160 and more
    "units": [[1] * n for n in (160, 200, 255, 256, 257, 700, 1, 9)] * 19,
    "lengths": [[1, 2, 3, 5, 6, 7, 12, 13, 40] * 4, [700, 1, 33], [6] * 64, [2] * 300, [1]] * 16,
    "heavy": [[1], [1, 2, 3, 1] * 4700, [1], [2, 1] * 100],   # one slice through many runs and workgroups
}


@pytest.mark.parametrize("dtype,R", [("f32", 16), ("f32", 32), ("f64", 16)])
@pytest.mark.parametrize("name", sorted(MTTKRPS))
def test_mttkrp_over_steps(oracle, name, dtype, R):
    """Pieces of fibers in eights and sixteens, chunks, runs inside slices."""
    dims, coords, rng = _fibers(MTTKRPS[name])
    cfg = dict(kind="mttkrp3", dims=dims, nnz=coords[0].size, ranks=(R,), dtype=dtype, expr=synth.KINDS["mttkrp3"][0])
    dt = np.float64 if dtype == "f64" else np.float32
    factors = [rng.standard_normal(s).astype(dt) for s in synth.factor_shapes(cfg)]
    data = dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(dt), factors=factors)
    for leaves in (0, 32):   # the built-in runs, and runs of eight steps
        sc.tuning_set("tile_leaves", leaves)
        try:
            con = _check(oracle, cfg, data, "fused")
        finally:
            sc.tuning_set("tile_leaves", 0)
    assert "slice products" in sc.plan_describe(con.plan)


@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("dtype,R", [("f32", 16), ("f32", 32), ("f64", 16)])
def test_mttkrp_over_steps_with_infinities(oracle, dtype, R, at):
    """An infinity or a NaN in rows of C or D reaches the outputs that refer to it only, and infinite sums stay infinite: also where a run begins inside a group,
    some of whose pieces end in the run before."""
    for name, shape in MTTKRPS.items():
        least = 540_000 if (dtype, R) == ("f32", 16) else 280_000   # chunks of 16 steps: runs begin inside them
        dims, coords, rng = _fibers(shape * -(-least // sum(map(sum, shape))))
        cfg = dict(kind="mttkrp3", dims=dims, nnz=coords[0].size, ranks=(R,), dtype=dtype, expr=synth.KINDS["mttkrp3"][0])
        dt = np.float64 if dtype == "f64" else np.float32
        factors = [rng.uniform(0.5, 1.5, s).astype(dt) for s in synth.factor_shapes(cfg)]   # one sign: infinities stay infinities in any order
        for n in range(factors[at].shape[0]):
            factors[at][n, n % (R // 2)] = np.nan if n % 16 == 5 else np.inf
        data = dict(coords=coords, vals=rng.uniform(0.5, 1, coords[0].size).astype(dt), factors=factors)
        for leaves in (0, 32):
            sc.tuning_set("tile_leaves", leaves)
            try:
                _poisoned(oracle, cfg, data, "fused")
            finally:
                sc.tuning_set("tile_leaves", 0)


@pytest.mark.parametrize("dtype,R", [("f32", 16), ("f32", 32), ("f64", 16)])
@pytest.mark.parametrize("least", [33_000, 200_000, 500_000, 600_000])
def test_mttkrp_over_steps_long_fibers(oracle, dtype, R, least):
    """Pieces of sixteen leaves, in chunks of 8 steps (whose pieces are of 8) and longer ones."""
    lengths = np.random.default_rng(1).integers(9, 41, size=least // 24)
    dims, coords, rng = _fibers([list(s) for s in np.array_split(lengths, least // 500)])
    assert coords[0].size >= 12 * lengths.size
    cfg = dict(kind="mttkrp3", dims=dims, nnz=coords[0].size, ranks=(R,), dtype=dtype, expr=synth.KINDS["mttkrp3"][0])
    dt = np.float64 if dtype == "f64" else np.float32
    factors = [rng.standard_normal(s).astype(dt) for s in synth.factor_shapes(cfg)]
    con = _check(oracle, cfg, dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(dt), factors=factors), "fused")
    assert "slice products" in sc.plan_describe(con.plan)


@pytest.mark.parametrize("least,slices", [(300_000, 1800), (1_100_000, 400)])
def test_mttkrp_over_steps_longer_chunks(oracle, least, slices):
    """Chunks of 16 and 32 steps, listed by one thread and by several."""
    cfg, data = _problem("mttkrp3", (slices + 3, 89, 97), [(i, least // slices + i % 7) for i in range(slices)], (32,))
    con = _check(oracle, cfg, data, "fused")
    assert "slice products" in sc.plan_describe(con.plan)


# ---- chains of order 4 from the leaves: pairs of steps, pieces of (i,j) fibers, chunks, runs ----
def _chain(shape, seed=0):
    """shape: per slice a list of (i,j) fibers, each a list of (i,j,k) fiber lengths; coordinates are drawn."""
    rng = np.random.default_rng(seed)
    fibers = [f for s in shape for f in s]
    J, K, P = max(map(len, shape)) + 3, max(map(len, fibers)) + 2, max(max(f) for f in fibers) + 5
    cols = ([], [], [], [])
    for i, sl in enumerate(shape):
        for j, f in zip(np.sort(rng.choice(J, size=len(sl), replace=False)), sl):
            for k, n in zip(np.sort(rng.choice(K, size=len(f), replace=False)), f):
                for c, x in zip(cols, (np.full(n, i), np.full(n, j), np.full(n, k), np.sort(rng.choice(P, size=n, replace=False)))):
                    c.append(x)
    return (len(shape) + 1, J, K, P), [np.concatenate(c).astype(np.int32) for c in cols], rng


CHAINS = {
    "singles": [[[1]] * n for n in (1, 2, 3, 4, 5, 8, 63, 64, 65, 255, 256, 257, 1)] + [[[1]]] * 80,   # odd steps at chunks' and slices' ends
    "children": [[[1] * n] for n in range(1, 13)] + [[[1] * 4] * 64, [[1] * 5, [1] * 6, [1]] * 9, [[1] * 300]],   # pieces of (i,j) fibers
    "lengths": [[[n] for n in range(1, 20)], [[3, 1, 1, 2, 1, 17, 4]] * 5, [[2], [1], [1], [1], [1], [5, 1]], [[16] * 4] * 4, [[40, 1]], [[700]], [[1, 15, 16, 17, 33]] * 3],
    "heavy": [[[1]], [[1, 3, 1], [1], [2], [1, 1]] * 900, [[1]]],   # one slice through many runs and workgroups
}


@pytest.mark.parametrize("name", sorted(CHAINS))
@pytest.mark.parametrize("L", [1, 4, 8, 13, 16])
def test_chain_of_order_4(oracle, name, L):
    dims, coords, rng = _chain(CHAINS[name])
    cfg = dict(kind="ttmc4", dims=dims, nnz=coords[0].size, ranks=(L, 8, 8), dtype="f32", expr=synth.KINDS["ttmc4"][0])
    factors = [rng.standard_normal(s).astype(np.float32) for s in synth.factor_shapes(cfg)]
    data = dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(np.float32), factors=factors)
    for leaves in (0, 32):   # the built-in runs, and runs of a batch
        sc.tuning_set("tile_leaves", leaves)
        try:
            con = _check(oracle, cfg, data, "fused")
        finally:
            sc.tuning_set("tile_leaves", 0)
    for n, f in enumerate(con.factors):   # rows too far apart for offsets by products of 24 bits
        con.factors[n] = torch.nn.functional.pad(f, (0, 128 - f.shape[1]), value=float("nan"))[:, : f.shape[1]]
    con.out.fill_(float("nan"))
    con.run()
    assert_parity(oracle, cfg, data, con.result())


@pytest.mark.parametrize("least,cap", [(300_000, 32), (560_000, 64)])
def test_chain_of_order_4_longer_chunks(oracle, least, cap):
    """Chunks of 32 and 64 steps; above 512,000 entries the steps are listed by several threads."""
    for name, shape in CHAINS.items():
        dims, coords, rng = _chain(shape * -(-least // sum(sum(map(sum, s)) for s in shape)))
        cfg = dict(kind="ttmc4", dims=dims, nnz=coords[0].size, ranks=(8, 8, 8), dtype="f32", expr=synth.KINDS["ttmc4"][0])
        factors = [rng.standard_normal(s).astype(np.float32) for s in synth.factor_shapes(cfg)]
        con = _check(oracle, cfg, dict(coords=coords, vals=rng.uniform(-1, 1, coords[0].size).astype(np.float32), factors=factors), "fused")
        assert int(re.search(r"runs of (\d+) chunks", sc.plan_describe(con.plan)).group(1)) >= coords[0].size / 4 / cap


@pytest.mark.parametrize("at", [0, 1, 2])
def test_chain_of_order_4_with_infinities(oracle, at):
    """Only the outputs that refer to a row with an infinity or a NaN are not finite."""
    for name, shape in CHAINS.items():
        dims, coords, rng = _chain(shape * -(-300_000 // sum(sum(map(sum, s)) for s in shape)))   # chunks of 32 steps: runs begin inside them
        cfg = dict(kind="ttmc4", dims=dims, nnz=coords[0].size, ranks=(8, 8, 8), dtype="f32", expr=synth.KINDS["ttmc4"][0])
        factors = [rng.uniform(0.5, 1.5, s).astype(np.float32) for s in synth.factor_shapes(cfg)]   # one sign: infinities stay infinities in any order
        for n in range(factors[at].shape[0]):
            factors[at][n, n % 4] = np.nan if n % 16 == 5 else np.inf
        data = dict(coords=coords, vals=rng.uniform(0.5, 1, coords[0].size).astype(np.float32), factors=factors)
        for leaves in (0, 32):   # runs of a batch begin inside children and groups
            sc.tuning_set("tile_leaves", leaves)
            try:
                _poisoned(oracle, cfg, data, "fused")
            finally:
                sc.tuning_set("tile_leaves", 0)


@pytest.mark.parametrize("which,dims,lengths,ranks", [
    ("fused", (9000, 41, 97), [(i, 17 + i % 7) for i in range(9000)], (64, 64)),               # 147 MB, slices of some length
    ("fused", (280_000, 41, 97), [(i, 1 + i % 3) for i in range(0, 280_000, 2)], (16, 16)),    # 287 MB, half of it zeroed
    ("linear", (500_000, 41, 97), [(i, 1 + i % 3) for i in range(0, 500_000, 2)], (12, 12)),   # the same at the edge of a tile
    ("fused", (26_000, 41, 97), [(i, 1 + i % 7) for i in range(0, 26_000, 2)], (64, 64)),      # 426 MB, short slices
    ("fused", (26_000, 41, 97), [(i, 1 + i % 7) for i in range(0, 26_000, 5)], (64, 64)),      # all of it zeroed: through the caches
    ("fissioned", (88_000, 41, 97), [(i, 1 + i % 7) for i in range(0, 88_000, 2)], (64, 16)),  # 360 MB
    ("fused", (88_000, 41, 97), [(i, 1 + i % 7) for i in range(0, 88_000, 2)], (64, 16))])     # the same through the caches
def test_slice_products_stored_past_the_caches(oracle, which, dims, lengths, ranks):
    """Outputs on the sides of the rule by which rows are stored with the non-temporal hint."""
    cfg, data = _problem("ttmc3", dims, lengths, ranks)
    _check(oracle, cfg, data, which)


# ---- tiles of few leaves: small problems and wide gathered rows; rows shared by several tiles ----
@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kind,dims,ranks,most", [("sddmm_spmm", (11, 4000), (16, 16), 64), ("sddmm_spmm", (11, 4000), (32, 32), 64), ("sddmm_spmm", (11, 4000), (64, 64), 64),
                                                  ("sddmm_spmm", (11, 4000), (128, 128), 64), ("mttkrp3", (11, 41, 97), (8,), 64), ("mttkrp3", (11, 41, 97), (128,), 64),
                                                  ("ttmc3", (11, 41, 97), (16, 16), 64), ("sddmm_spmm", (40, 40000), (64, 64), 192)])
def test_small_tiles(oracle, kind, dims, ranks, most, dtype, deterministic):
    lengths = LENGTHS if dims[0] == 11 else [(i, 30000 if i == 3 else 3000) for i in range(39)]
    cfg, data = _problem(kind, dims, lengths, ranks, dtype)
    con = _check(oracle, cfg, data, "fused", deterministic)
    first = sc.plan_tile(con.plan, 0)
    if not deterministic and not (kind == "ttmc3" and dtype == "f32"):   # the fp32 chain runs as slice products
        assert first[1] - first[0] <= most
    if kind == "sddmm_spmm":
        _check(oracle, cfg, data, "fissioned", deterministic)
