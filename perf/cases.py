"""Timing cases of libsparsecontract: what a user of the library has it do, through `driver.Contraction`.

A case names an expression, a sparse tensor (dims, stored entries, skew of each mode's coordinates), the ranks of the
dense factors, a precision and a schedule.  `prepare` draws the tensor and the factors on the GPU from a seed, hands them
to the library as sorted host coordinates (as a user's loader would) and keeps the planned contraction; `run` is one
execution of it, the part that an iterative decomposition or a serving loop repeats with the same sparse structure.

The sizes are those of the repository's benchmark workloads (`synth.CONFIGS`), scaled and made odd where the
benchmark has only round numbers.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2311_09549_amd import binding as sc
from paper_2311_09549_amd import synth
from paper_2311_09549_amd.driver import Contraction

DEVICE = "cuda:0"


def _case(name, kind, dims, nnz, ranks, skew, dtype="f32", schedule="fused", deterministic=False):
    """Plain values only: lists are written as text.  `skew`: per mode the exponent of a Zipf law, 0 = uniform."""
    case = dict(kind=kind, dims="x".join(str(d) for d in dims), nnz=nnz, ranks="x".join(str(r) for r in ranks),
                skew=",".join(str(s) for s in skew), dtype=dtype, schedule=schedule, deterministic=deterministic)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # a tiny TTM chain in double precision: one call is a few launches, so latency is what the user sees
        _case("ttmc3-tiny-f64", "ttmc3", (200, 200, 200), 8_000, (8, 8), (0, 0, 0), dtype="f64"),
        # the MTTKRP of a small decomposition, called many times per sweep; the library picks the schedule
        _case("mttkrp-small", "mttkrp3", (5_003, 3_001, 2_003), 99_991, (16,), (1.1, 1.1, 1.1), schedule="auto"),
        # a CP decomposition's MTTKRP on a large power-law tensor
        _case("mttkrp-20m", "mttkrp3", (50_000, 20_000, 10_000), 20_000_000, (32,), (1.2, 1.2, 1.2)),
        # a Tucker decomposition's TTM chain with the intermediate materialised
        _case("ttmc3-30m-fissioned", "ttmc3", (100_000, 50_000, 20_000), 30_000_000, (16, 16), (1.1, 1.1, 1.1), schedule="fissioned"),
        # the same chain at wider ranks, on chip, odd sizes throughout
        _case("ttmc3-wide", "ttmc3", (60_013, 30_011, 12_007), 6_000_011, (64, 32), (1.1, 1.1, 1.1)),
        # graph attention: a sampled product of node features, then aggregation over the neighbours
        _case("sddmm-spmm-16m", "sddmm_spmm", (1_000_000, 1_000_000), 16_000_000, (64, 64), (1.3, 0)),
        # the order-4 TTM chain, the largest workload of the benchmark
        _case("ttmc4-50m", "ttmc4", (10_000,) * 4, 50_000_000, (8, 8, 8), (1.1,) * 4),
        # the same under the two-level nest with both intermediates materialised, odd sizes
        _case("ttmc4-12m-fissioned", "ttmc4", (7_001, 8_003, 9_001, 6_007), 12_000_017, (8, 8, 8), (1.1,) * 4, schedule="fissioned"),
        # the core tensor of a Tucker decomposition (a factor on every mode), small and large core
        _case("ttmc-all-16", "ttmc_all", (40_000, 20_000, 8_000), 4_000_000, (16, 16, 16), (1.1, 1.1, 1.1), schedule="auto"),
        _case("ttmc-all-128", "ttmc_all", (40_000, 20_000, 8_000), 4_000_000, (128, 128, 128), (1.1, 1.1, 1.1), schedule="auto"),
        # a reproducible double-precision run: bit-identical from call to call, dense product behind the MTTKRP
        _case("mttkrp-gemm-f64-det", "mttkrp_gemm", (30_011, 12_007, 6_007), 3_000_017, (32, 64), (1.1, 1.1, 1.1), dtype="f64",
              deterministic=True),
        # ranks that are no power of two: the library's choice among the schedules that take them
        _case("ttmc3-odd-rank", "ttmc3", (20_011, 10_007, 5_003), 1_500_007, (12, 20), (1.1, 1.1, 1.1), schedule="auto"),
    ]


# most stored entries drawn per expression: the largest listed case of that expression, or of the one it is built on
_MOST = {"mttkrp3": 20_000_000, "ttmc3": 30_000_000, "sddmm_spmm": 16_000_000, "ttmc4": 30_000_000, "ttmc_all": 4_000_000,
         "mttkrp_gemm": 20_000_000, "sddmm_spmm_gemm": 16_000_000}
_MOST_OUT = 40_000 * 128 * 128   # elements of the output, or of the per-slice rows behind it, at most


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any expression, 5 thousand to 30 million entries, uniform or power-law, every rank the factored
    kernels are built for and now and then one that only the unfactored nest takes."""
    most_bytes = max(work(c)["bytes"] for c in listed())
    most_flops = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(sorted(_MOST))
        order = synth.KINDS[kind][1]
        dtype = "f64" if rng.random() < 0.2 else "f32"
        schedule = rng.choice(("fused", "fused", "fissioned", "auto"))
        deterministic = rng.random() < 0.2
        odd = rng.random() < 0.12 and kind in ("mttkrp3", "ttmc3", "ttmc4")
        nnz = _log_uniform(rng, 5_000, 1_500_000 if odd else _MOST[kind])
        if odd:   # rows of 16 bytes
            schedule, deterministic = "auto", False
            n = {"mttkrp3": 1, "ttmc3": 2, "ttmc4": 3}[kind]
            ranks = tuple(rng.choice((4, 12) if kind == "ttmc4" else (12, 20, 24, 36, 48)) for _ in range(n))
        elif kind == "mttkrp3":
            ranks = (rng.choice((8, 16, 32, 64, 128)),)
        elif kind == "ttmc3":
            ranks = (rng.choice((8, 16, 16, 32, 64, 128)), rng.choice((8, 16, 16, 32, 64, 128)))
        elif kind == "sddmm_spmm":
            ranks = (rng.choice((16, 32, 64, 128)),) * 2
        elif kind == "ttmc4":
            ranks = (16, 16, 16) if dtype == "f32" and rng.random() < 0.15 else (rng.choice((4, 8, 12, 16)), 8, 8)
            deterministic = deterministic and dtype == "f32" and ranks[1] == 8
        elif kind == "ttmc_all":
            ranks = tuple(rng.choice((16, 32, 64, 128)) for _ in range(3))
        elif kind == "mttkrp_gemm":
            ranks = (rng.choice((16, 32, 64)), rng.choice((16, 32, 64, 128)))
        else:
            ranks = (rng.choice((16, 32, 64)),) * 2 + (rng.choice((16, 32, 64, 128)),)
        lo, hi = {2: (2_000, 1_000_000), 3: (150, 100_000), 4: (40, 10_000)}[order]
        dims = tuple(_log_uniform(rng, lo, hi) for _ in range(order))
        if order == 2:
            skew = (rng.choice((0, 1.1, 1.3)), 0)
        else:
            skew = (rng.choice((0, 1.0, 1.1, 1.2)),) * order
        dense = 10 if not any(skew) else 300   # power laws fill their heads: leave room
        if math.prod(dims) < dense * nnz:
            continue
        row = math.prod(ranks[1:]) if kind == "ttmc_all" else ranks[-1] if order == 2 or kind.startswith("mttkrp") else math.prod(ranks)
        most = _MOST_OUT // 2 if dtype == "f64" else _MOST_OUT
        if dims[0] * row > most:
            continue
        case = _case("", kind, dims, nnz, ranks, skew, dtype, schedule, deterministic)
        cost = work(case)
        if cost["bytes"] <= most_bytes and cost["flops"] * (4 if dtype == "f64" else 1) <= most_flops:
            return case


def _fields(case):
    dims = tuple(int(d) for d in case["dims"].split("x"))
    ranks = tuple(int(r) for r in case["ranks"].split("x"))
    skew = tuple(float(s) for s in case["skew"].split(","))
    return dims, ranks, skew


def _zipf_weights(n, s):
    w = np.arange(1, n + 1, dtype=np.float64) ** (-s)
    return w / w.sum()


def _coords(dims, nnz, skew, gen):
    """nnz distinct coordinates, sorted (mode 0 slowest), as host int32 arrays; drawn on the GPU."""
    modes = []
    for n, s in zip(dims, skew):
        if s == 0:
            modes.append(None)
        else:
            cdf = torch.from_numpy(np.cumsum(_zipf_weights(n, s))).to(DEVICE)
            modes.append((cdf, torch.randperm(n, device=DEVICE, generator=gen)))
    have = torch.empty(0, dtype=torch.int64, device=DEVICE)
    while have.numel() < nnz:
        need = nnz - have.numel()
        count = int(need * 1.1) + 4096
        key = torch.zeros(count, dtype=torch.int64, device=DEVICE)
        for n, mode in zip(dims, modes):
            if mode is None:
                x = torch.randint(n, (count,), device=DEVICE, generator=gen)
            else:
                u = torch.rand(count, dtype=torch.float64, device=DEVICE, generator=gen)
                x = mode[1][torch.searchsorted(mode[0], u).clamp_(max=n - 1)]
            key.mul_(n).add_(x)
            del x
        have = torch.unique(torch.cat([have, key]))
        del key
    if have.numel() > nnz:
        keep = torch.randperm(have.numel(), device=DEVICE, generator=gen)[:nnz]
        have = have[torch.sort(keep).values]
    coords = []
    for n in reversed(dims):
        coords.append((have % n).to(torch.int32).cpu().numpy())
        have = have // n
    return coords[::-1]


def _inputs(case, seed):
    """Sorted host coordinates, values and factors, from the seed alone."""
    dims, ranks, skew = _fields(case)
    cfg = dict(kind=case["kind"], dims=dims, ranks=ranks, dtype=case["dtype"], nnz=case["nnz"])
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    coords = _coords(dims, case["nnz"], skew, gen)
    vals = (torch.rand(case["nnz"], dtype=dt, device=DEVICE, generator=gen) * 2 - 1).cpu().numpy()
    factors = [torch.randn(shape, dtype=dt, device=DEVICE, generator=gen).cpu().numpy() for shape in synth.factor_shapes(cfg)]
    return cfg, coords, vals, factors


def prepare(case, seed):
    cfg, coords, vals, factors = _inputs(case, seed)
    kind = cfg["kind"]
    sched = sc.schedule(case["schedule"], deterministic=case["deterministic"])
    return Contraction(synth.KINDS[kind][0], coords, vals, cfg["dims"], factors, sched, synth.output_shape(cfg))


def run(state):
    state.run()
    return state.out


def _add_up(count, width, into, part):
    """Row into[e] of the result is the sum of part(e) over all e, in chunks that fit the memory."""
    out = torch.zeros(count, width, dtype=torch.float64, device=DEVICE)
    step = max(1, (1 << 28) // width)
    for lo in range(0, into.numel(), step):
        at = slice(lo, lo + step)
        out.index_add_(0, into[at], part(at))
    return out


def exact(case, seed):
    """The output in double precision: sums over the last mode first, as the expressions factor."""
    cfg, coords, vals, factors = _inputs(case, seed)
    kind, dims = cfg["kind"], cfg["dims"]
    idx = [torch.from_numpy(c).to(DEVICE).long() for c in coords]
    v = torch.from_numpy(vals).to(DEVICE).double()
    f = [torch.from_numpy(x).to(DEVICE).double() for x in factors]
    if kind.startswith("sddmm"):
        i, j = idx
        out = _add_up(dims[0], f[2].shape[1], i,
                      lambda at: (v[at] * (f[0][i[at]] * f[1][j[at]]).sum(1))[:, None] * f[2][j[at]])
        return out @ f[3] if kind.endswith("gemm") else out
    # the factors on the modes 1, 2, ... from the leaf upwards: a row per (i, j, k), then a row per (i, j)
    lead = f[0] if kind == "ttmc_all" else None
    on = f[1:] if lead is not None else f[:len(dims) - 1]
    key = idx[0]
    for n, x in zip(dims[1:-1], idx[1:-1]):
        key = key * n + x
    nodes, up = torch.unique_consecutive(key, return_inverse=True)
    leaf = idx[-1]
    rows = _add_up(nodes.numel(), on[-1].shape[1], up, lambda at: v[at, None] * on[-1][leaf[at]])
    for mode in range(len(dims) - 2, 0, -1):
        here, key = nodes % dims[mode], nodes // dims[mode]
        if mode > 1:
            nodes, up = torch.unique_consecutive(key, return_inverse=True)
            count = nodes.numel()
        else:
            up, count = key, dims[0]
        below, g = rows, on[mode - 1]
        if kind.startswith("mttkrp"):
            rows = _add_up(count, g.shape[1], up, lambda at: g[here[at]] * below[at])
        else:
            rows = _add_up(count, g.shape[1] * below.shape[1], up,
                           lambda at: (g[here[at]][:, :, None] * below[at][:, None, :]).flatten(1))
    if lead is not None:
        rows = lead.t().contiguous() @ rows
    elif kind == "mttkrp_gemm":
        rows = rows @ f[2]
    return rows.reshape(synth.output_shape(cfg))


def _expected_prefixes(dims, skew, nnz):
    """Expected number of distinct coordinate prefixes of length 1, 2, ... among nnz draws: each mode's coordinates in
    groups of similar probability, sum over groups of size * (1 - exp(-nnz * p))."""
    size, prob = np.ones(1), np.ones(1)
    nodes = []
    for n, s in zip(dims[:-1], skew[:-1]):
        if s == 0:
            gs, gp = np.array([float(n)]), np.array([1.0 / n])
        else:
            w = _zipf_weights(n, s)
            edges = np.unique(np.concatenate([[0], np.geomspace(1, n, 60).astype(np.int64)]))
            gs = np.diff(edges).astype(np.float64)
            gp = np.add.reduceat(w, edges[:-1]) / gs
        size, prob = np.outer(size, gs).ravel(), np.outer(prob, gp).ravel()
        nodes.append(float(np.minimum(size, size * -np.expm1(-nnz * prob)).sum()))
    return nodes


def work(case):
    """Bytes: the stored entries with their coordinates, the nodes above them, every factor and the output, once.
    Flops: those of the factored nest (every stored entry and node times the width of what it is multiplied with)."""
    dims, ranks, skew = _fields(case)
    kind, nnz = case["kind"], case["nnz"]
    e = 8 if case["dtype"] == "f64" else 4
    cfg = dict(kind=kind, dims=dims, ranks=ranks)
    nodes = _expected_prefixes(dims, skew, nnz)
    nbytes = nnz * (4 + e) + 8 * sum(nodes)
    nbytes += e * sum(r * c for r, c in synth.factor_shapes(cfg)) + e * math.prod(synth.output_shape(cfg))
    if kind in ("mttkrp3", "mttkrp_gemm"):
        flops = 2 * ranks[0] * (nnz + nodes[1])
    elif kind == "ttmc3":
        flops = 2 * ranks[1] * nnz + 2 * ranks[0] * ranks[1] * nodes[1]
    elif kind in ("sddmm_spmm", "sddmm_spmm_gemm"):
        flops = nnz * (2 * ranks[0] + 1 + 2 * ranks[1])
    elif kind == "ttmc4":
        flops = 2 * ranks[2] * nnz + 2 * ranks[1] * ranks[2] * nodes[2] + 2 * math.prod(ranks) * nodes[1]
    else:
        flops = 2 * ranks[2] * nnz + 2 * ranks[1] * ranks[2] * nodes[1] + 2 * math.prod(ranks) * nodes[0]
    if kind in ("mttkrp_gemm", "sddmm_spmm_gemm"):
        flops += 2 * nodes[0] * ranks[-2] * ranks[-1]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times what the listed cases differ by from the same inputs run in double precision, and in double
    # precision from the same inputs under other tile sizes (rel 5e-7, max 8e-5; 5e-16, 4e-14).  The core tensor of
    # ttmc_all is one long sum over all slices: 1.3e-6 at 128 x 128 x 128.
    if case["dtype"] == "f64":
        return {"rel": 5e-15, "max": 4e-13}
    return {"rel": 5e-6 if case["kind"] == "ttmc_all" else 2e-6, "max": 3.5e-4}
