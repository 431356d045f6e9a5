"""GPU parity of s-segmented Top-k MLMC (uniform ladder k_l = s l, thousands of levels, Lemma 3.4 probabilities over
all of them) against the CPU oracle, bit for bit: norms of every band, drawn levels, the drawn segment, aggregate."""
import numpy as np
import pytest
import torch

import mlmc_workloads as W
import paper_2507_05508_amd as P
from oracle import mlmc as O
from gpu_util import check_topk_against_oracle, to_device

pytestmark = pytest.mark.gpu


def _run_and_check(G, s, dtype=P.MLMC_F32, steps=(0, 1, 2), seed=42, ld=None):
    M, d = G.shape
    plan = P.Plan(P.MLMC_STOPK, M, d, dtype, [s], None)
    ladder = O.stopk_ladder(d, s)
    assert plan.ladder == ladder and plan.L == len(ladder) - 1 and plan.sparse_capacity_worst == M * min(s, d)
    g = to_device(G, ld=ld)
    norms = P.mlmc_level_norms(plan, g)
    torch.cuda.synchronize()
    assert plan.status() == 0
    got = norms.cpu().numpy()
    for i in range(M):
        want, _ = O.level_norms_row(G[i], ladder)
        assert np.array_equal(got[i].view(np.uint64), np.array(want, dtype=np.float64).view(np.uint64)), f"row {i}: norms differ"
    for step in steps:
        msg = P.mlmc_compress_topk(plan, g, seed=seed, step=step)
        want = check_topk_against_oracle(plan, G, seed, step, msg, adaptive=True)
        assert plan.status() == 0
        assert np.array_equal(msg.norms.cpu().numpy().view(np.uint64), got.view(np.uint64))
        for use_tile in (True, False):
            out = P.mlmc_aggregate(plan, msg, 1.0 / M, use_tile_off=use_tile)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), O.aggregate_sparse(want, d, 1.0 / M).view(np.uint32))
        bits = P.mlmc_message_bits(plan, msg).cpu().numpy()
        assert bits.tolist() == [O.message_bits_topk(ladder, m["level"], d) for m in want]


@pytest.mark.parametrize("name,d,M,s", [("resnet18_topk", 3 * 8192 + 777, 3, 64), ("resnet50_adaptive_topk", 100_003, 2, 100),
                                         ("tiny_topk", 20_000, 2, 7), ("resnet18_topk", 40_000, 2, 1)])
def test_stopk_segmented_workloads(name, d, M, s):
    w = W.scaled(W.WORKLOADS[name], d=d, M=M)
    print(f"stopk {name} d={d} M={M} s={s}", flush=True)
    _run_and_check(W.generate(w), s)


def test_stopk_ties_zeros_denormals_and_padding():
    d = 2 * 8192 + 300
    G = np.stack(W.adversarial_rows(d))
    for s, ld in ((33, None), (1000, d + 3), (d, None), (d + 5, None), (d - 1, d + 1)):
        print(f"stopk adversarial s={s} ld={ld}", flush=True)
        _run_and_check(G, s, steps=(0, 5), ld=ld)


def test_stopk_bf16_rows():
    w = W.scaled(W.WORKLOADS["bert_adaptive_topk_bf16"], d=70_000, M=2)
    _run_and_check(W.generate(w), 512, dtype=P.MLMC_BF16)


def test_stopk_exponential_decay_draws_many_levels():
    """Assumption 3.5 input: the level probabilities decay geometrically, so repeated steps draw many distinct levels."""
    d, s = 4 * 8192, 32
    rng = np.random.default_rng(9)
    g = np.empty(d, dtype=np.float32)
    g[rng.permutation(d)] = (2.0 * np.exp(-0.5 * 0.0004 * np.arange(d))).astype(np.float32) * rng.choice(np.array([-1, 1], dtype=np.float32), size=d)
    G = np.stack([g, g[::-1].copy()])
    plan = P.Plan(P.MLMC_STOPK, 2, d, P.MLMC_F32, [s], None)
    gd = to_device(G)
    seen = set()
    for step in range(12):
        msg = P.mlmc_compress_topk(plan, gd, seed=3, step=step)
        want = check_topk_against_oracle(plan, G, 3, step, msg, adaptive=True)
        seen |= {m["level"] for m in want}
    assert len(seen) >= 10


def test_stopk_plan_validation():
    for bad in (dict(d=1000, s=0), dict(d=10_000_000, s=100)):   # s < 1; more than MLMC_MAX_SLEVELS levels
        with pytest.raises(P.MlmcError):
            P.Plan(P.MLMC_STOPK, 2, bad["d"], P.MLMC_F32, [bad["s"]], None, allocate=False)
    with pytest.raises(P.MlmcError):
        P.Plan(P.MLMC_STOPK, 2, 1000, P.MLMC_F32, [10], [0.5, 0.5], allocate=False)   # fixed p is not defined here


def _few_values(d, rng):
    """Most entries share a few magnitudes, so that many boundaries fall among equal keys and one key may hold a whole segment."""
    v = np.array([0.0, 1e-3, 1.0000001, 1.0000002, 3.5, 1e-42], dtype=np.float32)
    g = v[rng.integers(0, len(v), d)] * rng.choice(np.array([-1, 1], dtype=np.float32), d)
    g[:: 97] = rng.standard_normal(len(g[:: 97])).astype(np.float32)
    return g


def _misled_sample(d, rng):
    """Rows of 2^21 entries or more are sampled, every other block of 1024 of them: the sampled blocks are zero, the others lie in one
    coarse bucket of keys, so that a single bin holds a million distinct keys and most boundaries."""
    g = np.zeros(d, dtype=np.float32)
    even = (np.arange(d) >> 10) % 2 == 0
    g[even] = (1.0 + rng.random(int(even.sum())) * 0.03).astype(np.float32)
    return g


@pytest.mark.parametrize("what,d,s,dtype,ld", [
    ("normal", 4096 * 9, 9, "f32", None),              # 4096 levels: the most without a sort
    ("normal", 4097 * 9, 9, "f32", None),              # 4097: sorted
    ("normal", 4096, 1, "f32", None),                  # every entry a segment (short rows are sorted)
    ("normal", 8192, 2, "f32", None),                  # the shortest binned row, 4096 levels
    ("few", 8191, 2, "f32", None),
    ("normal", 300_001, 70_000, "f32", 300_003),       # segments of more than 2^16 entries, odd rows
    ("normal", 1025 * 64 - 1, 64, "f32", None),        # 1025 levels: two copies of the sums
    ("normal", 3, 2, "f32", None),
    ("few", 50_021, 37, "f32", None),
    ("few", 50_021, 9_000, "f32", None),
    ("few", 50_021, 37, "bf16", 50_023),
    ("misled", (1 << 21) + 777, 40_000, "f32", None),  # zones of more keys than LDS holds, with many boundaries each
])
def test_stopk_edges_of_the_binned_path(what, d, s, dtype, ld):
    rng = np.random.default_rng(d + s)
    make = {"normal": lambda: rng.standard_normal(d).astype(np.float32), "few": lambda: _few_values(d, rng), "misled": lambda: _misled_sample(d, rng)}[what]
    G = np.stack([make() for _ in range(8 if dtype == "bf16" else 2)])   # (fewer short 16-bit rows are sorted)
    dt = P.MLMC_F32
    if dtype == "bf16":
        dt = P.MLMC_BF16
        G = W.f32_to_bf16_bits(G)
    print(f"stopk binned {what} d={d} s={s} {dtype} ld={ld}", flush=True)
    _run_and_check(G, s, dtype=dt, steps=(0, 1), ld=ld)


@pytest.mark.parametrize("d,s,nnz,smallest", [(8192, 8191, 8191, 7), (9000, 4000, 8000, 1), (9000, 2000, 8000, 15), (40_000, 39, 39 * 1000, 3)])
def test_stopk_boundary_between_the_smallest_entries_and_zeros(d, s, nnz, smallest):
    """The non-zero entries fill whole segments, the least of them among the smallest subnormals, with zeros behind: no zero
    belongs to the last segment that has a norm."""
    rng = np.random.default_rng(d + s)
    G = np.zeros((2, d), dtype=np.float32)
    for r in range(2):
        at = rng.permutation(d)[:nnz]
        G[r, at] = (rng.standard_normal(nnz) + 3.0).astype(np.float32)
        G[r, at[: 2 - r]] = np.array([smallest, 20_000_000], dtype=np.uint32).view(np.float32)[: 2 - r]
    print(f"stopk subnormals before zeros d={d} s={s}", flush=True)
    _run_and_check(G, s, steps=(0, 1, 2, 3))


def _crowd(d, n, rng, key=0x3EB851EC):
    """n entries of one magnitude, the others spread far below them."""
    g = (rng.standard_normal(d) * np.exp(rng.uniform(-30, -10, d))).astype(np.float32)
    g[rng.permutation(d)[:n]] = np.array([key], dtype=np.uint32).view(np.float32)[0]
    return g * rng.choice(np.array([-1, 1], dtype=np.float32), d)


def _hidden(d, n, rng):
    """n distinct keys of one coarse bucket, in blocks that the sample passes over, among ordinary entries elsewhere."""
    g = rng.standard_normal(d).astype(np.float32)
    at = np.flatnonzero((np.arange(d) >> 10) % 2 == 0)[:n]
    g[at] = (1e-9 * (1.0 + rng.random(n) * 0.02)).astype(np.float32)
    return g


@pytest.mark.parametrize("what,d,s,dtype", [
    ("one", 8192, 2, "f32"), ("one", 8192, 2, "bf16"),                     # every boundary at one key
    ("one", 300_001, 300, "f32"), ("two", 300_001, 100, "f32"),
    ("two", 50_021, 37, "f32"), ("sixteen", 300_001, 77, "f32"),
    ("zeros", 16_384, 4, "f32"), ("zeros", 50_021, 37, "bf16"),
    ("crowd 2047", 100_003, 500, "f32"), ("crowd 2048", 100_003, 500, "f32"), ("crowd 2049", 100_003, 500, "f32"),
    ("crowd 65536", 100_003, 500, "f32"), ("crowd 81919", 100_003, 25, "f32"), ("crowd 81920", 100_003, 25, "f32"),
    ("crowd 81921", 100_003, 25, "f32"), ("crowd 131072", 150_001, 40, "f32"), ("crowd 131073", 150_001, 40, "f32"),
    ("hidden 60000", (1 << 21) + 5, 700, "f32"),                           # one workgroup, up to 16 keys to a sub-bin
    ("misled", (1 << 21) + 777, 513, "bf16"),                              # four keys in the widest bin
    ("misled", (1 << 21) + 777, 513, "f32"),                               # many workgroups, thousands of boundaries
])
def test_stopk_zones_of_many_entries(what, d, s, dtype):
    """Rows of few magnitudes and rows that the sample misjudges: bins of thousands of entries that hold boundaries, at the sizes
    where another kernel, or another number of workgroups, takes them."""
    rng = np.random.default_rng(d + s)
    sign = lambda: rng.choice(np.array([-1, 1], dtype=np.float32), d)
    kind, _, arg = what.partition(" ")
    if kind == "crowd":
        make = lambda: _crowd(d, int(arg), rng)
    elif kind == "hidden":
        make = lambda: _hidden(d, int(arg), rng)
    else:
        make = {"one": lambda: np.float32(0.37) * sign(), "two": lambda: rng.choice(np.array([1.0, 1.0000001], dtype=np.float32), d) * sign(),
                "sixteen": lambda: (rng.integers(1, 17, d) * 0.25).astype(np.float32) * sign(),
                "zeros": lambda: np.where(rng.random(d) < 0.9, 0.0, rng.standard_normal(d)).astype(np.float32),
                "misled": lambda: _misled_sample(d, rng)}[kind]
    G = np.stack([make() for _ in range(8 if dtype == "bf16" and d < 1 << 20 else 2)])   # (fewer short 16-bit rows are sorted)
    if dtype == "bf16":
        G = W.f32_to_bf16_bits(G)
    print(f"stopk zones {what} d={d} s={s} {dtype}", flush=True)
    _run_and_check(G, s, dtype=P.MLMC_BF16 if dtype == "bf16" else P.MLMC_F32, steps=(0, 1))


@pytest.mark.parametrize("L", [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 8191, 8192, 8193, 8192 + 33])
def test_stopk_draw_at_the_edges_of_its_stretches(L):
    """The running sums are taken sixteen levels at a time, in chunks of 8192, up to the one that settles the draw: rows whose draw ends
    anywhere (equal bands, a zero row), in the first levels (one large entry) and late (bands that differ little)."""
    rng = np.random.default_rng(L)
    G = np.stack([np.ones(L), np.zeros(L), np.r_[1e6, np.full(L - 1, 1e-6)], 1.0 + rng.random(L)]).astype(np.float32)
    print(f"stopk draw L={L}", flush=True)
    _run_and_check(G, 1, steps=(0, 1, 2, 3) if L < 1000 else (0, 1))


@pytest.mark.parametrize("what,M,d,s", [
    ("heavy", 16, 24_581, 50),        # one entry in a coarse bin carries most of a row: the forecast of the drawn level misses now and then
    ("heavy", 3, 8_192, 4_096),       # two levels
    ("loud", 2, 300_001, 300),        # the top segments lie in a few tiles, which are read whole
    ("normal", 2, 70_001, 23_334),    # three levels: a third of every tile
    ("normal", 4, 40_961, 41),        # a last block of one entry
    ("nan", 2, 20_011, 20),           # sums that are no numbers
])
def test_stopk_forecast_of_the_drawn_segment(what, M, d, s):
    """Messages whose entries the second read has marked, partly marked or not marked at all."""
    rng = np.random.default_rng(d + s)
    G = rng.standard_normal((M, d)).astype(np.float32)
    if what == "heavy":
        G = (np.tan(np.pi * (rng.random((M, d)) - 0.5)) ** 3).astype(np.float32)
    elif what == "loud":
        G[:, : d // 50] *= 1e4
    print(f"stopk forecast {what} M={M} d={d} s={s}", flush=True)
    if what == "nan":   # refused by the status word, and ended all the same
        G[0, 5], G[1, 7] = np.nan, np.inf
        plan = P.Plan(P.MLMC_STOPK, M, d, P.MLMC_F32, [s], None)
        P.mlmc_compress_topk(plan, to_device(G), seed=1, step=1)
        torch.cuda.synchronize()
        assert plan.status() & P.MLMC_DEV_NONFINITE
        return
    _run_and_check(G, s, steps=(0, 1, 2, 3))


@pytest.mark.parametrize("M,d,s,ties", [
    (2, 60_001, 20, False),       # zones of a few entries
    (1, 300_001, 100, False),     # of about ten
    (2, 600_001, 3_000, False),   # of up to 64 and more
    (2, 60_001, 40, True),        # boundaries among equal keys
])
def test_stopk_zones_of_at_most_a_wave(M, d, s, ties):
    """Zones with one boundary on both sides of one key per lane."""
    rng = np.random.default_rng(d + s)
    G = rng.standard_normal((M, d)).astype(np.float32)
    if ties:   # every key some twelve times, in zones of several keys
        G = np.repeat(G[:, : d // 12 + 1], 12, axis=1)[:, :d] * 1.0
        G = np.ascontiguousarray(rng.permuted(G, axis=1))
    print(f"stopk small zones M={M} d={d} s={s} ties={ties}", flush=True)
    _run_and_check(G, s, steps=(0, 1))
