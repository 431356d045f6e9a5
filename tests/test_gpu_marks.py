"""Which rows have the entries of their message marked by an earlier read, and that the marks hold the whole message where a forecast has to hold:
the messages of the other tests are the same with and without them."""
import numpy as np
import pytest
import torch

import mlmc_workloads as W
import paper_2507_05508_amd as P
from gpu_util import check_topk_against_oracle, launched, to_device, u32
from oracle import mlmc as O

pytestmark = pytest.mark.gpu


def _align(n):
    return (n + 255) // 256 * 256


def _region(plan, nbytes, *behind):
    """Bytes of the plan's workspace that are followed by regions of the given sizes, up to its end."""
    at = plan.workspace_bytes - sum(_align(n) for n in behind) - _align(nbytes)
    return plan.ws[at:at + nbytes]


def _marks(plan):
    """Marks of a 32-bit plan: [M, entries / 4] bits."""
    words = -(-plan.d // plan.chunk) * plan.chunk // 256
    return _region(plan, 8 * words * plan.M).view(plan.M, 8 * words)


def _marks16(plan):
    """Marks of a 16-bit plan: [M, entries / 8] bits."""
    M, tiles = plan.M, plan.num_tiles
    return _region(plan, 64 * tiles * M, 4 * 4096 * tiles * M, 16 * tiles * M, 16 * tiles * M, 4 * (tiles + 1) * M, 8 * plan.L * M).view(M, 64 * tiles)


def _covered(marks, msg, per, whole):
    """Per row: are all entries of the message (of the row's first `whole` ones) marked?"""
    off = msg.row_off.cpu().numpy()
    out = []
    for i in range(marks.shape[0]):
        at = msg.idx[off[i]:off[i + 1]].long()
        at = at[at < whole] // per
        out.append(bool(((marks[i][at >> 3].int() >> (at & 7).int()) & 1).all()))
    return out


def _one_hot(M, L, level):
    p = torch.zeros((M, L), dtype=torch.float64, device="cuda")
    p[:, level - 1] = 1.0
    return p


@pytest.mark.parametrize("M,d,wide", [
    (2, 65_537, True), (2, 1 << 22, True), (3, 300_001, True),       # several rows: bands of any width
    (1, 65_537, False), (1, 300_001, False),                         # one row: up to an eighth of it
    (2, (1 << 22) + 1, False),                                       # longer ones the same
])
def test_bands_that_are_marked(M, d, wide):
    """Drawn bands of an eighth of a row and just above: marked, or left to the second read."""
    G = np.random.default_rng(d).standard_normal((M, d)).astype(np.float32)
    g = to_device(G)
    k = d // 100
    plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_F32, [10, k, k + d // 8, k + d // 8 + d // 8 + 1], None)
    for level in (1, 2, 3):
        plan.ws.fill_(0)
        print(f"marked bands {M}x{d} level {level}", flush=True)
        p = _one_hot(M, 3, level)
        msg = P.mlmc_compress_topk(plan, g, seed=3, step=0, p=p)
        assert plan.status(informational=True) == 0
        marks = _marks(plan)
        if level < 3 or wide:
            assert all(_covered(marks, msg, 4, d)) and float((marks != 0).float().mean()) > 0.01
        else:
            assert not bool(marks.any())
        if d < 1 << 20:
            check_topk_against_oracle(plan, G, 3, 0, msg, adaptive=False, p=p[0].tolist())


def test_marking_kernels_only_where_something_is_marked():
    """Staging switched off, norms only, and plans too large for marks."""
    g = torch.randn((4, 300_001), device="cuda")
    for p in (None, [0.5, 0.5]):
        plan = P.Plan(P.MLMC_TOPK, 4, 300_001, P.MLMC_F32, [100, 3000, 30_000], p)
        call = lambda: P.mlmc_compress_topk(plan, g, seed=1, step=0)
        names = launched(call)
        assert "k_scan_marks" in names and "k_scan" not in names
        plan.set_staging(False)
        names = launched(call)
        assert "k_scan" in names and "k_scan_marks" not in names
        plan.set_staging(True)
        assert "k_scan_marks" in launched(call)
        names = launched(lambda: P.mlmc_level_norms(plan, g))
        assert "k_scan" in names and "k_scan_marks" not in names
    g = torch.randn((4, 100_000), device="cuda")      # adaptive plans of this size have staging off
    plan = P.Plan(P.MLMC_TOPK, 4, 100_000, P.MLMC_F32, [100, 3000, 30_000], None)
    assert "k_scan_marks" not in launched(lambda: P.mlmc_compress_topk(plan, g, seed=1, step=0))


def test_adaptive_forecasts_hold():
    """Rows of one distribution with few levels: the estimate from the whole row decides as the exact norms do, or within its margin."""
    M, d = 8, 200_003
    G = np.random.default_rng(1).standard_normal((M, d)).astype(np.float32)
    g = to_device(G)
    plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_F32, [50, 500, 5000, 20_000], None)
    for step in range(3):
        plan.ws.fill_(0)
        msg = P.mlmc_compress_topk(plan, g, seed=2, step=step)
        assert plan.status() == 0
        assert all(_covered(_marks(plan), msg, 4, d))


def _row16(what, d):
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(d, generator=gen, device="cuda")
    if what == "zeros":            # two entries in a hundred are not zero
        x[torch.rand(d, generator=gen, device="cuda") > 0.02] = 0.0
    elif what == "one":
        x.fill_(-0.75)
    elif what == "scales":         # stretches of scales of their own
        x *= torch.exp(-6.0 * torch.rand(64, generator=gen, device="cuda")).repeat_interleave(-(-d // 64))[:d]
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("what,base,band,marked", [
    ("normal", 0, 1000, True), ("normal", 1000, 100, True),
    ("normal", 0, 64, True),       # the marks are of 40 % of the eights
    ("normal", 0, 9, True),        # of 60 %: marked, but the rows are read whole
    ("scales", 0, 9, True),
    ("normal", 0, 6, False),       # a band of a sixth
    ("normal", 5, 1000, False),    # a base band of a fifth
    ("zeros", 0, 80, True),        # the band ends among the entries that are not zero
    ("zeros", 16, 32, False),      # in the zeros: whatever the band's width, most entries are equal to its boundary
    ("one", 0, 1000, False),
])
@pytest.mark.parametrize("M,d", [(8, 20_002_500), (2, 80_000_000)])
def test_forecast_marks_by_slices(what, base, band, marked, M, d):
    """Plans of 16-bit rows with a forecast, many slices a row: what is marked, and the message of either way of the second read against that of the same rows
    in 32 bits; levels given, fixed and from the norms."""
    g = _row16(what, d).repeat(M, 1)
    g32 = g.float()
    k0 = d // base if base else 0
    ladder = [k0, k0 + d // band, k0 + d // band + d // 16]
    for how in ("given", "fixed", "adaptive"):
        fixed = [0.5, 0.5] if how == "fixed" else None
        plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, fixed)
        wide = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_F32, ladder, fixed)
        p = _one_hot(M, 2, 1) if how == "given" else None
        plan.ws.fill_(0)
        print(f"forecast {what} {M}x{d} base {base} band {band} {how}", flush=True)
        msg = P.mlmc_compress_topk(plan, g, seed=5, step=1, p=p)
        want = P.mlmc_compress_topk(wide, g32, seed=5, step=1, p=p)
        assert plan.status() == 0 and wide.status() == 0
        n = int(want.row_off[M])
        assert torch.equal(msg.level, want.level) and torch.equal(msg.row_off, want.row_off) and torch.equal(msg.tile_off, want.tile_off)
        assert torch.equal(msg.idx[:n], want.idx[:n]) and torch.equal(msg.val[:n].view(torch.int32), want.val[:n].view(torch.int32))
        if how == "adaptive":
            assert torch.equal(msg.norms.view(torch.int64), want.norms.view(torch.int64))
        if how == "given":
            marks = _marks16(plan)
            if marked:
                assert all(_covered(marks, msg, 8, d // 4096 * 4096))
            else:
                assert not bool(marks.any())
        del plan, wide, msg, want


def _few(plan):
    """Per row, after an s-segmented Top-k call: 1 where the second read has marked the whole drawn segment."""
    return _region(plan, 32 * plan.M, 4 * (plan.num_tiles + 1) * plan.M, 8 * plan.L * plan.M).view(torch.int32).view(plan.M, 8)[:, 4].tolist()


@pytest.mark.parametrize("M,d,s,bf16,marks", [
    (16, 1 << 20, 1048, False, True), (16, 1 << 20, 1 << 15, False, True), (16, 1 << 20, 1048, True, True), (2, 8_400_001, 2100, True, True),
    (16, (1 << 20) - 1, 1048, False, False), (15, 1 << 20, 1048, True, False),       # fewer than 2^24 entries in all
    (16, 1 << 20, 33_826, False, False), (16, 1 << 20, 1 << 19, True, False),        # 31 levels, two
    (8, 16_384, 163, False, False), (1, 300_001, 3000, False, False),
])
def test_stopk_rows_that_are_marked(M, d, s, bf16, marks):
    """The plans with a forecast, and that it holds for nearly every normal row (levels within 2^-12 of the whole of where the drawn word falls)."""
    g = torch.randn((M, d), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda")
    plan = P.Plan(P.MLMC_STOPK, M, d, P.MLMC_BF16 if bf16 else P.MLMC_F32, [s], None)
    g, few = g.to(torch.bfloat16) if bf16 else g, []
    for step in range(3):
        P.mlmc_compress_topk(plan, g, seed=1, step=step)
        assert plan.status() == 0
        few += _few(plan)
    print(f"stopk marks {M}x{d} s={s} bf16={bf16}: {sum(few)} of {len(few)}", flush=True)
    assert sum(few) >= 0.75 * len(few) if marks else few == [0] * len(few)


@pytest.mark.parametrize("what,s,bf16", [
    ("normal", 3001, False), ("normal", 32_769, False), ("normal", 262, True),
    ("heavy", 3001, False),      # one entry in a coarse bin carries most of a row: the forecast misses now and then
    ("loud", 3001, False),       # the top segments lie in a few tiles, which are read whole
    ("few", 3001, False), ("few", 262, True),     # boundaries among equal keys
])
def test_stopk_messages_from_marked_entries(what, s, bf16):
    """Rows with a last block of one entry: the message of marked, partly marked and unmarked segments against the oracle."""
    M, d = 16, (1 << 20) + 1
    rng = np.random.default_rng(s)
    G = rng.standard_normal((3, d)).astype(np.float32)
    if what == "heavy":
        G = (np.tan(np.pi * (rng.random((3, d)) - 0.5)) ** 3).astype(np.float32)
    elif what == "loud":
        G[:, : d // 50] *= 1e4
    elif what == "few":
        G = (np.round(G * 4) / 4).astype(np.float32)
    if bf16:
        G = W.f32_to_bf16_bits(G)
    g = to_device(G).repeat(6, 1)[:M].contiguous()
    plan = P.Plan(P.MLMC_STOPK, M, d, P.MLMC_BF16 if bf16 else P.MLMC_F32, [s], None)
    norms = [O.level_norms_row(G[i], plan.ladder)[0] for i in range(3)]
    few = []
    for step in range(2):
        plan.ws.fill_(0xFF)
        print(f"stopk marked message {what} s={s} bf16={bf16} step={step}", flush=True)
        msg = P.mlmc_compress_topk(plan, g, seed=2, step=step)
        assert plan.status() == 0
        few += _few(plan)
        off, level, got = msg.row_off.cpu().numpy(), msg.level.cpu().numpy(), msg.norms.cpu().numpy()
        for i in range(M):
            assert np.array_equal(got[i].view(np.uint64), np.array(norms[i % 3]).view(np.uint64))
            assert level[i] == O.draw_level(O.adaptive_p(norms[i % 3]), 2, step, i)
        for i in (0, 4, 11, 15):
            want = O.compress_topk_row(G[i % 3], plan.ladder, O.adaptive_p(norms[i % 3]), 2, step, i)
            assert np.array_equal(u32(msg.idx[off[i]:off[i + 1]]), want["idx"])
            assert np.array_equal(u32(msg.val[off[i]:off[i + 1]]), want["val"].view(np.uint32))
            bounds = np.searchsorted(want["idx"], np.arange(plan.num_tiles + 1, dtype=np.int64) * P.MLMC_TILE)
            assert np.array_equal(u32(msg.tile_off[i]), bounds.astype(np.uint32))
    assert any(few)


def test_stopk_rows_with_nan_and_inf_end():
    """Sums that are no numbers: refused by the status word, and ended all the same."""
    g = torch.randn((16, 1 << 20), device="cuda")
    g[0, 5], g[1, 7] = float("nan"), float("inf")
    plan = P.Plan(P.MLMC_STOPK, 16, 1 << 20, P.MLMC_F32, [3001], None)
    P.mlmc_compress_topk(plan, g, seed=1, step=1)
    assert plan.status() & P.MLMC_DEV_NONFINITE
