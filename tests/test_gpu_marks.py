"""Which rows have the entries of their message marked by an earlier read, and that the marks hold the whole message where a forecast has to hold:
the messages of the other tests are the same with and without them."""
import numpy as np
import pytest
import torch

import paper_2507_05508_amd as P
from gpu_util import check_topk_against_oracle, launched, to_device

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
