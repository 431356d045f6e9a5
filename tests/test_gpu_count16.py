"""Top-k of 16-bit rows, whose magnitudes are counted: both ways of the message read (slices, tile lists), at the edges of a
step, a slice and a tile, with thresholds whose equal entries are split, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import mlmc_workloads as W
import paper_2507_05508_amd as P
from gpu_util import check_topk_against_oracle, launched, to_device, u32
from oracle import mlmc as O

pytestmark = pytest.mark.gpu


def _rows(what, M, d, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, d)).astype(np.float32)
    if what == "few":
        x = (np.round(x * 4) / 4).astype(np.float32)
    if what == "one":
        x = np.full((M, d), -0.75, np.float32)
    if what == "zeros":
        x[:, rng.random(d) < 0.9] = 0.0
        x[M - 1] = 0.0
    if what == "loud":      # one stretch holds nearly every large entry
        x[:, : max(1, d // 9)] *= 1000.0
    if what == "tiny":      # subnormal entries, and one Inf
        x = (x * 1e-39).astype(np.float32)
        x[0, d // 2] = np.inf
    return W.f32_to_bf16_bits(x)


@pytest.mark.parametrize("what", ["normal", "few", "one", "zeros", "loud", "tiny"])
@pytest.mark.parametrize("M,d,pad", [(1, 1, 0), (2, 16384, 0), (3, 16385, 3), (1, 3 * 16384 - 1, 0), (5, 70_001, 1), (2, 300_000, 8)])
def test_message_by_slices(what, M, d, pad):
    G = _rows(what, M, d, 31 * d + M)
    g = to_device(G, ld=d + pad)
    for ladder in ([[0, 1]] if d == 1 else [[0, d // 7 + 1, d // 3 + 2, d], [d // 50, d // 50 + 1, d // 2 + 1, d - 1]]):
        L = len(ladder) - 1
        for p in (None, O.geometric_p(L)):
            plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, p)
            plan.ws.fill_(0xFF)      # nothing is expected in it
            for step in range(2 * L):
                print(f"slices {what} {M}x{d}+{pad} {ladder} adaptive={p is None} step={step}", flush=True)
                msg = P.mlmc_compress_topk(plan, g, seed=9, step=step)
                check_topk_against_oracle(plan, G, 9, step, msg, adaptive=p is None)
                assert plan.status() == (P.MLMC_DEV_NONFINITE if what == "tiny" else 0)
            if p is None:
                norms = P.mlmc_level_norms(plan, g).cpu().numpy()
                for i in range(M):
                    assert np.array_equal(norms[i].view(np.uint64), np.array(O.level_norms_row(G[i], ladder)[0]).view(np.uint64))


@pytest.mark.parametrize("d", [1 << 18, (1 << 18) + 5, (1 << 18) + 4096 * 3 + 1030])
def test_message_by_tile_lists(d):
    """256 rows, a slice each, long enough for the tile lists; a few rows of every kind are compared."""
    M, kinds = 256, ["normal", "few", "one", "zeros", "loud", "tiny"]
    few = np.concatenate([_rows(k, 1, d, 7 + i) for i, k in enumerate(kinds)])
    g = to_device(few).repeat(-(-M // len(kinds)), 1)[:M].contiguous()
    picks = list(range(6)) + list(range(M - 7, M))
    for ladder in ([0, 5000, d // 3 + 2, d], [d // 50, d // 50 + 1, d // 2 + 1, d - 1]):
        plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, None)
        plan.ws.fill_(0xFF)
        for step in range(3):
            print(f"tile lists d={d} {ladder} step={step}", flush=True)
            msg = P.mlmc_compress_topk(plan, g, seed=2, step=step)
            torch.cuda.synchronize()
            assert plan.status() == P.MLMC_DEV_NONFINITE
            off = msg.row_off.cpu().numpy()
            level = msg.level.cpu().numpy()
            assert np.array_equal(np.diff(off), [ladder[0] + ladder[l] - ladder[l - 1] for l in level])
            for i in picks:
                want = O.compress_topk_row(few[i % len(kinds)], ladder, None, 2, step, i)
                assert level[i] == want["level"]
                assert np.array_equal(msg.norms[i].cpu().numpy().view(np.uint64), np.array(want["norms"]).view(np.uint64))
                assert np.array_equal(u32(msg.idx[off[i]:off[i + 1]]), want["idx"]), (i, step)
                assert np.array_equal(u32(msg.val[off[i]:off[i + 1]]), want["val"].view(np.uint32)), (i, step)
                bounds = np.searchsorted(want["idx"], np.arange(plan.num_tiles + 1, dtype=np.int64) * P.MLMC_TILE)
                assert np.array_equal(u32(msg.tile_off[i]), bounds.astype(np.uint32))


def _check_rows(plan, msg, rows, picks, ladder, seed, step):
    """Rows `picks` of the message against the oracle; `rows`: the kinds that take turns."""
    torch.cuda.synchronize()
    off, level = msg.row_off.cpu().numpy(), msg.level.cpu().numpy()
    assert np.array_equal(np.diff(off), [ladder[0] + ladder[l] - ladder[l - 1] for l in level])
    for i in picks:
        want = O.compress_topk_row(rows[i % len(rows)], ladder, None, seed, step, i)
        assert level[i] == want["level"]
        assert np.array_equal(msg.norms[i].cpu().numpy().view(np.uint64), np.array(want["norms"]).view(np.uint64))
        assert np.array_equal(u32(msg.idx[off[i]:off[i + 1]]), want["idx"]), (i, step)
        assert np.array_equal(u32(msg.val[off[i]:off[i + 1]]), want["val"].view(np.uint32)), (i, step)
        bounds = np.searchsorted(want["idx"], np.arange(plan.num_tiles + 1, dtype=np.int64) * P.MLMC_TILE)
        assert np.array_equal(u32(msg.tile_off[i]), bounds.astype(np.uint32))


@pytest.mark.parametrize("what", ["normal", "few", "one"])
@pytest.mark.parametrize("M,d", [(1, 64 * 16384 + 1), (2, 128 * 16384 - 9), (1, 256 * 16384 - 9)])
def test_more_than_64_slices(what, M, d):
    """One or two rows in 65, 128 and 256 slices: the counts of eight groups of up to 32 slices are added up, with and without the counts
    before every slice (a message, norms alone)."""
    G = _rows(what, M, d, d + M)
    g = to_device(G)
    ladder = [d // 50, d // 3 + 2, d // 2 + 1, d - 1]
    plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, None)
    plan.ws.fill_(0xFF)
    norms = P.mlmc_level_norms(plan, g).cpu().numpy()
    assert plan.status() == 0
    for i in range(M):
        assert np.array_equal(norms[i].view(np.uint64), np.array(O.level_norms_row(G[i], ladder)[0]).view(np.uint64))
    plan.ws.fill_(0xFF)
    for step in range(3):
        print(f"many slices {what} {M}x{d} step={step}", flush=True)
        msg = P.mlmc_compress_topk(plan, g, seed=4, step=step)
        assert plan.status() == 0
        _check_rows(plan, msg, G, range(M), ladder, 4, step)


@pytest.mark.parametrize("d", [4 * 16384 * 3, 4 * 16384 * 4 + 1030, 290_011])
def test_slices_of_several_steps(d):
    """64 rows in four slices each, of three to five steps, the last step whole, short, or ending inside a block: thresholds whose equals run out in the
    first, a middle or the last step, several thresholds on one key, and all of a step's entries in the message."""
    M, kinds = 64, ["normal", "few", "one", "zeros", "loud", "tiny"]
    few = np.concatenate([_rows(k, 1, d, 11 + i) for i, k in enumerate(kinds)])
    g = to_device(few).repeat(-(-M // len(kinds)), 1)[:M].contiguous()
    for ladder in ([0, d // 7, d // 3 + 2, d], [d // 50, d // 50 + 1, d // 2 + 1, d - 1], [3, d // 4 + 16384, d // 4 + 20000, d // 2 - 77]):
        plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, None)
        plan.ws.fill_(0xFF)
        assert "k_c16_mark" not in launched(lambda: P.mlmc_compress_topk(plan, g, seed=6, step=0))
        for step in range(3):
            print(f"several steps d={d} {ladder} step={step}", flush=True)
            msg = P.mlmc_compress_topk(plan, g, seed=6, step=step)
            assert plan.status() == P.MLMC_DEV_NONFINITE
            _check_rows(plan, msg, few, list(range(12)) + [M - 1], ladder, 6, step)


def test_ties_in_more_tiles_than_a_workgroup_takes():
    """Rows of 1065 tiles, whose places two workgroups find: a threshold splits entries equal to it in the first one's tiles and in the second one's."""
    M, d = 16, 16 * (1 << 18) + 40 * 4096 + 77
    kinds = ["one", "few", "zeros"]
    few = np.concatenate([_rows(k, 1, d, 3 + i) for i, k in enumerate(kinds[:2])] + [_rows("zeros", 2, d, 5)[:1]])
    g = to_device(few).repeat(6, 1)[:M].contiguous()
    for ladder in ([d // 50, d // 2, d - 50_000, d], [1, d - 100_001, d - 3]):
        plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, None)
        plan.ws.fill_(0xFF)
        assert "k_c16_mark" in launched(lambda: P.mlmc_compress_topk(plan, g, seed=8, step=0))
        for step in range(2):
            print(f"ties over workgroups {ladder} step={step}", flush=True)
            msg = P.mlmc_compress_topk(plan, g, seed=8, step=step)
            assert plan.status() == 0
            _check_rows(plan, msg, few, [0, 1, 2, M - 1], ladder, 8, step)


@pytest.mark.parametrize("M,d", [(3, 50_003), (256, 1 << 18)])
def test_entries_past_the_capacity_are_not_written(M, d):
    G = _rows("normal", 1, d, 5)
    g = to_device(G).repeat(M, 1).contiguous()
    ladder = [100, d // 2, d]
    plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, None)
    whole = P.mlmc_compress_topk(plan, g, seed=1, step=0)
    cap = int(whole.row_off[1]) + 1001
    cut = P.SparseMessage(plan, capacity=plan.sparse_capacity_worst, with_norms=True)
    cut.idx.fill_(-7)
    cut.capacity = cap
    P.mlmc_compress_topk(plan, g, seed=1, step=0, out=cut)
    assert plan.status() == P.MLMC_DEV_CAPACITY
    assert torch.equal(cut.idx[:cap], whole.idx[:cap]) and torch.equal(cut.val[:cap], whole.val[:cap])
    assert bool((cut.idx[cap:] == -7).all())


@pytest.mark.parametrize("how", ["adaptive", "fixed", "given"])
@pytest.mark.parametrize("M,d", [(616, (1 << 18) + 4096 * 2 + 2500), (640, 1 << 18)])
def test_forecast_marks_of_narrow_bands(M, d, how):
    """Messages of a sixteenth of a row or less, whose entries the first read marks: rows whose sampled blocks (one of 1024 entries in 32) tell the band,
    rows with all their large entries outside of these blocks or nearly all zero, split thresholds, bands in a few tiles; every way the level is drawn."""
    kinds = ["normal", "few", "loud", "zeros", "normal", "tiny"]
    few = np.concatenate([_rows(k, 1, d, 23 + i) for i, k in enumerate(kinds)])
    block = np.arange(d) >> 10
    few[4, (block % 32) == 16] = 0          # the sample has nothing of the row
    few[5, 77_777] = W.f32_to_bf16_bits(np.array([3e38], np.float32))[0]   # one entry is all of the first band's norm
    g = to_device(few).repeat(-(-M // len(kinds)), 1)[:M].contiguous()
    picks = list(range(6)) + [M - 1]
    for ladder in ([d >> 12, d >> 11, d >> 9, d >> 7, d >> 5], [0, 3, d // 100, d // 40]):
        L = len(ladder) - 1
        p = O.geometric_p(L) if how == "fixed" else None
        plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_BF16, ladder, p)
        plan.ws.fill_(0xFF)
        norms = P.mlmc_level_norms(plan, g) if how == "given" else None
        for step in range(2):
            print(f"marks {how} {M}x{d} {ladder} step={step}", flush=True)
            msg = P.mlmc_compress_topk(plan, g, seed=5, step=step, p=norms, p_is_norms=norms is not None)
            torch.cuda.synchronize()
            assert plan.status() == P.MLMC_DEV_NONFINITE
            off, level = msg.row_off.cpu().numpy(), msg.level.cpu().numpy()
            assert np.array_equal(np.diff(off), [ladder[0] + ladder[l] - ladder[l - 1] for l in level])
            for i in picks:
                want = O.compress_topk_row(few[i % len(kinds)], ladder, p, 5, step, i)
                assert level[i] == want["level"]
                assert np.array_equal(u32(msg.idx[off[i]:off[i + 1]]), want["idx"]), (i, step)
                assert np.array_equal(u32(msg.val[off[i]:off[i + 1]]), want["val"].view(np.uint32)), (i, step)
                bounds = np.searchsorted(want["idx"], np.arange(plan.num_tiles + 1, dtype=np.int64) * P.MLMC_TILE)
                assert np.array_equal(u32(msg.tile_off[i]), bounds.astype(np.uint32))
