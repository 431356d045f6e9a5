"""Top-k of short 32-bit rows, a workgroup per row: the lengths at which its pieces, stretches and waves change, rows whose
equal entries a threshold splits, candidate lists that do and do not fit, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import paper_2507_05508_amd as P
from gpu_util import check_topk_against_oracle, launched, to_device
from oracle import mlmc as O

pytestmark = pytest.mark.gpu


def _rows(what, M, d, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((M, d)).astype(np.float32)
    if what == "few":
        x = (np.round(x * 4) / 4).astype(np.float32)
    if what == "one":
        x = np.full((M, d), -0.75, np.float32)
    if what == "near":      # one first digit, many second and third ones
        x = (1.0 + x * 1e-4).astype(np.float32)
    if what == "zeros":
        x[:, rng.random(d) < 0.9] = 0.0
        x[M - 1] = 0.0
    if what == "third":     # a good part zeros, the rest dense
        x[:, rng.random(d) < 0.3] = 0.0
    if what == "wide":      # every exponent, subnormals, and one Inf
        x = np.ldexp(x, rng.integers(-149, 120, size=(M, d))).astype(np.float32)
        x[0, d // 2] = np.inf
    return x


@pytest.mark.parametrize("what", ["normal", "few", "one", "near", "zeros", "third", "wide"])
@pytest.mark.parametrize("M,d,pad", [(3, 8192, 0), (2, 8193, 1), (1, 16384 + 255, 0), (2, 3 * 16384 + 257, 3), (1, 65535, 0), (2, 65536, 4)])
def test_short_rows(what, M, d, pad):
    G = _rows(what, M, d, 17 * d + M)
    g = to_device(G, ld=d + pad)
    for ladder in ([0, d // 7 + 1, d // 3 + 2, d], [d // 50, d // 50 + 1, d // 40, d // 2 + 1, d - 1]):
        L = len(ladder) - 1
        for p in (None, O.geometric_p(L)):
            plan = P.Plan(P.MLMC_TOPK, M, d, P.MLMC_F32, ladder, p)
            plan.ws.fill_(0xFF)      # nothing is expected in it
            assert "k_row_select" in launched(lambda: P.mlmc_compress_topk(plan, g, seed=9, step=0))
            for step in range(2 * L):
                print(f"short rows {what} {M}x{d}+{pad} {ladder} adaptive={p is None} step={step}", flush=True)
                msg = P.mlmc_compress_topk(plan, g, seed=9, step=step)
                check_topk_against_oracle(plan, G, 9, step, msg, adaptive=p is None)
                assert plan.status() == (P.MLMC_DEV_NONFINITE if what == "wide" else 0)
            if p is None:
                norms = P.mlmc_level_norms(plan, g).cpu().numpy()
                assert plan.status() == (P.MLMC_DEV_NONFINITE if what == "wide" else 0)
                for i in range(M):
                    assert np.array_equal(norms[i].view(np.uint64), np.array(O.level_norms_row(G[i], ladder)[0]).view(np.uint64))


def test_thresholds_in_one_bucket():
    """All 33 thresholds between entries of one first digit, so that the candidates do not fit the list."""
    d, L = 40_000, 32
    G = _rows("near", 2, d, 3)
    ladder = [7 + 1200 * l for l in range(L + 1)]
    plan = P.Plan(P.MLMC_TOPK, 2, d, P.MLMC_F32, ladder, None)
    for step in range(4):
        msg = P.mlmc_compress_topk(plan, to_device(G), seed=1, step=step)
        check_topk_against_oracle(plan, G, 1, step, msg, adaptive=True)
        assert plan.status() == 0


@pytest.mark.parametrize("what", ["normal", "near", "few", "third", "wide"])
@pytest.mark.parametrize("L", [1, 2, 4, 8, 16, 32])
def test_copies_of_the_counts(what, L):
    """From one to 33 thresholds, each in a bucket of its own where the values allow it: how many copies of the counts there are
    depends on that, and with 33 there is no room for a list at all."""
    d = 65_536 - 3
    G = _rows(what, 2, d, L)
    ladder = [0 if L == 1 else d // 1000] + [(d * l) // L for l in range(1, L + 1)]
    g = to_device(G)
    for p in (None, O.geometric_p(L)):
        plan = P.Plan(P.MLMC_TOPK, 2, d, P.MLMC_F32, ladder, p)
        for step in range(3):
            print(f"copies {what} L={L} adaptive={p is None} step={step}", flush=True)
            msg = P.mlmc_compress_topk(plan, g, seed=3, step=step)
            check_topk_against_oracle(plan, G, 3, step, msg, adaptive=p is None)
            assert plan.status() == (P.MLMC_DEV_NONFINITE if what == "wide" else 0)


def test_capacity_of_short_rows():
    d = 20_001
    G = _rows("normal", 3, d, 5)
    plan = P.Plan(P.MLMC_TOPK, 3, d, P.MLMC_F32, [100, d // 2, d], None)
    g = to_device(G)
    whole = P.mlmc_compress_topk(plan, g, seed=1, step=0)
    cap = int(whole.row_off[1]) + 1001
    cut = P.SparseMessage(plan, capacity=plan.sparse_capacity_worst, with_norms=True)
    cut.idx.fill_(-7)
    cut.capacity = cap
    P.mlmc_compress_topk(plan, g, seed=1, step=0, out=cut)
    assert plan.status() == P.MLMC_DEV_CAPACITY
    assert torch.equal(cut.idx[:cap], whole.idx[:cap]) and torch.equal(cut.val[:cap], whole.val[:cap])
    assert bool((cut.idx[cap:] == -7).all())
