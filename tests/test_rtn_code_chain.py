"""Round-to-Nearest ladders whose widths divide the widest: the codes of every level follow from the widest level's."""
import numpy as np
import pytest

import paper_2507_05508_amd as P


@pytest.mark.parametrize("B", range(2, 17))
def test_codes_follow_from_the_widest(B):
    """Every quarter of a unit of the widest level (its codes' middles, ties and the points between): rounding the widest code, cut, divided by q gives the
    code that the entry itself has, cut.  In whole numbers, and as the multiply-add in doubles forms it."""
    DB = 2**B - 1
    x4 = np.arange(0, 2 * DB + 1, dtype=np.int64)   # 4 x, x = |g| D / 2c up to D / 2

    def rne(num, den):   # num / den to the nearest integer, ties to even; both non-negative
        n, r = num // den, num % den
        return n + ((2 * r > den) | ((2 * r == den) & (n & 1 == 1)))

    top = np.minimum(rne(x4, 4), 2 ** (B - 1) - 1)
    for b in (w for w in range(1, B) if B % w == 0):
        q = DB // (2**b - 1)
        own = np.minimum(rne(x4, 4 * q), 2 ** (b - 1) - 1)
        assert np.array_equal(rne(top, q), own)
        magic = 1.5 * 2.0**52
        formed = (top * ((2**b - 1) / DB) + magic) - magic
        assert np.array_equal(formed.astype(np.int64), own)


@pytest.mark.gpu
@pytest.mark.parametrize("B", [[1, 2, 4, 8, 16], [0, 3, 6, 12], [0, 1, 5, 15], [2, 14], [7, 14]])
@pytest.mark.parametrize("dtype", [P.MLMC_F32, P.MLMC_BF16])
def test_ladders_whose_widths_divide_the_widest(B, dtype):
    import mlmc_workloads as W
    from gpu_util import to_device
    from oracle import mlmc as O
    from test_gpu_rtn import _check

    rng = np.random.default_rng(sum(B))
    d, c = 3 * 4096 + 77, 2.0**-7
    G = rng.standard_normal((4, d)).astype(np.float32) * 0.01
    G[1] = (rng.integers(-(2**B[-1] - 1), 2**B[-1], d) * (c / (2**B[-1] - 1))).astype(np.float32)   # near the ties
    G[2] = rng.integers(-128, 129, d) * (c / 128)
    G[3] = 0.0
    G[1:3, 5] = c
    if dtype == P.MLMC_BF16:
        raw = W.f32_to_bf16_bits(G)
        g, G = to_device(raw), (raw.astype(np.uint32) << 16).view(np.float32)
    else:
        g = to_device(G)
    plan = P.Plan(P.MLMC_RTN, 4, d, dtype, B, None)
    for step in range(3):
        print(f"rtn chain B={B} dtype={dtype} step={step}", flush=True)
        msg = P.mlmc_compress_rtn(plan, g, seed=4, step=step)
        _check(plan, G, B, None, 4, step, msg)
