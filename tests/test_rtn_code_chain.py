"""Round-to-Nearest ladders whose widths divide the widest: the codes of every level follow from the widest level's."""
import numpy as np
import pytest

import paper_2507_05508_amd as P


@pytest.mark.parametrize("B", range(2, 17))
def test_codes_follow_from_the_widest(B):
    """Every quarter of a unit of the widest level (its codes' middles, ties and the points between): rounding the widest code, cut, divided by q gives the
    code that the entry itself has, cut.  In whole numbers, and as a fused multiply-add in doubles forms it from the rounded reciprocal.  (The kernel's own codes are
    compared in the test below.)"""
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
        # fma(n, fl(D_b / D_B), 1.5 2^52) rounds the exact product once, to a whole number (the addend's unit is one and it is even)
        num, den = ((2**b - 1) / DB).as_integer_ratio()
        assert np.array_equal(rne(top.astype(object) * num, den).astype(np.int64), own)


@pytest.mark.gpu
@pytest.mark.parametrize("B", [[1, 2, 4, 8, 16], [0, 3, 6, 12], [0, 1, 5, 15], [2, 14], [7, 14]])
@pytest.mark.parametrize("dtype", [P.MLMC_F32, P.MLMC_BF16])
def test_ladders_whose_widths_divide_the_widest(B, dtype):
    import mlmc_workloads as W
    from gpu_util import to_device
    from oracle import mlmc as O
    from test_gpu_rtn import _check

    rng = np.random.default_rng(sum(B))
    d, c, D = 3 * 4096 + 77, 2.0**-7, 2**B[-1] - 1
    G = rng.standard_normal((4, d)).astype(np.float32) * 0.01
    G[1] = (rng.integers(-D, D + 1, d) * (c / D)).astype(np.float32)   # where ties would be; none is one, since c is a power of two and D odd
    G[2] = rng.integers(-128, 129, d) * (c / 128)
    G[3] = 0.0
    G[1:3, 5] = c
    # Ties: |g| D / 2c is a half-integer where |g| is an odd multiple of c / D.  So rows of whole units with c = D units (more bits than a 16-bit entry has) and with
    # c = a units, a dividing D, of up to 8 bits.
    scales = ([D] if dtype == P.MLMC_F32 else []) + [a for a in range(3, 256) if D % a == 0]
    ties = {b: 0 for b in B if b}
    for a in scales:
        k = rng.integers(-a, a + 1, d)
        for b in ties:   # some on multiples of the least number of units that is a whole or half code of this width
            step = a // np.gcd(a, 2**b - 1)
            at = rng.random(d) < 0.2
            k[at] = k[at] // step * step
        k[5] = a
        G = np.vstack([G, (k * 2.0**-20).astype(np.float32)])
        for b in ties:
            whole = np.abs(k) * (2**b - 1) % a == 0
            ties[b] += int(np.sum(whole & (np.abs(k) * (2**b - 1) // a % 2 == 1) & (np.abs(k) < a)))
    assert all(n > 0 for b, n in ties.items() if b > 1), ties   # width 1 has none below c: its codes are all zero
    if dtype == P.MLMC_BF16:
        raw = W.f32_to_bf16_bits(G)
        assert np.array_equal((raw[4:].astype(np.uint32) << 16).view(np.float32), G[4:])
        g, G = to_device(raw), (raw.astype(np.uint32) << 16).view(np.float32)
    else:
        g = to_device(G)
    plan = P.Plan(P.MLMC_RTN, len(G), d, dtype, B, None)
    for step in range(3):
        print(f"rtn chain B={B} dtype={dtype} step={step} ties={ties}", flush=True)
        msg = P.mlmc_compress_rtn(plan, g, seed=4, step=step)
        _check(plan, G, B, None, 4, step, msg)
