"""GPU parity of the plane packing itself: blocks of 2048 elements dealt to lanes of 32, at the edges of lanes, words and
blocks, for rows that start at any element, both input types and every plane count class, bit for bit."""
import numpy as np
import pytest
import torch

import mlmc_workloads as W
import paper_2507_05508_amd as P
from oracle import mlmc as O
from gpu_util import launched, to_device

pytestmark = pytest.mark.gpu

KINDS = {  # kind, ladders (with and without a base field; one, two and three bytes of level planes), oracle
    "bits": (P.MLMC_BITS, [[0, 1, 2, 4, 8, 16], [3, 24], [0, 24]], O.compress_bits, O.aggregate_bits),
    "vbits": (P.MLMC_VBITS, [[0, 1, 2, 4, 8, 16], [3, 24], [0, 24]], O.compress_vbits, O.aggregate_vbits),
    "fbits": (P.MLMC_FBITS, [[0, 1, 2, 3, 5, 8, 23], [9, 16, 23], [2, 7, 15]], O.compress_fbits, O.aggregate_fbits),
    "rtn": (P.MLMC_RTN, [[0, 2, 4, 8, 16], [5, 9, 16], [0, 1]], O.compress_rtn, O.aggregate_rtn),
}


def _one(kind, F, G, g, step, alpha, tag):
    code, _, compress, aggregate = KINDS[kind]
    M, d = G.shape
    G32 = W.bf16_bits_to_f32(G) if G.dtype == np.uint16 else G
    p = O.geometric_p(len(F) - 1)
    plan = P.Plan(code, M, d, P.MLMC_BF16 if G.dtype == np.uint16 else P.MLMC_F32, F, p)
    print(f"planes {kind} F={F} M={M} d={d} {G.dtype} {tag} step={step}", flush=True)
    msg = P.mlmc_compress_rtn(plan, g, 4, step) if kind == "rtn" else P.mlmc_compress_bits(plan, g, 4, step)
    out = P.mlmc_aggregate(plan, msg, alpha)
    torch.cuda.synchronize()
    assert plan.status() == 0
    want = compress(G32, F, p, 4, step)
    planes = msg.planes.cpu().numpy().view(np.uint64)
    for i in range(M):
        n = want[i]["planes"].shape[0]
        assert int(msg.level[i]) == want[i]["level"]
        assert np.array_equal(planes[i, :n], want[i]["planes"]), f"row {i}"
    assert np.array_equal(out.cpu().numpy().view(np.uint32), aggregate(want, F, d, alpha).view(np.uint32))


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("bf16", [False, True])
def test_planes_at_the_edges_of_lanes_words_and_blocks(kind, bf16):
    rng = np.random.default_rng(9)
    for n, d in enumerate([1, 31, 32, 33, 64, 65, 2047, 2048, 2049, 4 * 2048 + 2016, 9 * 2048 + 1]):
        G = (rng.standard_normal((2, d)) * np.exp(rng.uniform(-6, 3, size=(2, d)))).astype(np.float32)
        if bf16:
            G = W.f32_to_bf16_bits(G)
        base = to_device(G, ld=d + 5 + n % 3)
        M = base.shape[0]
        buf = torch.zeros(M * (d + 11) + 8, dtype=base.dtype, device="cuda")
        for off in (0, 1, 3):   # rows that start at any element
            ld = d + 11 if off else d + 5
            g = torch.as_strided(buf, (M, d), (ld, 1), off)
            g.copy_(base)
            for F in KINDS[kind][1]:
                _one(kind, F, G, g, n + off, 0.5, f"offset {off} ld {ld}")


@pytest.mark.parametrize("kind", ["bits", "vbits"])
def test_planes_of_rows_with_non_finite_entries(kind):
    """A row that holds Inf or NaN takes its scale from the largest bit pattern, read as a number: digits by integer arithmetic."""
    d, F = 4096 + 77, [0, 3, 8]
    rng = np.random.default_rng(3)
    G = (rng.standard_normal((2, d)) * np.exp(rng.uniform(-80, 88, size=(2, d)))).astype(np.float32)
    G[0, 5] = np.inf
    G[1, 9] = -np.inf
    G[1, 4000] = np.nan
    p = O.geometric_p(2)
    plan = P.Plan(KINDS[kind][0], 2, d, P.MLMC_F32, F, p)
    for step in range(3):
        print(f"non-finite {kind} step={step}", flush=True)
        msg = P.mlmc_compress_bits(plan, to_device(G), 4, step)
        torch.cuda.synchronize()
        assert plan.status() == P.MLMC_DEV_NONFINITE
        planes = msg.planes.cpu().numpy().view(np.uint64)
        for i in range(2):
            key = (G[i].view(np.uint32) & np.uint32(0x7FFFFFFF)).astype(np.int64)
            E = np.maximum(key >> 23, 1)
            sig = np.where(key >> 23, (key & 0x7FFFFF) | 0x800000, key)
            k = int(np.argmax(key))
            if kind == "bits":
                m = [int(s) >> (24 - 8 + 255 - int(e)) for s, e in zip(sig, E)]
            else:
                m = [min((int(s) << 8) * 2 ** int(e) // (int(sig[k]) * 2 ** int(E[k])), 255) for s, e in zip(sig, E)]
            level = int(msg.level[i])
            field = (np.array(m) >> (8 - F[level])) & ((1 << (F[level] - F[level - 1])) - 1)
            assert np.array_equal(planes[i, 0], O.pack_plane((G[i].view(np.uint32) >> 31).astype(np.uint8)))
            for b in range(F[level] - F[level - 1]):
                assert np.array_equal(planes[i, 1 + b], O.pack_plane(((field >> b) & 1).astype(np.uint8))), (i, b)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("M,d", [(2, 64 * 8192), (2, 65 * 8192 - 2049), (1, 71 * 8192 + 5), (16, 199 * 8192 + 77), (16, 500 * 8192 - 5)])
def test_planes_of_grids_rounded_up_to_the_dies(kind, M, d):
    """Workgroups in multiples of eight, dealt by die: as many as the rows' quadruples of blocks, a few past the last one, one block or several a wave."""
    code, ladders, *_ = KINDS[kind]
    row = {"bits": O.compress_bits_row, "vbits": O.compress_vbits_row, "fbits": O.compress_fbits_row, "rtn": O.compress_rtn_row}[kind]
    F = ladders[0]
    p = O.geometric_p(len(F) - 1)
    g = torch.randn((M, d), generator=torch.Generator(device="cuda").manual_seed(d), device="cuda") * 0.01
    plan = P.Plan(code, M, d, P.MLMC_F32, F, p)
    msg = P.BitsMessage(plan)
    msg.planes.fill_(0x5555)
    print(f"grid {kind} M={M} d={d}", flush=True)
    P.mlmc_compress_rtn(plan, g, 4, 1, out=msg) if kind == "rtn" else P.mlmc_compress_bits(plan, g, 4, 1, out=msg)
    assert plan.status() == 0
    for i in sorted({0, M - 1}):
        want = row(g[i].cpu().numpy(), F, p, 4, 1, i)
        planes = msg.planes[i].cpu().numpy().view(np.uint64)
        n = want["planes"].shape[0]
        assert int(msg.level[i]) == want["level"]
        assert np.array_equal(planes[:n], want["planes"]) and bool((planes[n:] == 0x5555).all())


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("M,d,off", [(6, 262_144, 0), (6, 262_145, 1), (3, 524_288, 1), (3, 524_289 + 2046, 3)])
def test_planes_on_both_sides_of_the_words_limit(kind, bf16, M, d, off):
    """The last sizes that go by words and the first ones that go by blocks of 2048 (extraction: 1572864 entries in all; aggregate: 2^18 or 2^19 a row)."""
    rng = np.random.default_rng(d)
    G = (rng.standard_normal((M, d)) * np.exp(rng.uniform(-6, 3, size=(M, 1)))).astype(np.float32)
    G[:, :: 7] *= np.float32(1e-3)
    G[0, 11] = 0.0
    if bf16:
        G = W.f32_to_bf16_bits(G)
    base = to_device(G)
    g = torch.as_strided(torch.zeros(M * (d + 11) + 8, dtype=base.dtype, device="cuda"), (M, d), (d + 11, 1), off)
    g.copy_(base)
    for n, F in enumerate(KINDS[kind][1][:2]):
        _one(kind, F, G, g, n + off, 0.5, f"offset {off}")


@pytest.mark.parametrize("kind,bf16,M,d,words", [
    ("bits", False, 6, 262_143, True), ("bits", False, 6, 262_145, False),      # ragged last blocks: 1572864 entries in all
    ("bits", False, 8, 196_608, True), ("bits", False, 8, 198_656, False),      # whole blocks: the same for few rows,
    ("bits", False, 16, 65_536, True), ("bits", False, 16, 67_584, False),      # 2^20 for more
    ("bits", False, 32, 2_048, True), ("bits", False, 33, 2_048, False), ("bits", False, 33, 2_049, True),
    ("bits", True, 8, 2_048, True), ("bits", True, 9, 2_048, False), ("bits", True, 9, 2_047, True),
    ("vbits", False, 32, 4_096, True), ("vbits", False, 33, 4_096, False), ("vbits", True, 9, 4_096, False),
    ("fbits", False, 1, 2_048, False), ("fbits", False, 1, 2_047, True), ("fbits", True, 6, 262_144, False),
])
def test_extraction_by_words_or_by_blocks(kind, bf16, M, d, words):
    """The sizes that take either kernel, and the first and the last row's message."""
    row = {"bits": O.compress_bits_row, "vbits": O.compress_vbits_row, "fbits": O.compress_fbits_row}[kind]
    F = KINDS[kind][1][0]
    p = O.geometric_p(len(F) - 1)
    G = np.random.default_rng(d).standard_normal((M, d)).astype(np.float32)
    if bf16:
        G = W.f32_to_bf16_bits(G)
    plan = P.Plan(KINDS[kind][0], M, d, P.MLMC_BF16 if bf16 else P.MLMC_F32, F, p)
    msg, g = P.BitsMessage(plan), to_device(G)
    print(f"extraction {kind} bf16={bf16} M={M} d={d}", flush=True)
    names = launched(lambda: P.mlmc_compress_bits(plan, g, 4, 1, out=msg))
    assert ("k_bits_extract_words" in names, "k_bits_extract" in names) == (words, not words)
    for i in {0, M - 1}:
        want = row(W.bf16_bits_to_f32(G[i]) if bf16 else G[i], F, p, 4, 1, i)
        assert int(msg.level[i]) == want["level"]
        assert np.array_equal(msg.planes[i].cpu().numpy().view(np.uint64)[: want["planes"].shape[0]], want["planes"])


@pytest.mark.parametrize("kind,M,d,words", [
    ("bits", 1, 262_144, True), ("bits", 2, 264_192, False), ("bits", 2, 264_193, True), ("bits", 8, 524_288, True),
    ("vbits", 7, 264_192, False), ("vbits", 8, 264_192, True), ("vbits", 1, 524_289, False),
    ("fbits", 1, 262_144, True), ("fbits", 1, 262_145, False),
    ("rtn", 2, 196_608, True), ("rtn", 2, 198_656, False), ("rtn", 2, 198_657, True), ("rtn", 8, 262_144, True), ("rtn", 8, 262_145, False),
])
def test_aggregate_by_words_or_by_blocks(kind, M, d, words):
    """The sizes that take either kernel, and the update."""
    code, ladders, compress, aggregate = KINDS[kind]
    F = ladders[0]
    p = O.geometric_p(len(F) - 1)
    G = np.random.default_rng(d).standard_normal((M, d)).astype(np.float32)
    plan = P.Plan(code, M, d, P.MLMC_F32, F, p)
    print(f"aggregate {kind} M={M} d={d}", flush=True)
    msg = P.mlmc_compress_rtn(plan, to_device(G), 4, 1) if kind == "rtn" else P.mlmc_compress_bits(plan, to_device(G), 4, 1)
    out = torch.empty(d, dtype=torch.float32, device="cuda")
    names = launched(lambda: P.mlmc_aggregate(plan, msg, 0.5, out=out))
    assert ("k_agg_words" in names, "k_agg_bits" in names) == (words, not words)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), aggregate(compress(G, F, p, 4, 1), F, d, 0.5).view(np.uint32))
