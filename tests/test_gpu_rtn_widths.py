"""Round-to-Nearest messages at the code widths where the aggregate changes its way (both codes in one byte, a byte each, two bytes for
the drawn code, two for both, a base code as the previous one) and where the planes fill their last byte or not, bit for bit."""
import numpy as np
import pytest
import torch

import mlmc_workloads as W
import paper_2507_05508_amd as P
from oracle import mlmc as O
from gpu_util import to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("F", [[0, 1, 3, 4, 5, 8, 9], [0, 4, 7, 11, 16], [0, 9, 16], [1, 2, 4, 6, 13], [3, 4, 12], [8, 10], [9, 11], [10, 16]])
def test_rtn_code_widths(F, bf16):
    L = len(F) - 1
    rng = np.random.default_rng(sum(F) + bf16)
    d = 3 * 2048 + 77
    G = (rng.standard_normal((5, d)) * np.exp(rng.uniform(-5, 1, size=(5, d)))).astype(np.float32)
    G[4] = 0.0
    G[3] *= np.float32(2.0 ** -130)
    if bf16:
        bits = W.f32_to_bf16_bits(G)
        G, g = W.bf16_bits_to_f32(bits), to_device(bits)
    else:
        g = to_device(G)
    for level in range(1, L + 1):   # nearly all of the probability on one level
        p = np.full(L, 1e-3 / max(L - 1, 1))
        p[level - 1] = 1.0 - p.sum() + p[level - 1]
        plan = P.Plan(P.MLMC_RTN, 5, d, P.MLMC_BF16 if bf16 else P.MLMC_F32, F, p)
        print(f"widths {F} level {level} bf16 {bf16}", flush=True)
        msg = P.mlmc_compress_rtn(plan, g, 11, level)
        out = P.mlmc_aggregate(plan, msg, 0.25)
        torch.cuda.synchronize()
        assert plan.status() == 0
        want = O.compress_rtn(G, F, p, 11, level)
        planes = msg.planes.cpu().numpy().view(np.uint64)
        for i in range(5):
            assert int(msg.level[i]) == want[i]["level"]
            n = want[i]["planes"].shape[0]
            assert np.array_equal(planes[i, :n], want[i]["planes"]), f"row {i}"
        assert np.array_equal(out.cpu().numpy().view(np.uint32), O.aggregate_rtn(want, F, d, 0.25).view(np.uint32))
