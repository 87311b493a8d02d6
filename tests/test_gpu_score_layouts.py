"""GPU parity of the matrix-core score kernel where its tiles end: every key layout (head dimension), every
number of 32-row query blocks, prompt lengths around the 32-key block and the slices of the key axis, shots of
a few tokens next to long ones.  Scores against the float64 oracle; selection and copies as everywhere."""
import math

import numpy as np
import pytest
import torch

from helpers import check_prefill_problem, oracle_prefill
from oracle import shotkv_oracle as orc

pytestmark = pytest.mark.gpu

# A logit is a sum of head_dim products in float32 (those of bf16 values are exact): at most 2 * head_dim
# roundings of 2^-24 of its terms, and its absolute error is the weight's relative error.  2e-5 covers that for
# the |logit| < 20 drawn here with the exponential's and the log's own few units in the last place.
SCORE_RTOL = 2e-5

LENGTHS = (33, 255, 256, 257, 511, 2049)
ROWS = [(1, 32), (2, 32), (4, 24), (5, 32), (8, 32), (7, 9), (1, 1)]   # (query heads per KV head, window)


@pytest.fixture(scope="module")
def kv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_01941_amd import shotkv
    shotkv.load_library()
    return shotkv


def _offsets(rng, N, n):
    """n shots between a short prefix and the prompt's end: one-token shots first, then whatever is left."""
    few = min(n // 2, N // 4)
    cuts = np.sort(rng.choice(np.arange(4 + few, N + 1), size=n - few, replace=False))
    return np.concatenate([3 + np.arange(few + 1), cuts]).astype(np.int32)


@pytest.mark.parametrize("G,W", ROWS)
@pytest.mark.parametrize("D,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
def test_tile_edges(kv, D, dtype, G, W):
    Hkv, P = 2, 2
    rng = np.random.default_rng(17 * G + W + D)
    scale = 1.0 / math.sqrt(D)
    for N in LENGTHS:
        n = int(rng.integers(1, 12))
        q = torch.from_numpy(rng.standard_normal((P, Hkv * G, W, D), dtype=np.float32) * 2).to(dtype).cuda()
        k = torch.from_numpy(rng.standard_normal((P, Hkv, N, D), dtype=np.float32)).to(dtype).cuda()
        v = torch.from_numpy(rng.standard_normal((P, Hkv, N, D), dtype=np.float32)).to(dtype).cuda()
        offs = np.stack([_offsets(rng, N, n) for _ in range(P)])
        bud = torch.tensor([N, max(1, (2 * N) // 3)], dtype=torch.int32, device="cuda")
        res = kv.prefill_compress(q, k, v, torch.from_numpy(offs).cuda(), bud, N, scale)
        torch.cuda.synchronize()
        for p in range(P):
            budget = int(bud[p].item())
            ref = oracle_prefill(q[p], k[p], v[p], offs[p], budget, scale)
            np.testing.assert_allclose(res.shot_scores[p].cpu().numpy(), ref["scores"], rtol=SCORE_RTOL, atol=0,
                                       err_msg=f"N={N} p={p}")
            check_prefill_problem(res, p, q[p], k[p], v[p], offs[p], budget, N, scale, orc.SELECT_PREFIX, ref=ref)
