"""GPU parity of the matrix-core score kernel where its tiles end: every key layout (head dimension), every
number of 32-row query blocks, prompt lengths around the 32-key block and the slices of the key axis, shots of
a few tokens next to long ones.  Scores against the float64 oracle; selection and copies as everywhere."""
import math

import numpy as np
import pytest
import torch

from helpers import check_prefill_problem, oracle_prefill, to_np
from oracle import shotkv_oracle as orc

pytestmark = pytest.mark.gpu

# A logit is a sum of head_dim products in float32 (those of bf16 values are exact): at most 2 * head_dim
# roundings of 2^-24 of its terms (what the split of float32 elements drops is below one more per element), and its
# absolute error is the weight's relative error.  2e-5 covers that for
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


@pytest.mark.parametrize("attention", [False, True])
def test_offsets_out_of_order_stay_harmless(kv, attention):
    """Problems whose offsets are unsorted or out of range, between healthy ones: status BAD_OFFSETS, nothing kept,
    zero scores, and the healthy problems' results are those of a batch without them."""
    Hkv, G, W, D, N, n = 2, 4, 32, 128, 900, 6
    H, scale = Hkv * G, 1.0 / math.sqrt(128)
    good = np.array([10, 150, 290, 300, 555, 556, 850], dtype=np.int32)
    bad = [[10, 290, 150, 300, 555, 556, 850], [-5, 150, 290, 300, 555, 556, 850], [10, 150, 290, 300, 555, 556, 2**31 - 1],
           [899, 800, 700, 500, 300, 100, 5], [10, 10, 10, 10, 10, 10, 10], [-2**31, 2**31 - 1, 0, -1, 901, 450, 900]]
    offs = np.stack([good] + [np.array(b, dtype=np.int64).astype(np.int32) for b in bad] + [good])
    P = len(offs)
    rng = np.random.default_rng(5)
    q = torch.from_numpy(rng.standard_normal((P, H, N, D), dtype=np.float32)).to(torch.bfloat16).cuda()
    k = torch.from_numpy(rng.standard_normal((P, Hkv, N, D), dtype=np.float32)).to(torch.bfloat16).cuda()
    v = torch.from_numpy(rng.standard_normal((P, Hkv, N, D), dtype=np.float32)).to(torch.bfloat16).cuda()
    bud = torch.full((P,), 500, dtype=torch.int32, device="cuda")

    def call(rows):
        a = [t[rows].contiguous() for t in (q, k, v)]
        o, b = torch.from_numpy(offs).cuda()[rows].contiguous(), bud[rows].contiguous()
        if attention:
            return kv.prefill_attention_compress(*a, o, b, 600, W, scale)[1]
        return kv.prefill_compress(a[0][:, :, -W:].contiguous(), a[1], a[2], o, b, 600, scale)

    res, ref = call(list(range(P))), call([0, P - 1])
    scores, status = kv.prefill_scores(q[:, :, -W:].contiguous(), k, torch.from_numpy(offs).cuda(), scale)
    torch.cuda.synchronize()
    want = [0] + [kv.ST_BAD_OFFSETS] * len(bad) + [0]
    assert res.status.cpu().tolist() == want and status.cpu().tolist() == want
    for p in range(1, P - 1):
        assert int(res.kept_count[p]) == 0 and not res.shot_selected[p].any()
        assert not res.shot_scores[p].any() and not scores[p].any()
    for i, p in enumerate((0, P - 1)):
        assert torch.equal(res.shot_scores[p], ref.shot_scores[i]) and torch.equal(res.shot_selected[p], ref.shot_selected[i])
        kept = int(ref.kept_count[i])
        assert int(res.kept_count[p]) == kept and torch.equal(res.k_out[p, :, :kept], ref.k_out[i, :, :kept])


def _scores_and_oracle(kv, q, k, off, scale):
    q, k = (torch.from_numpy(x.astype(np.float32)).cuda() for x in (q, k))
    scores, status = kv.prefill_scores(q, k, torch.from_numpy(off[None]).cuda(), scale)
    torch.cuda.synchronize()
    assert status.cpu().tolist() == [0]
    with np.errstate(invalid="ignore"):
        ref = oracle_prefill(q[0], k[0], k[0], off, k.shape[2], scale)
    return scores[0].cpu().numpy(), ref["scores"]


@pytest.mark.parametrize("D", [64, 128])
def test_float32_products_are_rounded_not_truncated(kv, D):
    """Mantissas whose low parts are as large and of one sign as they get, 1 + 2^-7 - 2^-23 on both sides, in a product
    of 65 that an exact -65 takes away again.  A float32 multiply-add rounds such a term by 65 * 2^-24; the logit is a
    handful of roundings, here at most four, and its error is the weight's relative error.  A truncated low part would
    be worth 65 * 2^-21, eight times the unit."""
    N, W, x = 600, 8, 8 * (1 + 2.0**-7 - 2.0**-23)
    q, k = np.zeros((1, 2, W, D)), np.zeros((1, 2, N, D))
    q[..., 0], q[..., 33] = x, 65.0
    k[:, :, 100:110, 0], k[:, :, 100:110, 33] = x, -1.0
    off = np.array([0, 100, 110, N], dtype=np.int32)
    got, want = _scores_and_oracle(kv, q, k, off, 1.0)
    np.testing.assert_allclose(got, want, rtol=4 * 65 * 2.0**-24, atol=0)


@pytest.mark.parametrize("G,W", [(1, 8), (2, 32), (4, 32), (8, 32)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("case", ["minus_infinity", "largest_keys", "huge_queries"])
def test_float32_values_over_the_whole_range(kv, D, G, W, case):
    """Keys at minus infinity get no weight; keys near the largest float32 and queries far from one, whose product is
    an ordinary number, count like any others."""
    N, Hkv = 700, 2
    rng = np.random.default_rng(G + D)
    q = rng.standard_normal((1, Hkv * G, W, D), dtype=np.float32)
    k = rng.standard_normal((1, Hkv, N, D), dtype=np.float32)
    if case == "minus_infinity":
        q[..., 5] = np.abs(q[..., 5]) + 0.1
        k[:, :, 97:130, 5] = -np.inf
        k[:, :, 400, 5] = -np.inf
    elif case == "largest_keys":
        q[..., 5] = 2.0**-126 * (1 + rng.random(q.shape[:3], dtype=np.float32))
        k[..., 5] = 3.4e38 * rng.choice([-1, 1], size=k.shape[:3])
    else:
        q[..., 5] = 2.0**120 * rng.standard_normal(q.shape[:3], dtype=np.float32)
        k[..., 5] = 2.0**-120 * rng.standard_normal(k.shape[:3], dtype=np.float32)
    off = np.array([0, 50, 97, 130, 131, 400, 401, 690], dtype=np.int32)
    got, want = _scores_and_oracle(kv, q, k, off, 1.0 / math.sqrt(D))
    np.testing.assert_allclose(got, want, rtol=SCORE_RTOL, atol=0)


@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("D", [64, 128])
def test_float32_forms_side_by_side(kv, D, G):
    """One query head that bf16 parts cannot hold: its wave takes the fp32 form while the others of the workgroup read the
    block's parts that all of them have made."""
    N, Hkv, W = 700, 2, 32
    rng = np.random.default_rng(G + D)
    q = rng.standard_normal((1, Hkv * G, W, D), dtype=np.float32)
    k = rng.standard_normal((1, Hkv, N, D), dtype=np.float32)
    q[:, 1, :, 5] = 2.0**120 * rng.standard_normal((1, W), dtype=np.float32)
    k[..., 5] = 2.0**-120 * rng.standard_normal(k.shape[:3], dtype=np.float32)
    off = np.array([0, 50, 97, 130, 131, 400, 401, 690], dtype=np.int32)
    got, want = _scores_and_oracle(kv, q, k, off, 1.0 / math.sqrt(D))
    np.testing.assert_allclose(got, want, rtol=SCORE_RTOL, atol=0)


def test_float32_launches_that_share_their_parts_and_not(kv):
    """Four waves at head_dim 128 split blocks between them, except in launches of 513 to 767 workgroups with a whole slice
    of 256 keys: 32, 33, 47 and 48 problems of two such slices and 8 KV heads.  Same bits either way; one head of every
    third problem has queries that bf16 parts cannot hold."""
    P, Hkv, G, W, N, D = 48, 8, 4, 32, 600, 128
    assert 48 << 10 <= 32 * Hkv * N and P * Hkv * N < 256 << 10     # slices of 256 keys
    gen = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn((P, Hkv * G, W, D), generator=gen, device="cuda")
    k = torch.randn((P, Hkv, N, D), generator=gen, device="cuda")
    q[::3, 1, :, 5] *= 2.0**120
    k[::3, :, :, 5] *= 2.0**-120
    off = torch.tensor([0, 50, 97, 130, 131, 400, 401, 590], dtype=torch.int32, device="cuda").expand(P, 8).contiguous()
    scale = 1.0 / math.sqrt(D)
    got = {n: kv.prefill_scores(q[:n], k[:n], off[:n], scale)[0] for n in (32, 33, 47, 48)}
    torch.cuda.synchronize()
    for n in (32, 33, 47):
        assert torch.equal(got[n], got[48][:n])
    for p in (0, 31, 46):
        ref = oracle_prefill(q[p], k[p], k[p], off[p].cpu().numpy(), N, scale)
        np.testing.assert_allclose(got[47][p].cpu().numpy(), ref["scores"], rtol=SCORE_RTOL, atol=0)


def test_a_unit_of_many_slices(kv):
    """One unit over 128 slices of the key axis and 8 KV heads: its first key takes nearly all of the mass, 8, and the
    other thousand (slice, head) parts 2.2e-7 each, just under half a unit in the last place below 8, 2.8e-5 of it
    together.  Added one after the other in float32 they would all be lost; in 64 sums side by side each addition is off
    by at most half a unit below 1, 16 of them by 5e-7."""
    H, W, D, N = 8, 1, 64, 32768
    q, k = np.zeros((1, H, W, D)), np.zeros((1, H, N, D))
    q[..., 0] = 1.0
    k[:, :, 0, 0] = 30.125
    off = np.array([0, N - 8], dtype=np.int32)
    got, want = _scores_and_oracle(kv, q, k, off, math.log(2.0))
    np.testing.assert_allclose(got, want, rtol=1e-5, atol=0)


def _check_scores(kv, rng, P, G, Hkv, W, D, dtype, N, offs, problems):
    """prefill_scores of P random problems against the oracle on some of them."""
    scale = 1.0 / math.sqrt(D)
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
    q = 2 * torch.randn((P, Hkv * G, W, D), generator=gen, device="cuda")
    k = torch.randn((P, Hkv, N, D), generator=gen, device="cuda")
    q, k = q.to(dtype), k.to(dtype)
    scores, status = kv.prefill_scores(q, k, torch.from_numpy(offs).cuda(), scale)
    torch.cuda.synchronize()
    assert not status.any()
    for p in problems:
        mass = orc.token_mass(orc.window_attention(to_np(q[p]), to_np(k[p]), scale))
        np.testing.assert_allclose(scores[p].cpu().numpy(), orc.shot_scores_from_mass(mass, offs[p]), rtol=SCORE_RTOL, atol=0,
                                   err_msg=f"p={p}")


def test_head_dim_64_in_two_waves(kv):
    """128 query rows of head_dim 64 take two waves per workgroup from 1.5 M keys in a launch on, with 1024-key slices."""
    P, Hkv, N, n = 12, 8, 16411, 70
    rng = np.random.default_rng(3)
    assert P * Hkv * N >= 3 << 19
    offs = np.stack([_offsets(rng, N, n) for _ in range(P)])
    _check_scores(kv, rng, P, 4, Hkv, 32, 64, torch.bfloat16, N, offs, (0, P - 1))


def _tiny_units(rng, P, N, n):
    """n units of one or two tokens between a prefix of three tokens and the tail"""
    lengths = rng.integers(1, 3, size=(P, n))
    offs = 3 + np.concatenate([np.zeros((P, 1), dtype=np.int64), np.cumsum(lengths, axis=1)], axis=1)
    assert offs.max() <= N
    return offs.astype(np.int32)


@pytest.mark.parametrize("G,D,dtype", [(4, 128, torch.bfloat16), (6, 128, torch.bfloat16), (8, 64, torch.bfloat16),
                                       (1, 64, torch.bfloat16), (4, 128, torch.float32), (8, 64, torch.float32)])
def test_more_ends_in_a_slice_than_are_kept(kv, G, D, dtype):
    """256-key slices (51200 keys in the launch) with units of one or two tokens: about 170 ends in a slice, more than
    the 128 that are kept in LDS, so the ends come from memory while blocks are in flight."""
    P, Hkv, N, n = 1, 8, 6400, 4096
    rng = np.random.default_rng(G + D)
    _check_scores(kv, rng, P, G, Hkv, 32, D, dtype, N, _tiny_units(rng, P, N, n), (0,))


def test_short_units_in_two_waves(kv):
    """The same in the two-wave form that launches of 0.5 M keys take for such units (2 M for units of 16 to 63 tokens),
    with 512-key slices."""
    P, Hkv, N, n = 41, 8, 6400, 4096
    rng = np.random.default_rng(11)
    assert P * Hkv * N >= 2 << 20
    _check_scores(kv, rng, P, 4, Hkv, 32, 128, torch.bfloat16, N, _tiny_units(rng, P, N, n), (0, P - 1))


@pytest.mark.parametrize("unit", [7, 8, 31, 33])
@pytest.mark.parametrize("G,D,dtype", [(4, 128, torch.bfloat16), (8, 64, torch.bfloat16), (6, 64, torch.bfloat16),
                                       (1, 128, torch.float32)])
def test_ends_at_every_row_of_a_block(kv, G, D, dtype, unit):
    """Units whose ends take every place in a block and in its groups of eight rows: one end a block or several, on the
    edges of groups (8) and inside all of them, with one to three row blocks per wave."""
    N, n = 2400, 2200 // unit
    rng = np.random.default_rng(G * unit + D)
    offs = (5 + unit * np.arange(n + 1, dtype=np.int32))[None]
    _check_scores(kv, rng, 1, G, 2, 32, D, dtype, N, offs, (0,))


@pytest.mark.parametrize("D,dtype", [(128, torch.bfloat16), (64, torch.bfloat16), (128, torch.float32)])
def test_poisoned_keys_stay_in_their_unit(kv, D, dtype):
    """NaN keys take their slice out of the row denominators and their unit out of the slice; the other units keep finite
    scores, the same whether one key is NaN or two next to each other in a block that holds a unit's end."""
    P, Hkv, G, W, N = 1, 2, 4, 32, 600
    gen = torch.Generator(device="cuda").manual_seed(D)
    q, k = (torch.randn((P, h, n, D), generator=gen, device="cuda").to(dtype) for h, n in ((Hkv * G, W), (Hkv, N)))
    offs = torch.arange(0, 561, 20, dtype=torch.int32, device="cuda")[None]

    def scores(*keys):
        x = k.clone()
        x[:, :, list(keys)] = float("nan")
        s, status = kv.prefill_scores(q, x, offs, D ** -0.5)
        torch.cuda.synchronize()
        assert not status.any()
        return s[0].cpu().numpy()

    for key in (32, 36, 160, 288):      # rows 0 and 4 of a block, the first elements of a lane of either half
        unit = key // 20
        one, two = np.delete(scores(key + 1), unit), np.delete(scores(key, key + 1), unit)
        assert np.isfinite(one).all() and (one > 0).all()
        np.testing.assert_allclose(two, one, rtol=SCORE_RTOL, atol=0, err_msg=str(key))


@pytest.mark.parametrize("attention", [False, True])
@pytest.mark.parametrize("N,n", [(4001, 24), (16384, 600)])
def test_scores_have_no_bias(kv, N, n, attention):
    """The mean over all shots of the scores' relative error.  A rounding to nearest in a chunk's statistic, in a
    denominator or in a sum averages out over shots, rows and heads; what would stay is an error of one sign, such as a
    logarithm that errs low by a part of its last place (1e-7 to 2.8e-7 here).  5e-8 is a third of a float32's last
    place (the mean of the final divisions' own roundings is 2^-24 / sqrt(n) at most)."""
    if attention and N > 4001:
        pytest.skip("the statistics are those of the smaller case")
    H, Hkv, W, D, scale = 32, 8, 32, 128, 1.0 / math.sqrt(128)
    gen = torch.Generator(device="cuda").manual_seed(N)
    q = torch.randn((1, H, N if attention else W, D), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((1, Hkv, N, D), generator=gen, device="cuda").to(torch.bfloat16)
    off = torch.linspace(0, N - 200, n + 1).int()[None].cuda()
    if attention:
        bud = torch.tensor([N // 2], dtype=torch.int32, device="cuda")
        scores = kv.prefill_attention_compress(q, k, k, off, bud, N // 2, W, scale)[1].shot_scores
    else:
        scores, _ = kv.prefill_scores(q, k, off, scale)
    torch.cuda.synchronize()
    off = off[0].cpu().numpy()
    mass = orc.token_mass(orc.window_attention(to_np(q[0, :, -W:]), to_np(k[0]), scale))
    want = orc.shot_scores_from_mass(mass, off)
    rel = scores[0].cpu().numpy().astype(np.float64) / want - 1
    assert abs(rel.mean()) < 5e-8, rel.mean()
