"""GPU parity of the fused attention pass where its softmax reference has to move late: rows whose logits grow along
the prompt, by a little in every block or at once by far more than fp16 holds, and rows whose first keys are the
heaviest; what its position does to the weights' precision, and values that are not finite."""
import math

import numpy as np
import pytest
import torch

from helpers import to_np
from oracle import shotkv_oracle as orc

pytestmark = pytest.mark.gpu

OUT_TOL = 1e-3        # |dO| <= OUT_TOL * max|O| per query row (weights reach the matrix cores with 11 significant bits)


@pytest.fixture(scope="module")
def kv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_01941_amd import shotkv
    shotkv.load_library()
    return shotkv


@pytest.mark.parametrize("growth", ["steady", "late_jump", "jump_each_block", "falling", "huge"])
@pytest.mark.parametrize("N", [513, 1100])
def test_logits_that_grow_along_the_prompt(kv, N, growth):
    H, Hkv, W, D, n = 4, 2, 32, 128, 5
    rng = np.random.default_rng(N + len(growth))
    q = np.abs(rng.standard_normal((1, H, N, D), dtype=np.float32))
    k = 0.05 * rng.standard_normal((1, Hkv, N, D), dtype=np.float32)
    t = np.arange(N, dtype=np.float32)[:, None]
    k += {"steady": 0.25 * t / N, "late_jump": 0.4 * (t >= 512 + 7), "jump_each_block": 0.02 * (t // 32),
          "falling": 0.4 * (1 - t / N), "huge": 8.0 * (t >= 40) * (t % 97 == 3)}[growth]
    scale = 1.0 / math.sqrt(D)
    q, k = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (q, k))
    v = torch.from_numpy(rng.standard_normal((1, Hkv, N, D), dtype=np.float32)).to(torch.bfloat16).cuda()
    off = torch.from_numpy(np.linspace(3, N - 40, n + 1).astype(np.int32)[None]).cuda()
    bud = torch.tensor([N // 2], dtype=torch.int32, device="cuda")
    attn, res = kv.prefill_attention_compress(q, k, v, off, bud, N // 2, W, scale)
    torch.cuda.synchronize()
    ref = orc.causal_attention(to_np(q[0]), to_np(k[0]), to_np(v[0]), scale)
    got = attn[0].cpu().numpy()
    assert np.all(np.abs(got - ref) <= OUT_TOL * np.abs(ref).max(axis=2, keepdims=True))
    want = orc.prefill_compress(to_np(q[0, :, -W:]), to_np(k[0]), to_np(v[0]), off[0].cpu().numpy(), N // 2, scale)
    # shots that get less than 1e-30 of the weight may underflow to zero
    np.testing.assert_allclose(res.shot_scores[0].cpu().numpy(), want["scores"], rtol=2e-5, atol=1e-30)


@pytest.mark.parametrize("heavy", [0, 300])
def test_light_keys_keep_their_bits_behind_a_heavy_one(kv, heavy):
    """One key takes nearly all of the weight and carries a zero value, so the output is made by keys of 2^-28 .. 2^-29
    of it.  The softmax reference sits 15 (log2) below the maximum: their fp16 weights are at least 2^-14, the smallest
    with all 11 bits, and each is off by at most 2^-11; the values are positive, so that bounds the sum's error too."""
    H, Hkv, W, D, N, n = 4, 2, 32, 128, 700, 4
    rng = np.random.default_rng(heavy)
    q = np.zeros((1, H, N, D), dtype=np.float32)
    q[..., 0] = 1.0
    k = 0.1 * rng.standard_normal((1, Hkv, N, D), dtype=np.float32)
    k[..., 0] = -rng.random((1, Hkv, N), dtype=np.float32)      # light logits -1 .. 0 in the log2 domain
    k[..., heavy, 0] = 28.0
    v = 0.5 + rng.random((1, Hkv, N, D), dtype=np.float32)
    v[..., heavy, :] = 0.0
    scale = math.log(2.0)
    q, k, v = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (q, k, v))
    off = torch.from_numpy(np.linspace(3, N - 40, n + 1).astype(np.int32)[None]).cuda()
    bud = torch.tensor([N // 2], dtype=torch.int32, device="cuda")
    attn, _ = kv.prefill_attention_compress(q, k, v, off, bud, N // 2, W, scale)
    torch.cuda.synchronize()
    ref = orc.causal_attention(to_np(q[0]), to_np(k[0]), to_np(v[0]), scale)
    got = attn[0].cpu().numpy()
    assert np.all(np.abs(got - ref) <= OUT_TOL * np.abs(ref).max(axis=2, keepdims=True))


def test_rows_that_two_keys_share(kv):
    """Two keys of nearly the same weight and opposite values, behind a first key whose weight is a little less and whose
    value is zero.  Every fp16 weight but the row's largest, which is a power of two, is off by at most 2^-11 of itself, and
    the sum of the weights is taken before they are rounded, so an output is off by at most 2^-11 of what the lighter of the
    two adds to it (and 2^-18 for the fp32 sums).  Weights rounded in the sum too, or a largest weight that is not a power of
    two, give up to twice that."""
    H, Hkv, W, D, N, n = 4, 2, 32, 128, 700, 4
    rng = np.random.default_rng(2)
    heavy = [40, 75]
    q = np.zeros((1, H, N, D), dtype=np.float32)
    q[..., 0] = 1.0
    q[..., 1:3] = 0.5 * rng.random((1, H, N, 2), dtype=np.float32)      # logits (log2 domain) of the two
    k = np.zeros((1, Hkv, N, D), dtype=np.float32)
    k[..., 1:, 0] = -100.0                                              # every key but the first: no weight
    k[..., heavy, 0] = 0.0
    k[..., heavy[0], 1] = k[..., heavy[1], 2] = 1.0
    v = np.zeros((1, Hkv, N, D), dtype=np.float32)
    v[..., heavy, :] = np.where(rng.random((1, Hkv, 2, D)) < 0.5, -1.0, 1.0)
    scale = math.log(2.0)
    q, k, v = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (q, k, v))
    off = torch.from_numpy(np.linspace(3, N - 40, n + 1).astype(np.int32)[None]).cuda()
    bud = torch.tensor([N // 2], dtype=torch.int32, device="cuda")
    attn, _ = kv.prefill_attention_compress(q, k, v, off, bud, N // 2, W, scale)
    torch.cuda.synchronize()
    got = attn[0].cpu().numpy().astype(np.float64)
    qh, vh = to_np(q[0]).astype(np.float64), to_np(v[0]).astype(np.float64)
    rows = slice(heavy[1], N)
    logits = np.concatenate([np.zeros((H, N, 1)), qh[..., 1:3]], axis=2)[:, rows]
    p = np.exp2(logits)
    p /= p.sum(axis=2, keepdims=True)
    lighter = np.minimum(p[..., 1], p[..., 2])
    ref = np.stack([p[h, :, 1:] @ vh[h // (H // Hkv), heavy] for h in range(H)])
    assert np.all(np.abs(got[:, rows] - ref) <= 2.0 ** -11 * lighter[..., None] + 2.0 ** -18)


@pytest.mark.parametrize("what,value", [("q", math.nan), ("q", math.inf), ("k", math.nan), ("k", math.inf), ("k", -math.inf),
                                        ("v", math.nan), ("v", math.inf)])
def test_values_that_are_not_finite_stay_where_they_belong(kv, what, value):
    """One infinite or NaN query, key or value element, in tiles with and without window rows.  Queries are positive in that
    dimension.  A query shows in its own row, a key in the rows of its query heads from its position on (minus infinity: as
    a key that is not there), a value in its column of the rows that can see its block of 32 keys.  Everything else is bit
    for bit what it is without it: no other row of the wave, which shares the rescaling, is touched."""
    H, Hkv, W, D, N, n, dim = 4, 2, 32, 128, 700, 4, 9
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, h, N, D), generator=gen, device="cuda") for h in (H, Hkv, Hkv))
    q[..., dim] = q[..., dim].abs() + 0.5
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    off = torch.from_numpy(np.linspace(3, N - 40, n + 1).astype(np.int32)[None]).cuda()
    bud = torch.tensor([N // 2], dtype=torch.int32, device="cuda")

    def run(q, k, v):
        attn, _ = kv.prefill_attention_compress(q, k, v, off, bud, N // 2, W, D ** -0.5)
        torch.cuda.synchronize()
        return attn[0]

    clean = run(q, k, v)
    for at in (0, 37, 300, 511, 660, 690):
        t = {"q": q.clone(), "k": k.clone(), "v": v.clone()}
        t[what][0, 1, at, dim] = value
        got = run(t["q"], t["k"], t["v"])
        touched = torch.zeros_like(clean, dtype=torch.bool)
        if what == "q":
            touched[1, at] = True
        elif what == "k":
            touched[2:, at:] = True         # query heads 2 and 3 read KV head 1
        else:
            touched[2:, at // 32 * 32:, dim] = True
        assert torch.equal(got[~touched], clean[~touched]), at
        if what == "k" and value < 0:       # no weight; row 0 has no other key
            with np.errstate(invalid="ignore"):
                ref = orc.causal_attention(to_np(q[0, 2:]), to_np(t["k"][0, 1:]), to_np(v[0, 1:]), D ** -0.5)[:, 1:]
            assert np.all(np.abs(got[2:, 1:].cpu().numpy() - ref) <= OUT_TOL * np.abs(ref).max(axis=2, keepdims=True)), at
        else:
            shown = got[2:, at:, dim] if what == "v" else got[touched]
            assert not torch.isfinite(shown).any(), at
