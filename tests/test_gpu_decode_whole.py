"""GPU parity of decode steps over many sequences, where one workgroup takes all of a (sequence, KV head), and of launches
just too small for that: prefill rows around the pieces that fit into LDS and around the blocks that are dealt to the waves,
every row size and group size, pools with one slot left, with holes and still filling up, poison in dead rows and free
slots; pools without a free slot among such pools."""
import numpy as np
import pytest
import torch

from helpers import to_np
from oracle import shotkv_oracle as orc
from test_gpu_decode_rows import RTOL, _check_steps, _state, kv  # noqa: F401

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


def _run(kv, S, G, Hkv, D, dtype, cap, n_slots, seed):
    rng = np.random.default_rng(seed)
    counts = [cap if s % 3 == 0 else int(rng.integers(0, cap + 1)) for s in range(S)]
    counts[1] = 0
    used = [np.arange(n_slots - 1) if s % 3 == 0 else np.sort(rng.choice(n_slots, size=n_slots // 2, replace=False)) if s % 3 == 1
            else np.arange(min(3, n_slots - 1)) for s in range(S)]
    budget, scale = max(1, n_slots - 1), 1.0 / np.sqrt(D)
    state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, counts, n_slots, used, budget, scale, on_gpu=True)
    _check_steps(kv, rng, state, budget, 1, scale, sequences=range(0, S, 2 if S > 150 else 1))  # (of all kinds)


def _sequences(G):
    """Of 8 KV heads: two rounds of the workgroups that share the chip, two to four per CU, from which on one workgroup takes a
    (sequence, KV head) of two to four query heads, or of seven or eight with rows of 128 bytes.  (All others are always taken
    in ranges.)"""
    return {2: 256, 3: 192, 4: 192}.get(G, 128)


@pytest.mark.parametrize("D,dtype", [(64, BF16), (128, BF16), (64, F32), (128, F32)])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
def test_one_workgroup_for_a_short_sequence(kv, G, D, dtype):  # noqa: F811
    """Two rounds of (sequence, KV head) pairs, and two and a half."""
    S = _sequences(G)
    _run(kv, S, G, 8, D, dtype, 230, 840, G)
    _run(kv, S + S // 4, G, 8, D, dtype, 1031, 43, G + 1)


@pytest.mark.parametrize("G,D,dtype,over", [(2, 128, BF16, 0), (4, 128, BF16, 1), (2, 64, BF16, 1), (8, 64, BF16, 0),
                                            (3, 128, F32, 1), (4, 64, F32, 17), (7, 64, BF16, 31)])
def test_one_workgroup_for_several_pieces(kv, G, D, dtype, over):  # noqa: F811
    """Prefill rows up to the end of a piece of four waves and past it, then the slots in a piece of their own."""
    piece = {128: 1152, 256: 1088, 512: 1056}[D * (2 if dtype == BF16 else 4)]
    _run(kv, _sequences(G), G, 8, D, dtype, piece + over, 65, 10 * G + over)


def test_as_many_slots_as_the_map_holds(kv):  # noqa: F811
    for n_slots in (1088, 1089):  # the second takes more than one workgroup
        _run(kv, 256, 2, 8, 128, BF16, 20, n_slots, n_slots)


@pytest.mark.parametrize("G,D,S,whole", [(4, 128, 191, False), (4, 128, 192, True), (3, 128, 200, False), (3, 64, 216, True),
                                         (2, 64, 255, False), (2, 64, 287, False), (2, 64, 288, True),
                                         (8, 64, 127, False), (7, 64, 144, True), (6, 64, 128, False)])
def test_rounds_that_are_not_full(kv, G, D, S, whole):  # noqa: F811
    """One pair less than two rounds, and a third round that is begun, or has a quarter of its places taken, from which on
    (`whole`) one workgroup takes a sequence."""
    _run(kv, S, G, 8, D, BF16, 900, 257, S + G)


@pytest.mark.parametrize("G,S,cap", [(4, 128, 4000), (2, 192, 3100), (8, 128, 4200)])
def test_more_ranges_than_a_round(kv, G, S, cap):  # noqa: F811
    """Launches of few sequences that are over a round of workgroups in ranges of 1024 tokens."""
    _run(kv, S, G, 2, 64, BF16, cap, 150, S + G)


@pytest.mark.parametrize("S,Hkv,G,D,cap,n_slots", [
    (192, 8, 4, 64, 2000, 2),       # one workgroup for a sequence, two full rounds of them
    (1536, 1, 4, 64, 2000, 2),      # the same as caches with a slot map for every KV head
    (256, 8, 2, 64, 1500, 40), (128, 8, 8, 64, 1500, 40),
    (128, 2, 4, 64, 4000, 150)])    # ranges
def test_full_pools_among_others(kv, S, Hkv, G, D, cap, n_slots):  # noqa: F811
    """A sequence whose pool has no free slot reports that and changes nothing, neither its own caches nor the scores of
    other sequences of the launch, finished long before or still running."""
    rng = np.random.default_rng(S + Hkv)
    full = [s >= S // 3 and s % 4 == 1 for s in range(S)]
    counts = [cap if full[s] else int(rng.integers(1, cap // 8)) for s in range(S)]
    used = [np.arange(n_slots) if full[s] else np.arange(n_slots - 1) for s in range(S)]
    budget, scale = n_slots - 1, D ** -0.5
    state = _state(kv, rng, S, Hkv * G, Hkv, D, BF16, cap, counts, n_slots, used, budget, scale)
    before = [t.clone() for t in (state.k_dec, state.v_dec, state.slot_pos)]
    new = [torch.from_numpy(rng.standard_normal((S, h, D), dtype=np.float32)).to(BF16).cuda() for h in (Hkv * G, Hkv, Hkv)]
    state.out.fill_(7.0)
    state.token_scores.fill_(7.0)
    kv.decode_step(state, 1000, *new)
    torch.cuda.synchronize()
    is_full = torch.tensor(full, device="cuda")
    assert torch.equal(state.status == orc.STATUS_NO_FREE_SLOT, is_full) and bool((state.status[~is_full] == orc.STATUS_OK).all())
    assert not state.out[is_full].any() and not state.token_scores[is_full].any()
    assert bool((state.evicted_pos[is_full] == -1).all())
    for now, then in zip((state.k_dec, state.v_dec, state.slot_pos), before):
        assert torch.equal(now[is_full].nan_to_num(1.25), then[is_full].nan_to_num(1.25))
    for s in np.flatnonzero(~np.array(full)):
        kd, vd, sp = (to_np(t[s]).copy() if t.is_floating_point() else t[s].cpu().numpy() for t in before)
        kp, vp = to_np(state.k_prefill[s, :, :counts[s]]), to_np(state.v_prefill[s, :, :counts[s]])
        with np.errstate(invalid="ignore", over="ignore"):
            r = orc.decode_step(kp, vp, counts[s], kd, vd, sp, budget, 1000, *[to_np(t[s]) for t in new], scale)
        np.testing.assert_allclose(state.token_scores[s].cpu().numpy(), r["token_scores"], rtol=RTOL, atol=1e-30)
        got = state.out[s].cpu().numpy()
        assert np.all(np.abs(got - r["out"]) <= RTOL * np.abs(r["out"]).max(axis=1, keepdims=True)), s
        assert int(state.evicted_pos[s]) == r["evicted_pos"]


@pytest.mark.parametrize("S,Hkv,G,D,dtype,cap,n_slots", [
    (192, 8, 4, 128, BF16, 700, 600), (256, 8, 2, 64, BF16, 1200, 800), (128, 8, 8, 64, BF16, 500, 700),
    (192, 8, 3, 128, F32, 700, 600), (1536, 1, 4, 64, F32, 700, 600)])
def test_tokens_of_equal_keys_score_the_same_in_every_wave(kv, S, Hkv, G, D, dtype, cap, n_slots):  # noqa: F811
    """Twelve slots, in blocks of every wave, hold one key that is opposed to the queries: their scores are the lowest and
    equal to the last bit, whatever logits the waves that take them saw beside them, so the newest token goes."""
    rng = np.random.default_rng(S + G)
    scale = D ** -0.5
    state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, [cap - s % 100 for s in range(S)], n_slots,
                   [np.arange(n_slots - 1)] * S, n_slots - 1, scale)
    q, kn, vn = (torch.from_numpy(rng.standard_normal((S, h, D), dtype=np.float32)).to(dtype).cuda()
                 for h in (Hkv * G, Hkv, Hkv))
    block = 4096 // (D * (2 if dtype == BF16 else 4))
    at = np.concatenate([np.arange(12)[:, None] * block + [3]])[:, 0]      # in twelve blocks that follow one another
    assert at[-1] < n_slots - 1
    toward = q.float().reshape(S, Hkv, G, D).mean(dim=2)
    state.k_dec[:, :, at] = (-1.5 * toward).to(dtype)[:, :, None]
    kv.decode_step(state, 5000, q, kn, vn)
    torch.cuda.synchronize()
    scores = state.token_scores[:, at]
    assert torch.equal(scores, scores[:, :1].expand_as(scores))
    others = torch.cat([state.token_scores[:, :n_slots - 1][:, np.setdiff1d(np.arange(n_slots - 1), at)]], dim=1)
    lowest = scores[:, 0] < others.min(dim=1).values
    assert int(lowest.sum()) > S // 2                                       # the case is really hit
    assert bool((state.evicted_pos[lowest] == int(at[-1])).all())


@pytest.mark.parametrize("S,Hkv,G,D,dtype,cap,n_slots", [
    (192, 8, 4, 128, BF16, 1200, 300), (256, 8, 2, 64, F32, 1300, 300), (128, 8, 7, 64, BF16, 500, 700),   # one workgroup
    (64, 4, 4, 64, BF16, 4000, 150), (20, 8, 8, 64, BF16, 500, 700), (3, 8, 4, 128, BF16, 700, 300)])      # ranges
def test_values_that_are_not_finite(kv, S, Hkv, G, D, dtype, cap, n_slots):  # noqa: F811
    """Infinite values show in their column, keys that leave a head no finite logit make its outputs NaN and, as sums over the
    heads, the scores; a NaN query likewise.  Other heads and other sequences are as the oracle has them."""
    rng = np.random.default_rng(S + G)
    budget, scale = n_slots - 1, D ** -0.5
    counts = [cap - 3 * (s % 7) for s in range(S)]
    state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, counts, n_slots, [np.arange(n_slots - 1)] * S, budget, scale)
    new = [torch.from_numpy(rng.standard_normal((S, h, D), dtype=np.float32)).to(dtype).cuda() for h in (Hkv * G, Hkv, Hkv)]
    state.v_prefill[0, :, counts[0] - 1, 5], state.v_dec[0, :, n_slots - 2, 9] = float("inf"), float("-inf")
    for t in (state.k_prefill[1, 0, :counts[1]], state.k_dec[1, 0, :n_slots - 1], new[1][1, 0]):
        t[..., 0] = float("-inf")
    new[0][1, :G, 0] = 1.0                  # sequence 1, KV head 0: every logit is minus infinity
    new[0][2, G - 1, 7] = float("nan")      # sequence 2: one query head
    before = [t.clone() for t in (state.k_dec, state.v_dec, state.slot_pos)]
    kv.decode_step(state, 1000, *new)
    torch.cuda.synchronize()
    for s in [0, 1, 2, S // 2 + 1, S - 1]:
        kd, vd, sp = (to_np(t[s]).copy() if t.is_floating_point() else t[s].cpu().numpy() for t in before)
        kp, vp = to_np(state.k_prefill[s, :, :counts[s]]), to_np(state.v_prefill[s, :, :counts[s]])
        with np.errstate(invalid="ignore", over="ignore"):
            r = orc.decode_step(kp, vp, counts[s], kd, vd, sp, budget, 1000, *[to_np(t[s]) for t in new], scale)
        assert int(state.status[s]) == orc.STATUS_OK
        got, want = state.out[s].cpu().numpy(), r["out"]
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want)), s
        assert np.array_equal(np.isneginf(got), np.isneginf(want)), s
        assert np.isfinite(want).all() == (s > 2)
        finite = np.isfinite(want)
        top = np.abs(np.where(finite, want, 0)).max(axis=1, keepdims=True)
        assert np.all(np.abs(got[finite] - want[finite]) <= np.broadcast_to(RTOL * top, got.shape)[finite]), s
        np.testing.assert_allclose(state.token_scores[s].cpu().numpy(), r["token_scores"], rtol=RTOL, atol=1e-30)
