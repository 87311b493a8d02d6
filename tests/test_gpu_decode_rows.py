"""GPU parity of the decode step where its blocks end: every row size (dtype, head dimension), group size and cache
length around the blocks of rows a wave takes, with dead prefill rows and free slots holding values that would
show (huge, infinite, NaN), pools with holes, and a context long enough for a range to be taken in pieces."""
import numpy as np
import pytest
import torch

from helpers import to_np
from oracle import shotkv_oracle as orc

pytestmark = pytest.mark.gpu

# float32 logits, weights and sums over up to a few hundred rows against float64: a logit is off by at most
# 2 * head_dim roundings of 2^-24 of its terms (|logit| < 30 here), which is the weight's relative error
RTOL = 2e-5


@pytest.fixture(scope="module")
def kv():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_01941_amd import shotkv
    shotkv.load_library()
    return shotkv


def _state(kv, rng, S, H, Hkv, D, dtype, cap, counts, n_slots, used, budget, scale, on_gpu=False):
    """Random caches (on_gpu: drawn there, for large ones); rows past a sequence's count and slots that are not in `used` hold
    poison."""
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30))) if on_gpu else None

    def normal(*shape):
        if on_gpu:
            return torch.randn(shape, generator=gen, device="cuda").to(dtype)
        return torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)).to(dtype).cuda()
    kp, vp = normal(S, Hkv, cap, D), normal(S, Hkv, cap, D)
    kd, vd = normal(S, Hkv, n_slots, D), normal(S, Hkv, n_slots, D)
    slot_pos = torch.full((S, n_slots), -1, dtype=torch.int32, device="cuda")
    poison_k, poison_v = [3e30, float("nan"), float("-inf")], [float("nan"), float("inf"), -3e30]
    for s in range(S):
        kp[s, :, counts[s]:] = poison_k[s % 3]
        vp[s, :, counts[s]:] = poison_v[s % 3]
        free = np.setdiff1d(np.arange(n_slots), used[s])
        kd[s, :, free], vd[s, :, free] = poison_k[(s + 1) % 3], poison_v[(s + 1) % 3]
        slot_pos[s, used[s]] = torch.arange(len(used[s]), dtype=torch.int32, device="cuda")
    count = torch.tensor(counts, dtype=torch.int32, device="cuda")
    return kv.DecodeState(kp, vp, count, kd, vd, slot_pos, budget, H, scale)


def _check_steps(kv, rng, state, budget, n_steps, scale, first_step=1000, sequences=None):
    """Steps against the oracle: every sequence, or those given."""
    S, H, Hkv, D, dtype = state.S, state.H, state.H_kv, state.D, state.dtype
    sequences = range(S) if sequences is None else sequences
    host = {}
    for s in sequences:
        c = int(state.prefill_count[s].item())
        host[s] = [to_np(state.k_prefill[s, :, :c]), to_np(state.v_prefill[s, :, :c]), c, to_np(state.k_dec[s]).copy(),
                   to_np(state.v_dec[s]).copy(), state.slot_pos[s].cpu().numpy().copy()]
    for step in range(first_step, first_step + n_steps):
        new = [torch.from_numpy(rng.standard_normal((S, h, D), dtype=np.float32)).to(dtype).cuda() for h in (H, Hkv, Hkv)]
        kv.decode_step(state, step, *new)
        torch.cuda.synchronize()
        for s in sequences:
            kp, vp, c, kd, vd, sp = host[s]
            with np.errstate(invalid="ignore", over="ignore"):
                r = orc.decode_step(kp, vp, c, kd, vd, sp, budget, step, *[to_np(t[s]) for t in new], scale)
            assert int(state.status[s]) == r["status"]
            got = state.out[s].cpu().numpy()
            assert np.all(np.abs(got - r["out"]) <= RTOL * np.abs(r["out"]).max(axis=1, keepdims=True)), (step, s)
            np.testing.assert_allclose(state.token_scores[s].cpu().numpy(), r["token_scores"], rtol=RTOL, atol=1e-30)
            assert r["margin"] > 1e-6 and int(state.evicted_pos[s]) == r["evicted_pos"]
            np.testing.assert_array_equal(state.slot_pos[s].cpu().numpy(), sp)
            np.testing.assert_array_equal(to_np(state.k_dec[s]), kd)
            np.testing.assert_array_equal(to_np(state.v_dec[s]), vd)


@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("D,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
def test_row_counts_around_the_blocks(kv, D, dtype, G):
    rng = np.random.default_rng(100 * G + D + (dtype == torch.float32))
    S, Hkv = 3, 2
    for cap, n_slots in [(0, 5), (1, 1), (16, 17), (17, 33), (32, 130), (33, 9), (64, 64), (65, 257), (127, 128), (129, 40),
                         (300, 300)]:
        counts = [cap, int(rng.integers(0, cap + 1)), max(cap - 1, 0)]
        used = [np.arange(n_slots - 1),                                       # full but for the last slot
                np.sort(rng.choice(n_slots, size=n_slots // 2, replace=False)),  # holes
                np.arange(min(3, n_slots - 1))]                               # still filling up
        budget = max(1, n_slots - 1)
        scale = 1.0 / np.sqrt(D)
        state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, counts, n_slots, used, budget, scale)
        _check_steps(kv, rng, state, budget, 2 if n_slots > 1 else 1, scale)


@pytest.mark.parametrize("D,dtype,cap", [(64, torch.bfloat16, 1_049_000), (128, torch.float32, 1_100_003)])
def test_ranges_longer_than_the_logit_buffer(kv, D, dtype, cap):
    """More than 2^20 tokens: a range is taken in pieces of 1024 rows, the pool's slots in the last one."""
    rng = np.random.default_rng(cap)
    n_slots, scale = 700, 1.0 / np.sqrt(D)
    state = _state(kv, rng, 1, 4, 1, D, dtype, cap, [cap - 5], n_slots, [np.arange(n_slots - 1)], n_slots - 1, scale)
    _check_steps(kv, rng, state, n_slots - 1, 2, scale)


@pytest.mark.parametrize("D,dtype,cap,n_slots,free", [
    (64, torch.bfloat16, 1_049_000, 700, 597), (128, torch.float32, 1_049_000, 3000, 1613), (64, torch.bfloat16, 2_100_000, 5000, 3282)])
def test_new_token_in_a_later_piece(kv, D, dtype, cap, n_slots, free):
    """Ranges of 1026, 1028 and 2056 tokens in pieces of 1024; the free slot lies in the second (third) piece of its
    range, and the pool's slots lie in several pieces of several ranges."""
    per_range = -(-(cap + n_slots) // 1024)
    assert (cap + free) % per_range >= per_range // 1024 * 1024 >= 1024
    rng = np.random.default_rng(free)
    scale = 1.0 / np.sqrt(D)
    used = np.setdiff1d(np.arange(n_slots), [free])
    state = _state(kv, rng, 1, 4, 1, D, dtype, cap, [cap - 5], n_slots, [used], n_slots - 1, scale)
    _check_steps(kv, rng, state, n_slots - 1, 2, scale)


@pytest.mark.parametrize("S", [128, 129])
def test_ranges_of_nothing_but_slots(kv, S):
    """Caches without prefill rows, in launches of up to 1024 workgroups (128 sequences of 8 KV heads here) and larger ones;
    free slots hold poison, and the new token's slot lies at the start, inside and behind the occupied ones."""
    rng = np.random.default_rng(S)
    Hkv, D, n_slots, budget = 8, 64, 40, 39
    used = [np.setdiff1d(np.arange(n_slots), [0, 7, 31] if s % 3 == 0 else [5, 6, 39] if s % 3 == 1 else np.arange(20, 40))
            for s in range(S)]
    scale = D ** -0.5
    state = _state(kv, rng, S, Hkv, Hkv, D, torch.bfloat16, 0, [0] * S, n_slots, used, budget, scale)
    _check_steps(kv, rng, state, budget, 2, scale)


@pytest.mark.parametrize("S,Hkv,G,cap,n_slots,budget,first_step", [
    (3, 2, 4, 410, 205, 204, 1000),     # short ranges: rows requested ahead of the map
    (3, 2, 4, 409, 205, 204, 1000),
    (3, 2, 8, 410, 205, 204, 1000),
    (3, 2, 4, 410, 205, 40, 1000),      # a budget below, and a step before, what the pool holds: the blocks behind it are
    (3, 2, 4, 410, 205, 204, 60),       # requested after the map
    (64, 8, 1, 200, 400, 399, 1000),    # two ranges of 300 rows, the second of slots only: ahead
    (64, 8, 1, 200, 400, 399, 110),
    (103, 5, 1, 400, 700, 699, 1000),   # 1030 workgroups: after the map
])
@pytest.mark.parametrize("D,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
def test_slots_requested_ahead_of_their_map_and_not(kv, D, dtype, S, Hkv, G, cap, n_slots, budget, first_step):
    """Ranges of nothing but slots behind ranges of prefill rows, where their first rows are requested before the slot map
    is known and where they are not; free slots hold poison, and the new token's slot lies at the start of the pool, in the
    first block of a later range, and behind the occupied slots."""
    rng = np.random.default_rng(S + G + cap + first_step)
    mid = n_slots // 2 + 3
    free = [[0, mid, n_slots - 1], [mid, mid + 1, n_slots - 2], np.arange(n_slots // 4, n_slots)]
    used = [np.setdiff1d(np.arange(n_slots), free[s % 3]) for s in range(S)]
    scale = D ** -0.5
    state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, [cap - s % 7 for s in range(S)], n_slots, used, budget, scale)
    _check_steps(kv, rng, state, budget, 2, scale, first_step)


@pytest.mark.parametrize("D,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
def test_infinite_values_stay_in_their_column(kv, D, dtype):
    """The last live prefill row and the last occupied slot hold an infinite value each: it shows in its own output
    column as infinity, and nowhere else (padding rows that read it again must not turn it into NaN)."""
    rng = np.random.default_rng(D)
    cap, n_slots, H, Hkv, scale = 200, 40, 8, 2, 1.0 / np.sqrt(D)
    state = _state(kv, rng, 1, H, Hkv, D, dtype, cap, [77], n_slots, [np.arange(23)], 39, scale)
    state.v_prefill[0, :, 76, 5], state.v_dec[0, :, 22, 9] = float("inf"), float("-inf")
    kp, vp = to_np(state.k_prefill[0, :, :77]), to_np(state.v_prefill[0, :, :77])
    kd, vd, sp = to_np(state.k_dec[0]).copy(), to_np(state.v_dec[0]).copy(), state.slot_pos[0].cpu().numpy().copy()
    new = [torch.from_numpy(rng.standard_normal((1, h, D), dtype=np.float32)).to(dtype).cuda() for h in (H, Hkv, Hkv)]
    kv.decode_step(state, 1000, *new)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore", over="ignore"):
        ref = orc.decode_step(kp, vp, 77, kd, vd, sp, 39, 1000, *[to_np(t[0]) for t in new], scale)["out"]
    got = state.out[0].cpu().numpy()
    assert np.all(got[:, 5] == np.inf) and np.all(got[:, 9] == -np.inf)
    rest = np.setdiff1d(np.arange(D), [5, 9])
    assert np.all(np.abs(got[:, rest] - ref[:, rest]) <= RTOL * np.abs(ref[:, rest]).max(axis=1, keepdims=True))


def test_float32_rounding_of_the_output(kv):
    """Error of the attention output of float32 caches against float64, over the norm, mean of three seeds.  Logits of
    128 products in four chains per lane and a tree give 1.84e-7, as plain vector arithmetic did (four products per lane
    and a tree over the lanes); a single chain per lane gives 2.1e-7.  The bound lies between the two."""
    S, H, Hkv, D, cap, n_slots, scale = 4, 32, 8, 128, 500, 200, 1.0 / np.sqrt(128)
    errors = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        state = _state(kv, rng, S, H, Hkv, D, torch.float32, cap, [cap] * S, n_slots, [np.arange(n_slots - 1)] * S, n_slots,
                       scale)
        new = [torch.from_numpy(rng.standard_normal((S, h, D), dtype=np.float32)).cuda() for h in (H, Hkv, Hkv)]
        kd, vd, sp = to_np(state.k_dec).copy(), to_np(state.v_dec).copy(), state.slot_pos.cpu().numpy().copy()
        kv.decode_step(state, 1000, *new)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore", over="ignore"):
            want = np.stack([orc.decode_step(to_np(state.k_prefill[s]), to_np(state.v_prefill[s]), cap, kd[s], vd[s], sp[s],
                                             n_slots, 1000, *[to_np(t[s]) for t in new], scale)["out"] for s in range(S)])
        got = state.out.cpu().numpy().astype(np.float64)
        errors.append(np.linalg.norm(got - want) / np.linalg.norm(want))
    print("output error", errors)
    assert np.mean(errors) < 1.95e-7
