"""GPU parity of decode steps over many sequences, where one workgroup takes all of a (sequence, KV head) or a few take long
ranges: prefill rows around the pieces that fit into LDS and around the blocks that are dealt to the waves, every row size
and group size, pools full, with holes and still filling up, poison in dead rows and free slots."""
import numpy as np
import pytest
import torch

from test_gpu_decode_rows import _check_steps, _state, kv  # noqa: F401

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


def _run(kv, S, G, Hkv, D, dtype, cap, n_slots, seed):
    rng = np.random.default_rng(seed)
    counts = [cap if s % 3 == 0 else int(rng.integers(0, cap + 1)) for s in range(S)]
    counts[1] = 0
    used = [np.arange(n_slots - 1) if s % 3 == 0 else np.sort(rng.choice(n_slots, size=n_slots // 2, replace=False)) if s % 3 == 1
            else np.arange(min(3, n_slots - 1)) for s in range(S)]
    budget, scale = max(1, n_slots - 1), 1.0 / np.sqrt(D)
    state = _state(kv, rng, S, Hkv * G, Hkv, D, dtype, cap, counts, n_slots, used, budget, scale)
    _check_steps(kv, rng, state, budget, 1, scale)


def _round(G):
    """(Sequence, KV head) pairs that fill a round of workgroups: two, three or four per CU."""
    return 512 if G > 4 else 768 if G > 2 else 1024


@pytest.mark.parametrize("D,dtype", [(64, BF16), (128, BF16), (64, F32), (128, F32)])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 8])
def test_one_workgroup_for_a_short_sequence(kv, G, D, dtype):  # noqa: F811
    """A round of (sequence, KV head) pairs, and a little less."""
    S = _round(G) // 8
    _run(kv, S, G, 8, D, dtype, 230, 840, G)
    _run(kv, S - S // 16, G, 8, D, dtype, 1031, 43, G + 1)


@pytest.mark.parametrize("G,D,dtype,over", [(1, 128, BF16, 0), (4, 128, BF16, 1), (2, 64, BF16, 1), (8, 64, BF16, 0),
                                            (3, 128, F32, 1), (4, 64, F32, 17)])
def test_one_workgroup_for_several_pieces(kv, G, D, dtype, over):  # noqa: F811
    """Prefill rows up to the end of a piece of four waves and past it, then the slots in a piece of their own."""
    piece = {128: 1152, 256: 1088, 512: 1056}[D * (2 if dtype == BF16 else 4)]
    _run(kv, _round(G) // 8, G, 8, D, dtype, piece + over, 65, 10 * G + over)


def test_as_many_slots_as_the_map_holds(kv):  # noqa: F811
    for n_slots in (1088, 1089):  # the second takes more than one workgroup
        _run(kv, 128, 1, 8, 128, BF16, 20, n_slots, n_slots)


@pytest.mark.parametrize("G,D,S", [(4, 128, 65), (3, 128, 80), (4, 64, 64), (4, 128, 136), (8, 64, 112)])
def test_rounds_that_are_not_full(kv, G, D, S):  # noqa: F811
    """Shares of a round from which one workgroup takes a sequence: with many slots, short rows, in a second round."""
    _run(kv, S, G, 8, D, BF16, 900, 257, S + G)


@pytest.mark.parametrize("G,S,cap", [(4, 128, 4000), (2, 192, 3100), (8, 128, 4200)])
def test_few_long_ranges(kv, G, S, cap):  # noqa: F811
    """Launches that would be over a round of workgroups in ranges of 1024 tokens take two or three longer ones."""
    _run(kv, S, G, 2, 64, BF16, cap, 150, S + G)
