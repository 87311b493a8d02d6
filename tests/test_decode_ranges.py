"""How a decode step is cut into token ranges, seen through the workspace it asks for.  Needs no GPU."""
import ctypes

import pytest
import torch

from paper_2502_01941_amd import shotkv

MAX_RANGE = 1024    # tokens whose logits a workgroup holds at a time


def _ranges(S, H, Hkv, D, dtype, cap, n_slots):
    """Token ranges per (sequence, KV head): the count whose partial sums give the workspace's size."""
    def aligned(x):
        return -(-x // 256) * 256
    cfg = shotkv._config(H, Hkv, D, 1, dtype, 1.0, shotkv.SELECT_PREFIX, shotkv.HEADS_PER_LAYER)
    have = shotkv.load_library().shotkv_decode_workspace_bytes(ctypes.byref(cfg), S, cap, n_slots)
    for n in range(1, 1025):
        if aligned(S * H * n * 8) + aligned(S * H * n * D * 4) + aligned(S * H * n_slots * 4) + aligned(S * 4) == have:
            return n
    raise AssertionError(have)


@pytest.mark.parametrize("G", range(1, 9))
@pytest.mark.parametrize("D,dtype", [(64, torch.bfloat16), (128, torch.bfloat16), (64, torch.float32), (128, torch.float32)])
def test_workgroups_are_resident_at_once(D, dtype, G):
    """256 compute units hold four workgroups each, or three for more than four query heads per KV head and rows of up
    to 256 bytes; no launch has more than that unless a sequence takes one range, or ranges reach their largest size."""
    row = D * (2 if dtype == torch.bfloat16 else 4)
    fit = 256 * (3 if G > 4 and row <= 256 else 4)
    for total in (900, 2000, 3000):
        least = -(-total // MAX_RANGE)
        for S in range(1, 560, 1 if G > 4 else 7):
            n = _ranges(S, 2 * G, 2, D, dtype, total - 100, 100)
            assert n >= least and (n == max(least, 1) or 2 * S * n <= fit), (S, total, n)


@pytest.mark.parametrize("S,H,Hkv,dtype,cap,n_slots", [
    (64, 64, 8, torch.bfloat16, 2, 253), (64, 64, 8, torch.float32, 3, 252), (51, 32, 4, torch.float32, 1, 638),
    (51, 32, 4, torch.bfloat16, 2, 637)])
def test_short_ranges_do_not_outgrow_the_static_scratch(S, H, Hkv, dtype, cap, n_slots):
    """Shapes whose partial sums fit the static scratch array with ranges of at least 128 tokens but would not with
    shorter ones: the step takes them without a workspace of its own."""
    n = _ranges(S, H, Hkv, 128, dtype, cap, n_slots)
    assert S * H * (n * 130 + n_slots) * 4 <= 8 << 20
