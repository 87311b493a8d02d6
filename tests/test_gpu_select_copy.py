"""GPU parity of selection and copies where one launch does both (few rows) and where two do: shares of rows that are
uneven, one row, none; more problems than workgroups; every row size; rows behind the retained ones stay as they were."""
import numpy as np
import pytest
import torch

from oracle import shotkv_oracle as orc
from test_gpu_prefill import _ragged_problem, kv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,Hkv,D,dtype,N,n,cap,mode", [
    (1, 8, 128, torch.bfloat16, 4300, 30, 4300, orc.SELECT_PREFIX),        # shares of 17 rows
    (1, 2, 64, torch.float32, 130, 3, 130, orc.SELECT_FIRST_FIT),
    (5, 3, 64, torch.bfloat16, 900, 200, 333, orc.SELECT_PREFIX),
    (7, 2, 128, torch.float32, 700, 40, 700, orc.SELECT_PREFIX),           # 36 workgroups each
    (256, 1, 64, torch.bfloat16, 300, 9, 300, orc.SELECT_FIRST_FIT),       # one workgroup each
    (257, 1, 64, torch.bfloat16, 300, 9, 300, orc.SELECT_PREFIX),          # two launches
    (3, 8, 128, torch.bfloat16, 2500, 50, 1953, orc.SELECT_PREFIX),        # 48 MB and a little less
    (3, 8, 128, torch.bfloat16, 2500, 50, 2049, orc.SELECT_PREFIX)])       # 48 MB exactly and a little more
def test_selection_with_its_copies(kv, P, Hkv, D, dtype, N, n, cap, mode):  # noqa: F811
    rng = np.random.default_rng(P * 1000 + cap)
    _, k, v, off = _ragged_problem(P, Hkv, Hkv, D, 8, N, dtype, P + cap, n, 3, 20)
    scores = np.round(rng.standard_normal((P, n)) * 4).astype(np.float32) / 4
    offs = off.cpu().numpy()
    always = offs[:, 0] + N - offs[:, -1]
    budgets = always + rng.integers(0, N, size=P)
    budgets[0] = always[0] + np.diff(offs[0]).min() - 1     # no shot fits
    if P > 2: budgets[1], budgets[2] = always[1] - 1, N     # nothing is kept; everything, if the capacity allows
    orig = torch.empty

    def filled(shape, **kw):    # what the binding allocates for the copied rows starts from a known value
        t = orig(shape, **kw)
        return t.fill_(7) if t.dim() == 4 else t
    torch.empty = filled
    try:
        res = kv.select_and_compact(torch.from_numpy(scores).cuda(), k, v, off, torch.from_numpy(budgets.astype(np.int32)).cuda(),
                                    cap, Hkv, 8, mode)
    finally:
        torch.empty = orig
    torch.cuda.synchronize()
    for p in range(P):
        b = min(int(budgets[p]), cap) - int(always[p])
        kept = int(res.kept_count[p])
        if b < 0:
            assert int(res.status[p]) == orc.STATUS_BUDGET_TOO_SMALL and kept == 0
        else:
            keep = orc.select_shots(scores[p], np.diff(offs[p]), b, mode)
            pos = orc.kept_positions_from_mask(keep, offs[p], N)
            assert int(res.status[p]) == orc.STATUS_OK and kept == pos.size
            assert res.shot_selected[p].cpu().numpy().tolist() == keep.tolist()
            np.testing.assert_array_equal(res.kept_positions[p, :kept].cpu().numpy(), pos)
            idx = torch.from_numpy(pos).long().cuda()
            assert torch.equal(res.k_out[p, :, :kept], k[p][:, idx]) and torch.equal(res.v_out[p, :, :kept], v[p][:, idx])
        assert bool((res.k_out[p, :, kept:] == 7).all()) and bool((res.v_out[p, :, kept:] == 7).all())
