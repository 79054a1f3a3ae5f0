"""moe_combine in each form of its kernel (one, two, any number of experts per token) and type, with rows that do not fill a block, and pruned rows that hold
anything: the oracle's sums, whose terms are added in fp32 in the order of the slots."""
import numpy as np
import pytest
import torch

from helpers import to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu
F16, BF16, F32 = torch.float16, torch.bfloat16, torch.float32


@pytest.mark.parametrize("y_dt,out_dt", [(F16, F32), (F32, F32), (BF16, F16), (F16, BF16), (F32, BF16)])
@pytest.mark.parametrize("T,k,d", [(1, 1, 8), (1, 2, 8), (33, 1, 64), (257, 2, 72), (5, 3, 128), (129, 2, 1024)])
@pytest.mark.parametrize("prune", [False, True])
def test_combine_matches_fp32_sums_in_slot_order(T, k, d, y_dt, out_dt, prune):
    print(f"combine T={T} k={k} d={d} {y_dt} {out_dt} pruned={prune}", flush=True)
    rng = np.random.default_rng(T + k + d)
    R = T * k
    active = R * 2 // 3 if prune else R
    y = to_dev(rng.standard_normal((R, d)).astype(np.float32), y_dt)
    y[active:] = float("nan")
    inv = rng.permutation(R).astype(np.int32)
    scale = rng.random((T, k)).astype(np.float32)
    got = B.moe_combine(y, to_dev(inv, torch.int32), to_dev(scale, F32), T, k, out_dtype=out_dt, active_rows=to_dev(np.array([active], np.int32), torch.int32) if prune else None)
    torch.cuda.synchronize()
    v = y.double().cpu().numpy()
    want = np.zeros((T, d), np.float32)
    for j in range(k):                  # a fused multiply-add is the fp32 rounding of the sum in 64 bits: 24 + 24 bits of product, and no cancellation here exceeds the rest
        r = inv.reshape(T, k)[:, j]
        term = (want.astype(np.float64) + scale[:, j:j + 1].astype(np.float64) * v[r]).astype(np.float32)
        want = np.where((r < active)[:, None], term, want)
    assert torch.isfinite(got).all()
    want = torch.from_numpy(want).to(out_dt)
    ulp = {F32: 2.0 ** -23, F16: 2.0 ** -10, BF16: 2.0 ** -7}[out_dt]      # (the double rounding of the reference: at most one unit in the last place)
    assert bool(((got.cpu().float() - want.float()).abs() <= ulp * want.float().abs().clamp_min(2.0 ** -14)).all())
