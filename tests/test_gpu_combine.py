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


@pytest.mark.parametrize("T,k,d", [(1, 1, 8), (33, 1, 64), (257, 2, 72), (5, 3, 128), (129, 2, 1024)])
@pytest.mark.parametrize("y_dt", [F16, BF16, F32])
@pytest.mark.parametrize("share", [0.0, 0.6])
def test_rows_past_the_active_ones_need_not_be_there(T, k, d, y_dt, share):
    """y that holds the active rows only, and indices anywhere at or past them for the others."""
    print(f"combine, active rows only T={T} k={k} d={d} {y_dt} {share}", flush=True)
    rng = np.random.default_rng(T + k + d)
    R, active = T * k, int(share * T * k)
    y = to_dev(rng.standard_normal((max(active, 1), d)).astype(np.float32), y_dt)
    if not active:
        y.fill_(float("nan"))
    inv = rng.permutation(R).astype(np.int32)
    inv = np.where(inv < active, inv, rng.choice(np.array([active, R, 2 ** 20, 2 ** 31 - 1]), R)).astype(np.int32)
    scale = to_dev(rng.random((T, k)).astype(np.float32), F32)
    rows = to_dev(np.array([active], np.int32), torch.int32)
    got = B.moe_combine(y, to_dev(inv, torch.int32), scale, T, k, active_rows=rows)
    # the same rows where y has them all, and zeros where they are pruned
    full = torch.zeros((R, d), dtype=y_dt, device="cuda")
    full[:active] = y[:active]
    scale[to_dev(inv >= active, torch.bool).view(T, k)] = 0.0
    want = B.moe_combine(full, to_dev(np.minimum(inv, R - 1), torch.int32), scale, T, k)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and bool((got[to_dev((inv.reshape(T, k) >= active).all(1), torch.bool)] == 0).all())


@pytest.mark.parametrize("k", [1, 2])
def test_more_than_four_gigabytes_of_rows(k):
    """Beyond the reach of buffer loads: the bits of the same tokens a few at a time, pruned ones among them."""
    print(f"combine, 4 GiB and a bit, k={k}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(k)
    T, d = (1 << 20) // (8 * k) + 100, 8192
    R, active = T * k, T * k - 1000
    y = torch.randn((active, d), generator=gen, device="cuda")
    inv = torch.randperm(R, generator=gen, device="cuda").int()
    scale = torch.rand((T, k), generator=gen, device="cuda")
    rows = torch.tensor([active], dtype=torch.int32, device="cuda")
    assert R * d * 4 > 1 << 32
    got = B.moe_combine(y, inv, scale, T, k, active_rows=rows)
    for t in range(0, T, 8192):
        part = inv.view(T, k)[t:t + 8192]
        live = part < active
        few = y[part[live].long()]
        order = torch.full(part.shape, len(few), dtype=torch.int32, device="cuda")
        order[live] = torch.arange(len(few), dtype=torch.int32, device="cuda")
        want = B.moe_combine(few, order.view(-1), scale[t:t + 8192].contiguous(), len(part), k, active_rows=torch.tensor([len(few)], dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        assert torch.equal(got[t:t + 8192], want), t


@pytest.mark.parametrize("T,k,d", [(33, 1, 64), (257, 2, 72), (6, 3, 128)])
@pytest.mark.parametrize("y_dt", [F16, F32])
@pytest.mark.parametrize("prune", [False, True])
def test_a_few_tokens_of_a_batch_reach_all_of_its_rows(T, k, d, y_dt, prune):
    """A call for some of the tokens, whose rows lie anywhere in the batch's y: the bits of the call for all of them."""
    print(f"combine, part of the tokens T={T} k={k} d={d} {y_dt} pruned={prune}", flush=True)
    rng = np.random.default_rng(T + k + d)
    R = T * k
    y = to_dev(rng.standard_normal((R, d)).astype(np.float32), y_dt)
    inv = to_dev(rng.permutation(R).astype(np.int32), torch.int32)
    scale = to_dev(rng.random((T, k)).astype(np.float32), F32)
    rows = to_dev(np.array([R * 2 // 3], np.int32), torch.int32) if prune else None
    want = B.moe_combine(y, inv, scale, T, k, active_rows=rows)
    for t in range(0, T, 5):
        n = min(5, T - t)
        got = B.moe_combine(y, inv[t * k:(t + n) * k].contiguous(), scale[t:t + n].contiguous(), n, k, active_rows=rows)
        torch.cuda.synchronize()
        assert torch.equal(got, want[t:t + n]) and (prune or bool((got != 0).any(1).all()))
