"""The decode kernel (one launch per slice of d_ff for sort, fc1, activation and fc2, and the slice reduction) through the sliced
call: every weight width, kind of scales and row type against the oracle, at the edges of its row passes, K parts, slabs and slices."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from helpers import MAX_ABS_TOL, ORC_DT, REL_L2_TOL, TORCH_DT, error_metrics, to_dev
from paper_2211_10017_amd import MoEExpertLayer
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


def _routing(loads, T, k, E, rng):
    """Expert of every assignment, distinct per token: uniform for -1, else the first expert takes that many tokens and no others."""
    first = min(max(loads, 0), T)
    idx = np.stack([rng.choice(E, size=k, replace=False) if loads < 0 else 1 + rng.choice(E - 1, size=k, replace=False) for _ in range(T)]).astype(np.int32)
    idx[:first, 0] = 0
    return idx


# sizes: one unit of K; fewer units than K parts; odd numbers of units and of slabs per wavefront; longer than the wavefronts' rings
@pytest.mark.parametrize("d,F", [(64, 64), (64, 320), (192, 1152), (768, 512), (1088, 1024), (2176, 640)])
@pytest.mark.parametrize("act,bits,g", [("f16", 4, 0), ("f16", 8, 0), ("f16", 4, 64), ("f16", 8, 64), ("bf16", 4, 0), ("bf16", 8, 0), ("bf16", 4, 64),
                                        ("bf16", 8, 64)])
@pytest.mark.parametrize("T,k,E,load", [(1, 1, 3, -1), (5, 2, 70, -1), (18, 2, 6, 17), (40, 2, 6, 33)])      # 17, 33 rows: one more than an item takes
def test_sliced_ffn_matches_oracle(d, F, act, bits, g, T, k, E, load):
    _check(d, F, act, bits, g, T, k, E, load)


# slices of 128, 256 and 512 channels, one and two sixteens of rows per pass
@pytest.mark.parametrize("d,F", [(192, 1024), (64, 2048), (128, 4096)])
@pytest.mark.parametrize("act,bits,g", [("f16", 4, 0), ("f16", 8, 0), ("f16", 4, 64), ("f16", 8, 64), ("bf16", 4, 0), ("bf16", 8, 0), ("bf16", 4, 64),
                                        ("bf16", 8, 64)])
@pytest.mark.parametrize("T", [60, 150])
def test_wide_slices_match_oracle(d, F, act, bits, g, T):
    assert B.moe_grouped_ffn_wq_sliced_workspace_bytes(T, 2, 34, d, F, bits, g, TORCH_DT[act]) == T * 2 * d * 4 * 8       # eight slices
    _check(d, F, act, bits, g, T, 2, 34, 20 if T == 60 else 45)


# groups of two and three units, one and two sixteens of rows per item
@pytest.mark.parametrize("d,F,g", [(256, 1152, 128), (384, 1152, 192), (1152, 384, 192)])
@pytest.mark.parametrize("act,bits", [("f16", 4), ("f16", 8), ("bf16", 4)])
@pytest.mark.parametrize("T,E", [(30, 12), (90, 12)])
def test_longer_groups_match_oracle(act, bits, d, F, g, T, E):
    _check(d, F, act, bits, g, T, 2, E, 20)


# the reduction by the number of slices: up to 8, up to 32, more
@pytest.mark.parametrize("d,F", [(64, 512), (320, 576), (1088, 2048), (64, 2112), (1024, 4096), (1088, 4160)])
@pytest.mark.parametrize("T,k", [(1, 2), (3, 1)])
def test_few_rows_over_few_and_many_slices_match_oracle(d, F, T, k):
    _check(d, F, "f16", 4, 0, T, k, 5, -1)


# ... of partial sums in units of bf16 codes
@pytest.mark.parametrize("d,F,bits", [(64, 512, 4), (320, 576, 8), (1088, 2048, 4), (64, 2112, 4), (1088, 4160, 8)])
def test_few_bf16_rows_over_few_and_many_slices_match_oracle(d, F, bits):
    _check(d, F, "bf16", bits, 0, 3, 2, 5, -1)


# experts with far more rows than one item takes, beside experts with few or none; more experts than lanes, with spans of 5 and 64 experts
@pytest.mark.parametrize("T,k,E,load", [(256, 2, 2, -1), (256, 2, 70, 200), (200, 1, 1, -1), (130, 2, 300, 90), (60, 2, 4096, 40)])
@pytest.mark.parametrize("act,bits,g", [("f16", 4, 0), ("f16", 8, 64), ("bf16", 4, 64)])
def test_rows_of_crowded_experts_match_oracle(act, bits, g, T, k, E, load):
    _check(64, 128 if E > 1000 else 1024, act, bits, g, T, k, E, load)


def _check(d, F, act, bits, g, T, k, E, load):
    print(f"sliced T={T} k={k} E={E} d={d} F={F} {act} bits={bits} g={g}", flush=True)
    rng = np.random.default_rng(d + F + bits + T)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), TORCH_DT[act])
    w = [(rng.standard_normal((E, *s)) * 0.05).astype(np.float32) for s in ((d, F), (F, d))]
    (s1, p1), (s2, p2) = (B.moe_quantize_experts(to_dev(m, torch.float32), bits, g, want_canon=False)[1:] for m in w)
    (q1, o1), (q2, o2) = (oracle.quantize(m, bits, g) for m in w)
    idx = _routing(load, T, k, E, rng)
    if T > 4:
        idx[T - 1] = E                                           # a pruned token, none of the loaded ones
    scale = rng.uniform(0.1, 1.0, (T, k)).astype(np.float32)
    ob1, ob2 = ((rng.standard_normal((E, n)) * 0.1).astype(np.float16).astype(np.float32) for n in (F, d))
    bias = T != 5
    b = [to_dev(v, torch.float16) if bias else None for v in (ob1, ob2)]
    gelu = T == 40
    perm_src, inv_perm, off = oracle.permute(idx, E)
    active = int(off[E])
    assert load < 0 or int(off[1]) == min(load, T - 1)
    y = np.zeros((T * k, d), dtype=np.float32)
    y[:active] = oracle.grouped_ffn(oracle.gather_rows(x.float().cpu().numpy(), perm_src[:active], k), off, q1, o1, q2, o2, g, ORC_DT[act],
                                    ob1 if bias else None, ob2 if bias else None, activation=int(gelu))
    want = oracle.combine(y, inv_perm, scale, T, k, active_rows=active)
    args = (x, to_dev(idx, torch.int32), to_dev(scale, torch.float32), E, d, F, bits, g, p1, s1, p2, s2, *b)
    out, ps, ip, of = B.moe_grouped_ffn_wq_sliced(*args, activation="gelu" if gelu else "relu")
    again = B.moe_grouped_ffn_wq_sliced(*args, activation="gelu" if gelu else "relu")[0]
    half = B.moe_grouped_ffn_wq_sliced(*args, activation="gelu" if gelu else "relu", out_dtype=torch.bfloat16)[0]
    torch.cuda.synchronize()
    assert np.array_equal(of.cpu().numpy(), off) and np.array_equal(ps.cpu().numpy(), perm_src) and np.array_equal(ip.cpu().numpy(), inv_perm)
    assert torch.equal(out, again) and torch.equal(half, out.to(torch.bfloat16))
    assert not out.cpu().numpy()[(idx == E).all(axis=1)].any()
    max_abs, rel = error_metrics(out.cpu().numpy(), want)
    assert max_abs <= MAX_ABS_TOL * max(1.0, float(np.abs(want).max()) / 8) and rel <= REL_L2_TOL, (max_abs, rel)


@pytest.mark.parametrize("bits,g", [(4, 0), (4, 128), (8, 0)])
def test_bf16_rows_far_outside_the_fp16_range(bits, g):
    """Rows of very different sizes, each compared relative to its own: the power-of-two factors of x and h."""
    T, E, d, F = 24, 8, 512, 1024
    rng = np.random.default_rng(bits + g)
    size = 2.0 ** rng.integers(-60, 60, (T, 1))
    small = np.where(rng.random((T, d)) < 0.2, 2.0 ** -20, 1.0)
    x = to_dev((rng.standard_normal((T, d)) * size * small).astype(np.float32), torch.bfloat16)
    w = [(rng.standard_normal((E, *s)) * 0.05).astype(np.float32) for s in ((d, F), (F, d))]
    (s1, p1), (s2, p2) = (B.moe_quantize_experts(to_dev(m, torch.float32), bits, g, want_canon=False)[1:] for m in w)
    (q1, o1), (q2, o2) = (oracle.quantize(m, bits, g) for m in w)
    idx = rng.integers(0, E, (T, 1)).astype(np.int32)
    perm_src, inv_perm, off = oracle.permute(idx, E)
    y = oracle.grouped_ffn(oracle.gather_rows(x.float().cpu().numpy(), perm_src, 1), off, q1, o1, q2, o2, g, oracle.BF16)
    one = np.ones((T, 1), dtype=np.float32)
    want = oracle.combine(y, inv_perm, one, T, 1).astype(np.float64)
    got = B.moe_grouped_ffn_wq_sliced(x, to_dev(idx, torch.int32), to_dev(one, torch.float32), E, d, F, bits, g, p1, s1, p2, s2)[0].cpu().numpy().astype(np.float64)
    rel = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
    assert np.isfinite(got).all() and rel.max() <= REL_L2_TOL, rel.max()


def test_sliced_layer_equals_its_steps_and_refuses_what_does_not_fit():
    lib, f = B.load(), ctypes.c_void_p(0x1000)
    ok = lambda *a: lib.moe_grouped_ffn_wq_sliced_workspace_bytes(*a)          # noqa: E731
    assert ok(256, 2, 4096, 64, 64, 4, 64, 1) and ok(1, 1, 1, 64, 64, 8, 0, 0)
    for bad in [(257, 2, 8, 64, 64, 4, 0, 0), (8, 3, 8, 64, 64, 4, 0, 0), (8, 1, 4097, 64, 64, 4, 0, 0), (8, 1, 8, 96, 64, 4, 0, 0), (8, 1, 8, 64, 32, 4, 0, 0),
                (8, 1, 8, 64, 64, 16, 0, 0), (8, 1, 8, 128, 64, 4, 128, 0), (8, 1, 8, 64, 64, 4, 0, 2), (0, 1, 8, 64, 64, 4, 0, 0)]:
        T, k, E, d, F, bits, g, act = bad
        assert not ok(*bad) and lib.moe_grouped_ffn_wq_sliced(f, act, f, f, T, k, E, d, F, bits, g, 0, f, f, None, f, f, None, f, 2, f, f, f, f, 1 << 30, None) == 2, bad
    assert lib.moe_grouped_ffn_wq_sliced(f, 0, f, f, 8, 1, 8, 64, 64, 4, 0, 0, f, f, None, f, f, None, f, 2, f, f, f, f, 16, None) == 3       # workspace
    rng = np.random.default_rng(1)
    a = MoEExpertLayer(9, 256, 512, 16, 2, 4, 128, act_dtype=torch.bfloat16)
    assert a.sliced
    for e in range(16):
        a.load_expert(1, e, to_dev((rng.standard_normal((256, 512)) * 0.05).astype(np.float32), torch.float32))
        a.load_expert(2, e, to_dev((rng.standard_normal((512, 256)) * 0.05).astype(np.float32), torch.float32))
    a.wg.copy_(to_dev(rng.standard_normal((256, 16)).astype(np.float32), torch.bfloat16))
    x = to_dev(rng.standard_normal((9, 256)).astype(np.float32), torch.bfloat16)
    whole = a.forward(x).clone()
    a.out.zero_()
    a.gate(x), a.permute(x), a.ffn(x)
    assert torch.equal(a.combine(x), whole)
    idx, out = a.expert_idx, B.moe_grouped_ffn_wq_sliced(x, a.expert_idx, a.expert_scale, 16, 256, 512, 4, 128, a.w1_packed, a.s1, a.w2_packed, a.s2)[0]
    torch.cuda.synchronize()
    assert torch.equal(out, whole) and int(idx.max()) < 16
