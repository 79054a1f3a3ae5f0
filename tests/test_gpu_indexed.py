"""Rows fetched through the routing index for every size and row type: the same bits as permuted copies give in the same tiles.  And the
conversion of bf16 rows at the lengths where its form changes."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from helpers import MAX_ABS_TOL, REL_L2_TOL, error_metrics, to_dev
from paper_2211_10017_amd import MoEExpertLayer
from paper_2211_10017_amd import binding as B
from test_gpu_ring import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,E,d,F,bits,g,act", [
    (1, 2, 4, 1024, 512, 4, 0, torch.bfloat16), (64, 2, 32, 1024, 1024, 4, 0, torch.bfloat16), (40, 1, 8, 512, 768, 8, 0, torch.bfloat16),
    (150, 2, 16, 768, 1536, 4, 128, torch.float16), (200, 2, 8, 1024, 2048, 8, 0, torch.float16), (700, 1, 4, 256, 4224, 4, 64, torch.bfloat16),
    (2000, 2, 8, 192, 2048, 8, 0, torch.bfloat16), (3000, 2, 8, 128, 256, 4, 0, torch.bfloat16)])      # the last: index in two launches
@pytest.mark.parametrize("prune", [False, True])
def test_indexed_layer_equals_permuted_copies(T, k, E, d, F, bits, g, act, prune):
    print(f"indexed T={T} k={k} E={E} d={d} F={F} bits={bits} g={g} {act} pruned={prune}", flush=True)
    rng = np.random.default_rng(T + E + bits)
    a = MoEExpertLayer(T, d, F, E, k, bits, g, act_dtype=act, y_dtype=torch.float32)
    assert a.routed
    wg = to_dev((rng.standard_normal((d, E)) * 0.05).astype(np.float32), act)
    a.wg.copy_(wg)
    for e in range(E):
        a.load_expert(1, e, to_dev((rng.standard_normal((d, F)) * 0.05).astype(np.float32), torch.float32))
        a.load_expert(2, e, to_dev((rng.standard_normal((F, d)) * 0.05).astype(np.float32), torch.float32))
    b = MoEExpertLayer(T, d, F, E, k, bits, g, act_dtype=act, y_dtype=torch.float32, fuse_routing=False)
    b.share_weights_from(a)
    b.wg.copy_(wg)
    span = 20 if act == torch.bfloat16 else 6           # rows of very different sizes; fp16 must hold 4 * 2^span and the h of such a row
    x = to_dev((rng.standard_normal((T, d)) * 2.0 ** rng.integers(-span, span, (T, 1))).astype(np.float32), act)
    fin = to_dev((rng.random(T) < 0.3).astype(np.uint8), torch.uint8) if prune else None
    out_a, out_b = a.forward(x, fin), b.forward(x, fin)
    torch.cuda.synchronize()
    assert torch.equal(a.expert_idx, b.expert_idx) and torch.equal(a.perm_src, b.perm_src)
    if T * k > E:
        assert torch.equal(out_a, out_b)
    else:           # the permuted call streams here when the rows are fp16 only, so both run row tiles
        assert act == torch.bfloat16 and torch.equal(out_a, out_b)


LENGTHS = [(1024, 2), (1088, 8), (4096, 8), (4160, 8), (16384, 8), (16448, 0)]       # two, eight 16-byte vectors per lane; a block per row; read twice


@pytest.mark.parametrize("g", [0, 64])          # as they are up to 4160; converted (test_dispatch_cpu.py: by which form)
@pytest.mark.parametrize("K", [K for K, _ in LENGTHS])
def test_bf16_rows_of_every_length(K, g):
    rows = [3, 6]
    x, off, w, ((s1, p1), (s2, p2)), E, R = _case(rows, 64, K, 8, g, "bf16", K)
    y = B.moe_grouped_ffn_wq(x, to_dev(off, torch.int32), E, 64, K, 8, g, p1, s1, p2, s2, y_dtype=torch.float32)
    torch.cuda.synchronize()
    (q1, o1), (q2, o2) = (oracle.quantize(m, 8, g) for m in w)
    want = oracle.grouped_ffn(x.float().cpu().numpy(), off, q1, o1, q2, o2, g, oracle.BF16)
    max_abs, rel = error_metrics(y.cpu().numpy(), want)
    assert max_abs <= MAX_ABS_TOL * max(1.0, float(np.abs(want).max()) / 8) and rel <= REL_L2_TOL


# (assignments, experts, k, d, F, bits[, g]) whose tiles a layer takes otherwise than permuted copies would, and the rows per block of fc1 and fc2
# (test_dispatch_cpu.py), negative in register-fed tiles
TAKEN = [((800, 8, 1, 64, 2112, 4), [-32, 32]), ((1318, 8, 2, 64, 2112, 4, 64), [-64, 32]), ((1280, 32, 2, 64, 1088, 8), [-32, 32]),
         ((640, 128, 1, 1024, 1088, 4), [-32, -32])]


@pytest.mark.parametrize("load", ["even", "one", "pruned"])
@pytest.mark.parametrize("sizes,tiles", TAKEN)
def test_tiles_of_indexed_rows_match_oracle(sizes, tiles, load):
    R, E, k, d, F, bits, g = (*sizes, 0)[:7]
    print(f"indexed tiles {sizes} {load}", flush=True)
    x, _, w, ((s1, p1), (s2, p2)), _, _ = _case([1] * E, d, F, bits, g, "f16", R)
    rng, T = np.random.default_rng(R), R // k
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), torch.float16)
    idx = np.stack([(np.arange(T) + j * 3) % (1 if load == "one" and j == 0 else E) for j in range(k)], 1).astype(np.int32)
    if load == "pruned":
        idx[rng.random(T) < 0.3] = E
    y, src, _, off = B.moe_grouped_ffn_wq_unsorted(x, to_dev(idx, torch.int32), E, d, F, bits, g, p1, s1, p2, s2, out_dtype=torch.float32)
    torch.cuda.synchronize()
    off, src = off.cpu().numpy(), src.cpu().numpy()
    (q1, o1), (q2, o2) = (oracle.quantize(m, bits, g) for m in w)
    rows = src[:off[E]] // k
    want = oracle.grouped_ffn(x.float().cpu().numpy()[rows], off, q1, o1, q2, o2, g, oracle.F16)
    max_abs, rel = error_metrics(y.cpu().numpy()[:off[E]], want)
    print(f"   max_abs={max_abs:.3e} rel_l2={rel:.3e}", flush=True)
    assert max_abs <= MAX_ABS_TOL * max(1.0, float(np.abs(want).max()) / 8) and rel <= REL_L2_TOL


# (assignments, experts, k, d, F, bits, g): bf16 rows whose two-term weights in register-fed tiles, 256 times code times scale, would be no FP16 numbers;
# fc1 in the ring instead (test_dispatch_cpu.py)
LARGE_WEIGHTS = [(800, 8, 1, 256, 2048, 4, 64), (800, 8, 1, 256, 2048, 4, 256), (892, 64, 2, 128, 3072, 4, 64), (705, 32, 1, 256, 3072, 8, 64), (705, 32, 1, 256, 3072, 8, 256)]


@pytest.mark.parametrize("sizes", LARGE_WEIGHTS)
def test_group_scaled_weights_up_to_a_thousand_match_oracle(sizes):
    R, E, k, d, F, bits, g = sizes
    print(f"large weights {sizes}", flush=True)
    rng, T = np.random.default_rng(R + g), R // k
    w = [(rng.standard_normal((E, *s)) * 0.05).astype(np.float32) for s in ((d, F), (F, d))]
    v = w[0].reshape(E, d // g, g, F)
    v *= 1000.0 / np.abs(v).max(axis=2, keepdims=True) * 2.0 ** -rng.integers(0, 12, (E, d // g, 1, F))       # a group's largest: 1000 down to 0.5
    (s1, p1), (s2, p2) = (B.moe_quantize_experts(to_dev(m, torch.float32), bits, g, want_canon=False)[1:] for m in w)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), torch.bfloat16)
    idx = np.stack([(np.arange(T) * 5 + j * 3) % E for j in range(k)], 1).astype(np.int32)
    y, src, _, off = B.moe_grouped_ffn_wq_unsorted(x, to_dev(idx, torch.int32), E, d, F, bits, g, p1, s1, p2, s2, out_dtype=torch.float32)
    torch.cuda.synchronize()
    (q1, o1), (q2, o2) = (oracle.quantize(m, bits, g) for m in w)
    want = oracle.grouped_ffn(x.float().cpu().numpy()[src.cpu().numpy() // k], off.cpu().numpy(), q1, o1, q2, o2, g, oracle.BF16)
    max_abs, rel = error_metrics(y.cpu().numpy(), want)
    print(f"   max_abs={max_abs:.3e} rel_l2={rel:.3e} of {np.abs(want).max():.3e}", flush=True)
    assert max_abs <= MAX_ABS_TOL * max(1.0, float(np.abs(want).max()) / 8) and rel <= REL_L2_TOL


def test_indexed_refuses_what_does_not_fit():
    f = ctypes.c_void_p(0x1000)
    call = B.load().moe_grouped_ffn_wq_indexed
    tail = (4, 0, 64, 64, 4, 0, 0, f, f, None, f, f, None, f, 0, f, 1 << 20, None)
    assert call(f, 0, None, 1, None, f, 8, *tail) == 1          # no index
    assert call(f, 0, f, 3, None, f, 9, *tail) == 1             # k = 3
    assert call(f, 0, f, 2, None, f, 9, *tail) == 1             # odd number of rows with two experts per token
    assert call(f, 0, f, 2, f, f, 8, *tail) == 1                # un-permute with two experts per token
