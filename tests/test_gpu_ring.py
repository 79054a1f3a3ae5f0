"""The grouped GEMM with the LDS ring (few rows per expert, or fewer row tiles than compute units) against the oracle at
the edges of its tiles, and both builds of the library (counted waits / waits for all loads) bit for bit on every form
of it (test_dispatch_cpu.py checks that none is missing)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from helpers import MAX_ABS_TOL, ORC_DT, REL_L2_TOL, TORCH_DT, error_metrics, to_dev
from paper_2211_10017_amd import binding as B
from test_gpu_wait_guard import WAITALL, _ffn

pytestmark = pytest.mark.gpu


def _case(rows, d, F, bits, g, act, seed):
    rng = np.random.default_rng(seed)
    E, R = len(rows), int(sum(rows))
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    x = to_dev(rng.standard_normal((R, d)).astype(np.float32), TORCH_DT[act])
    w = [(rng.standard_normal((E, *s)) * 0.05).astype(np.float32) for s in ((d, F), (F, d))]
    packed = [B.moe_quantize_experts(to_dev(m, torch.float32), bits, g, want_canon=False)[1:] for m in w]
    return x, off, w, packed, E, R


# rows: 16-row blocks (at most ten per expert on average; experts of 16, 17 and 33 rows take one, two and three), 32-row
# blocks, 64-row blocks (few tiles).  d, F: one K step (the second K part is empty), odd numbers of steps, a last
# column block of one wavefront.
@pytest.mark.parametrize("rows", [[1], [16, 0, 17, 1, 2, 0, 33, 3, 5], [33, 32, 5, 0, 31], [64, 65, 1, 128]])
@pytest.mark.parametrize("d,F", [(64, 64), (64, 320), (192, 576), (704, 1216)])
@pytest.mark.parametrize("act,bits,g", [("f16", 4, 0), ("f16", 8, 0), ("f16", 4, 64), ("bf16", 8, 64), ("bf16", 4, 64), ("bf16", 4, 0)])
def test_ring_gemm_matches_oracle(rows, d, F, act, bits, g):
    print(f"ring rows={rows} d={d} F={F} {act} bits={bits} g={g}", flush=True)
    x, off, w, ((s1, p1), (s2, p2)), E, R = _case(rows, d, F, bits, g, act, sum(rows) + d + bits + g)
    y = B.moe_grouped_ffn_wq(x, to_dev(off, torch.int32), E, d, F, bits, g, p1, s1, p2, s2, y_dtype=torch.float32)
    torch.cuda.synchronize()
    (q1, o1), (q2, o2) = (oracle.quantize(m, bits, g) for m in w)
    want = oracle.grouped_ffn(x.float().cpu().numpy(), off, q1, o1, q2, o2, g, ORC_DT[act])
    max_abs, rel = error_metrics(y.cpu().numpy(), want)
    assert max_abs <= MAX_ABS_TOL and rel <= REL_L2_TOL


# 64-row tiles of 18 MB of 8-bit weights, one per compute unit at most: the longest ring, over odd and even numbers of K steps
@pytest.mark.parametrize("rows,d,F", [([70, 33, 64, 129, 5, 0, 96, 40], 1216, 1984), ([50] * 32, 320, 1792)])
@pytest.mark.parametrize("act,g", [("f16", 64), ("bf16", 64), ("bf16", 0), ("f16", 0)])
def test_long_rings_match_oracle_and_the_build_that_waits_for_all_loads(rows, d, F, act, g):
    test_ring_gemm_matches_oracle(rows, d, F, act, 8, g)
    test_counted_waits_equal_waiting_for_all_loads(rows, d, F, 8, g, act)


RING = [
    ([3, 9, 0, 17, 1], 1088, 704, 4, 0, "f16"), ([3, 9, 0, 17, 1], 1152, 1088, 8, 0, "f16"),            # ring, 16-row blocks
    ([3, 9, 0, 17, 1], 1152, 640, 4, 128, "f16"), ([3, 9, 0, 17, 1], 1152, 640, 4, 128, "bf16"),
    ([20, 40, 0, 33], 1088, 704, 4, 0, "f16"), ([20, 40, 0, 33], 1152, 640, 8, 128, "bf16"),            # 32-row blocks
    ([60, 70, 1, 64], 1088, 704, 4, 0, "f16"), ([60, 70, 1, 64], 1152, 640, 8, 128, "f16"),             # 64-row blocks
    ([20] * 40 + [0, 33], 192, 5120, 4, 0, "f16"), ([20] * 40 + [0, 33], 256, 5120, 8, 64, "f16"),      # fc2 alone (fc1 in register-fed tiles)
    ([60, 50, 33, 5] * 4, 256, 3072, 4, 64, "f16"), ([60, 50, 33, 5] * 4, 192, 3072, 8, 0, "bf16"),     # many 64-row blocks
    ([270, 257, 130, 20], 2112, 4416, 4, 0, "f16"), ([270, 257, 130, 20], 2176, 4480, 4, 64, "f16"),
    ([300, 290, 270], 2112, 5440, 8, 0, "f16"), ([270, 257, 130, 20], 2176, 4480, 4, 128, "bf16"),
    ([3, 9, 0, 17, 1], 1152, 640, 8, 128, "bf16"), ([20, 40, 0, 33], 1152, 640, 4, 128, "bf16"),        # the remaining forms of both scale modes
    ([20, 40, 0, 33], 1088, 704, 8, 0, "f16"), ([60, 70, 1, 64], 1152, 640, 8, 128, "bf16"),
    ([3, 9, 0, 17, 1], 1088, 704, 4, 0, "bf16"), ([3, 9, 0, 17, 1], 1152, 1088, 8, 0, "bf16"),          # bf16 rows and codes: 16-, 32- and 64-row blocks
    ([20, 40, 0, 33], 1088, 704, 4, 0, "bf16"), ([20, 40, 0, 33], 1152, 640, 8, 0, "bf16"),
    ([60, 70, 1, 64], 1088, 704, 4, 0, "bf16"), ([60, 50, 33, 5] * 4, 192, 3072, 8, 0, "f16")]


@pytest.mark.parametrize("rows,d,F,bits,g,act", RING)
def test_counted_waits_equal_waiting_for_all_loads(rows, d, F, bits, g, act):
    print(f"wait guard rows={rows} d={d} F={F} bits={bits} g={g} {act}", flush=True)
    x, off, _, ((s1, p1), (s2, p2)), E, R = _case(rows, d, F, bits, g, act, sum(rows) + d + bits)
    off = to_dev(off, torch.int32)
    plain, kernels = _ffn(B.load(), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, torch.float32)
    other, kernels2 = _ffn(ctypes.CDLL(WAITALL), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, torch.float32)
    assert kernels == kernels2 and kernels.split()[1] == "grouped_gemm_ring_kernel"
    assert torch.isfinite(plain).all() and torch.equal(plain, other)
