"""The grouped GEMMs with row tiles send their activation rows (fp16, bf16, or bf16 converted to scaled fp16 beforehand), and the kernel with the LDS ring
its weights as well, from global memory straight into LDS and wait for them with a hand-counted `s_waitcnt vmcnt(n)`, n = the loads issued after them.  The library is
built a second time (libmoe_wq_waitall.so) with every such wait replaced by a wait for ALL loads, which
needs no counting.  If a compiler change ever merged, split or reordered one of the counted loads, the
normal build would read stale rows; these tests run every direct-to-LDS variant of both kernels in both
builds and compare the outputs bit for bit.  test_dispatch_cpu.py checks that no variant is missing."""
import ctypes
import os

import numpy as np
import pytest
import torch

from helpers import to_dev
from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu
WAITALL = os.path.join(os.path.dirname(B.LIB_PATH), "libmoe_wq_waitall.so")


def _ffn(lib, x, off, R, E, d, F, bits, g, p1, s1, p2, s2, y_dtype):
    vp, i, sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
    lib.moe_grouped_ffn_wq.restype = i
    lib.moe_grouped_ffn_wq.argtypes = [vp, i, vp, i, i, i, i, i, i, i, i, vp, vp, vp, vp, vp, vp, vp, i, vp, sz, vp]
    lib.moe_last_ffn_kernels.restype = ctypes.c_char_p
    y = torch.full((R, d), float("nan"), dtype=y_dtype, device=x.device)
    ws = torch.empty(B.moe_grouped_ffn_wq_workspace_bytes(R, d, F, E, x.dtype), dtype=torch.uint8, device=x.device)
    rc = lib.moe_grouped_ffn_wq(x.data_ptr(), B._DT[x.dtype], off.data_ptr(), R, E, 0, d, F, bits, g, 0, p1.data_ptr(), s1.data_ptr(), None,
                                p2.data_ptr(), s2.data_ptr(), None, y.data_ptr(), B._DT[y_dtype], ws.data_ptr(), ws.numel(),
                                torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    return y, lib.moe_last_ffn_kernels().decode()


@pytest.mark.parametrize("rows,d,F,bits,g,y_dt,x_dt", [(*c, torch.float16) for c in [
    ([20, 31, 5, 0, 17], 192, 256, 4, 0, torch.float16),            # the ring's 32-row blocks; 3 and 4 K steps (odd, even)
    ([20, 31, 5, 0, 17], 192, 256, 8, 64, torch.float32),
    ([60, 50, 33, 5], 192, 320, 4, 64, torch.float32),              # its 64-row blocks, last blocks with one live row tile; 3 and 5 K steps
    ([60, 50, 33, 5], 256, 128, 8, 0, torch.float16),               # 4 and 2 K steps
    ([270, 257, 130, 20], 2112, 2176, 4, 0, torch.float16),         # several blocks per expert; 33 and 34 K steps
    ([270, 257, 130, 20], 2112, 2176, 4, 64, torch.float32),        # ... with a scale per group
    ([300, 290, 270], 2112, 2112, 8, 0, torch.float16),
    ([300, 290, 270], 2112, 2112, 8, 64, torch.float32)]] + [
    # bf16 rows: fc1 keeps the group scales out of the weights (exact codes, group sums folded in fp32)
    ([20, 31, 5, 0, 17], 256, 384, 4, 128, torch.float32, torch.bfloat16),
    ([60, 50, 33, 5], 384, 256, 8, 128, torch.float32, torch.bfloat16),
    ([270, 257, 130, 20], 2176, 2304, 4, 128, torch.float32, torch.bfloat16),
    ([60, 50, 33, 5], 192, 320, 4, 64, torch.float32, torch.bfloat16),
    ([270, 257, 130, 20], 2112, 2176, 8, 64, torch.float32, torch.bfloat16)])
def test_counted_waits_equal_waiting_for_all_loads(rows, d, F, bits, g, y_dt, x_dt):
    print(f"wait guard rows={rows} d={d} F={F} bits={bits} g={g} y={y_dt} x={x_dt}", flush=True)
    assert os.path.exists(WAITALL), "libmoe_wq_waitall.so is built by paper_2211_10017_amd.build together with the library"
    rng = np.random.default_rng(sum(rows) + d + bits + g)
    E = len(rows)
    off = to_dev(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32), torch.int32)
    R = int(sum(rows))
    x = to_dev(rng.standard_normal((R, d)).astype(np.float32), x_dt)
    w1 = to_dev((rng.standard_normal((E, d, F)) * 0.05).astype(np.float32), torch.float32)
    w2 = to_dev((rng.standard_normal((E, F, d)) * 0.05).astype(np.float32), torch.float32)
    _, s1, p1 = B.moe_quantize_experts(w1, bits, g, want_canon=False)
    _, s2, p2 = B.moe_quantize_experts(w2, bits, g, want_canon=False)
    plain, kernels = _ffn(B.load(), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, y_dt)
    other, kernels2 = _ffn(ctypes.CDLL(WAITALL), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, y_dt)
    assert kernels == kernels2 == "grouped_gemm_ring_kernel grouped_gemm_ring_kernel"
    assert torch.isfinite(plain.float()).all()
    assert torch.equal(plain, other)


# Register-fed tiles: launches of so many tiles that none of them goes to the ring.  (rows, d, F, bits, g, x, the kernel of fc1); K = d, so
# d / 64 steps.  Experts without rows, tiles with one live row tile, odd and even numbers of steps, a last column block that is
# partly there.
_T32, _T64, _T128 = [20] * 40 + [0, 33], [60, 50, 33, 5] * 4, [270, 257, 130, 20]
_F16, _BF16 = torch.float16, torch.bfloat16
REGISTER_FED = [
    (_T32, 192, 2752, 4, 0, _F16, "grouped_gemm_kernel<4, 0, 1>"), (_T32, 256, 2752, 8, 0, _F16, "grouped_gemm_kernel<8, 0, 1>"),
    (_T32, 256, 2816, 4, 128, _F16, "grouped_gemm_kernel<4, 1, 1>"), (_T32, 192, 2688, 8, 64, _F16, "grouped_gemm_kernel<8, 1, 1>"),
    (_T32, 192, 2688, 4, 64, _BF16, "grouped_gemm_kernel<4, 2, 1>"), (_T32, 256, 2688, 8, 64, _BF16, "grouped_gemm_kernel<8, 2, 1>"),
    (_T32, 384, 2816, 4, 128, _BF16, "grouped_gemm_kernel<4, 3, 1>"), (_T32, 256, 2816, 8, 128, _BF16, "grouped_gemm_kernel<8, 3, 1>"),
    (_T64, 256, 3392, 4, 0, _F16, "grouped_gemm_kernel<4, 0, 2>"), (_T64, 192, 3392, 8, 0, _F16, "grouped_gemm_kernel<8, 0, 2>"),
    (_T64, 192, 3392, 4, 64, _F16, "grouped_gemm_kernel<4, 1, 2>"), (_T64, 256, 3456, 8, 128, _F16, "grouped_gemm_kernel<8, 1, 2>"),
    (_T64, 256, 3392, 4, 64, _BF16, "grouped_gemm_kernel<4, 2, 2>"), (_T64, 192, 3392, 8, 64, _BF16, "grouped_gemm_kernel<8, 2, 2>"),
    (_T64, 256, 3456, 4, 128, _BF16, "grouped_gemm_kernel<4, 3, 2>"), (_T64, 384, 3456, 8, 128, _BF16, "grouped_gemm_kernel<8, 3, 2>"),
    (_T128, 2112, 4736, 4, 0, _F16, "grouped_gemm_kernel<4, 0, 4>"), ([300, 290, 270], 2176, 4224, 8, 0, _F16, "grouped_gemm_kernel<8, 0, 4>"),
    (_T128, 2176, 4736, 4, 64, _F16, "grouped_gemm_kernel<4, 1, 4>"), ([300, 290, 270], 2112, 4224, 8, 64, _F16, "grouped_gemm_kernel<8, 1, 4>"),
    (_T128, 2112, 4736, 4, 64, _BF16, "grouped_gemm_kernel<4, 2, 4>"), ([300, 290, 270], 2176, 4224, 8, 64, _BF16, "grouped_gemm_kernel<8, 2, 4>"),
    (_T128, 2176, 4864, 4, 128, _BF16, "grouped_gemm_kernel<4, 3, 2>"),                     # group sums stay on 64-row tiles
    # bf16 rows and codes
    (_T32, 192, 2752, 4, 0, _BF16, "grouped_gemm_kernel<4, 4, 1>"), (_T32, 256, 2752, 8, 0, _BF16, "grouped_gemm_kernel<8, 4, 1>"),
    (_T64, 256, 3392, 4, 0, _BF16, "grouped_gemm_kernel<4, 4, 2>"), (_T64, 192, 3392, 8, 0, _BF16, "grouped_gemm_kernel<8, 4, 2>"),
    (_T128, 2112, 4736, 4, 0, _BF16, "grouped_gemm_kernel<4, 4, 4>"), ([300, 290, 270], 2176, 4224, 8, 0, _BF16, "grouped_gemm_kernel<8, 4, 4>")]


@pytest.mark.parametrize("rows,d,F,bits,g,x_dt,fc1", REGISTER_FED)
def test_counted_waits_of_register_fed_tiles(rows, d, F, bits, g, x_dt, fc1):
    print(f"wait guard, {fc1}: rows={rows} d={d} F={F} bits={bits} g={g} x={x_dt}", flush=True)
    E, R = len(rows), sum(rows)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(R + d + F + bits)
    off = to_dev(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32), torch.int32)
    x = torch.randn((R, d), generator=gen, device="cuda:0").to(x_dt)
    packed = [B.moe_quantize_experts(torch.randn((E, *s), generator=gen, device="cuda:0") * 0.05, bits, g, want_canon=False)[1:] for s in ((d, F), (F, d))]
    (s1, p1), (s2, p2) = packed
    plain, kernels = _ffn(B.load(), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, torch.float32)
    other, kernels2 = _ffn(ctypes.CDLL(WAITALL), x, off, R, E, d, F, bits, g, p1, s1, p2, s2, torch.float32)
    assert kernels == kernels2 and kernels.split()[0] == "grouped_gemm_kernel"
    assert torch.isfinite(plain).all() and torch.equal(plain, other)
