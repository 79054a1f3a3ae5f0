"""Group scales in the row-tile kernels: a wavefront takes code times scale in one fused operation as long as its channels' scales stay
within a window around their first, and goes on in the general loop from the first that does not."""
import ctypes

import numpy as np
import pytest
import torch

from helpers import to_dev
from paper_2211_10017_amd import binding as B
from test_gpu_wait_guard import WAITALL, _ffn

pytestmark = pytest.mark.gpu


def _masters(gen, E, K, N, g):
    """Slabs of 64 channels: scales alike; scales up to 4 times apart; one later group 256 times as large; one group of zeros (in every
    other such slab the first, then with further ones 64 times smaller)."""
    w = torch.randn((E, K // g, g, N), generator=gen, device="cuda") * 0.05
    G, slabs = K // g, N // 64
    for s in range(slabs):
        v = w[..., 64 * s:64 * s + 64]
        if s % 4 == 1:
            v *= torch.exp2(torch.rand((E, G, 1, 64), generator=gen, device="cuda") * 2 - 1)
        elif s % 4 == 2:
            v[:, 1 + s % (G - 1), :, 7] *= 256.0
        elif s % 4 == 3:
            v[:, 0 if s % 8 == 3 else G - 1, :, 50] = 0.0
            if s % 8 == 3:
                v[:, G // 2, :, 3] /= 64.0
    return w.reshape(E, K, N)


def _dequantised(canon, scales, bits, g):
    q = canon.to(torch.int32)
    if bits == 4:
        q = torch.stack([(q << 28) >> 28, (q << 24) >> 28], dim=-1).reshape(*q.shape[:2], -1)
    return (q.half() * scales.repeat_interleave(g, dim=1)).double()          # (rounded once, as the kernels take it)


# 32-, 64- and 128-row tiles (8-bit codes: general loop only); odd and even numbers of K steps; one and two K steps per group
@pytest.mark.parametrize("E,rows,d,g", [(256, (20, 40), 512, 64), (64, (70, 130), 512, 128), (64, (33, 150), 576, 64), (8, (280, 330), 2112, 64),
                                        (8, (290, 390), 2176, 128)])
@pytest.mark.parametrize("bits", [4, 8])
def test_scales_in_and_out_of_the_window(E, rows, d, g, bits):
    print(f"scale window E={E} rows={rows} d={d} g={g} bits={bits}", flush=True)
    rng = np.random.default_rng(E + d + g + bits)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(E + d + bits)
    off = np.concatenate([[0], np.cumsum(rng.integers(*rows, E))]).astype(np.int32)
    x = torch.randn((int(off[-1]), d), generator=gen, device="cuda").half()
    c1, s1, p1 = B.moe_quantize_experts(_masters(gen, E, d, d, g), bits, g)
    eye = torch.eye(d, device="cuda").expand(E, d, d).contiguous()           # fc2: one product per output, groups of zeros but one
    c2, s2, p2 = B.moe_quantize_experts(eye, bits, g)
    y = B.moe_grouped_ffn_wq(x, to_dev(off, torch.int32), E, d, d, bits, g, p1, s1, p2, s2, y_dtype=torch.float32)
    torch.cuda.synchronize()
    assert B.load().moe_last_ffn_kernels().decode().split() == ["grouped_gemm_kernel"] * 2
    for e in range(E):
        lo, hi = int(off[e]), int(off[e + 1])
        w1 = _dequantised(c1[e:e + 1], s1[e:e + 1], bits, g)[0]
        diag = _dequantised(c2[e:e + 1], s2[e:e + 1], bits, g)[0].diagonal()
        want = (x[lo:hi].double() @ w1).clamp(min=0).half().double() * diag
        # h may round the other way where the fp32 sum is off: an FP16 unit in the last place, 2^-10, in every element at most.  A wrong
        # scale of one group of K / g is off by more than that in a channel by itself.
        err = (y[lo:hi].double() - want).norm(dim=0)
        assert (err <= 2.0 ** -10 * want.norm(dim=0) + 1e-12).all(), (e, int((err / (want.norm(dim=0) + 1e-12)).argmax()))


@pytest.mark.parametrize("E,rows,d,g", [(256, (20, 40), 512, 64), (64, (70, 130), 512, 128), (64, (33, 150), 576, 64), (8, (280, 330), 2112, 64),
                                        (8, (290, 390), 2176, 128)])
def test_counted_waits_where_wavefronts_leave_the_window(E, rows, d, g):
    """The general loop entered in the middle of K, by some of a block's wavefronts: both builds of the library (counted waits / waits for all loads) bit for bit."""
    print(f"scale window, wait guard E={E} rows={rows} d={d} g={g}", flush=True)
    rng = np.random.default_rng(E + d + g)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(E + d)
    off = np.concatenate([[0], np.cumsum(rng.integers(*rows, E))]).astype(np.int32)
    R = int(off[-1])
    x = torch.randn((R, d), generator=gen, device="cuda").half()
    (s1, p1), (s2, p2) = (B.moe_quantize_experts(_masters(gen, E, d, d, g), 4, g, want_canon=False)[1:] for _ in range(2))
    off = to_dev(off, torch.int32)
    plain, kernels = _ffn(B.load(), x, off, R, E, d, d, 4, g, p1, s1, p2, s2, torch.float32)
    other, kernels2 = _ffn(ctypes.CDLL(WAITALL), x, off, R, E, d, d, 4, g, p1, s1, p2, s2, torch.float32)
    assert kernels == kernels2 == "grouped_gemm_kernel grouped_gemm_kernel"
    assert torch.isfinite(plain).all() and torch.equal(plain, other)
