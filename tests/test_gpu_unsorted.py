"""Row tiles that sort for themselves: the bits of moe_permute and the indexed call, whatever the routing."""
import ctypes

import pytest
import torch

from paper_2211_10017_amd import binding as B

pytestmark = pytest.mark.gpu


def _weights(gen, E, K, N, bits, g):
    w = torch.randn((E, K, N), generator=gen, device="cuda") * 0.05
    _, s, p = B.moe_quantize_experts(w, bits, g, want_canon=False)
    return s, p


# assignments at the edges of the sort's steps (256 each) and of its range, experts at those of a wavefront, of the block's threads and of the range; row
# tiles of every kernel: rings of 16, 32 and 64 rows, register-fed tiles, converted and unconverted bf16 rows
SIZES = [(1, 1, 1, 64, 64, 4, 0, "f16"), (128, 2, 64, 128, 192, 4, 0, "f16"), (257, 1, 65, 64, 128, 8, 0, "bf16"), (256, 1, 8, 128, 320, 8, 0, "f16"),
         (511, 2, 255, 64, 64, 4, 64, "f16"), (300, 2, 5, 128, 256, 4, 128, "bf16"), (1023, 1, 2, 192, 64, 4, 0, "bf16"), (2048, 2, 16, 64, 128, 4, 0, "f16"),
         (4095, 1, 1024, 64, 64, 8, 0, "f16"), (4096, 1, 3, 128, 128, 8, 64, "bf16"), (700, 2, 4, 64, 2112, 8, 64, "f16"), (4096, 1, 7, 2176, 64, 4, 0, "f16")]


@pytest.mark.parametrize("routing", ["even", "one", "pruned", "all pruned", "out of range"])
@pytest.mark.parametrize("T,k,E,d,F,bits,g,act", SIZES)
def test_unsorted_call_equals_permute_and_the_indexed_call(T, k, E, d, F, bits, g, act, routing):
    print(f"unsorted T={T} k={k} E={E} d={d} F={F} bits={bits} g={g} {act} {routing}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + E)
    dt = {"f16": torch.float16, "bf16": torch.bfloat16}[act]
    (s1, p1), (s2, p2) = _weights(gen, E, d, F, bits, g), _weights(gen, E, F, d, bits, g)
    x = torch.randn((T, d), generator=gen, device="cuda").to(dt)
    idx = torch.randint(0, E, (T, k), generator=gen, device="cuda", dtype=torch.int32)
    if routing == "one":
        idx.fill_(E - 1)
    elif routing == "pruned":
        idx[torch.rand(T, generator=gen, device="cuda") < 0.4] = E
    elif routing == "all pruned":
        idx.fill_(E)
    elif routing == "out of range":
        idx[::3] = -5
        idx[1::3] = E + 9
    scale = torch.rand((T, k), generator=gen, device="cuda") if k == 1 else None
    y, src, inv, off = B.moe_grouped_ffn_wq_unsorted(x, idx, E, d, F, bits, g, p1, s1, p2, s2, expert_scale=scale, out_dtype=torch.float32)
    want_src, want_inv, want_off = (torch.empty_like(t) for t in (src, inv, off))
    ws = torch.empty(max(16, B.moe_permute_workspace_bytes(T, k, E)), dtype=torch.uint8, device="cuda")
    lib, ptr = B.load(), lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())  # noqa: E731
    stream = ctypes.c_void_p(B.current_stream_handle())
    assert lib.moe_permute(ptr(idx), None, B._DT[dt], T, k, E, d, None, ptr(want_src), ptr(want_inv), ptr(want_off), ptr(ws), ws.numel(), stream) == 0
    want = torch.empty_like(y)
    ws = torch.empty(B.moe_grouped_ffn_wq_workspace_bytes(T * k, d, F, E, dt), dtype=torch.uint8, device="cuda")
    assert lib.moe_grouped_ffn_wq_indexed(ptr(x), B._DT[dt], ptr(want_src), k, ptr(scale), ptr(want_off), T * k, E, T, d, F, bits, g, 0, ptr(p1), ptr(s1), None,
                                          ptr(p2), ptr(s2), None, ptr(want), B.MOE_F32, ptr(ws), ws.numel(), stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(src, want_src) and torch.equal(inv, want_inv) and torch.equal(off, want_off)
    active = int(off[E])
    rows = src[:active].long() if k == 1 else slice(0, active)          # what is written: the active tokens' rows, or the active sorted rows
    assert torch.equal(y[rows], want[rows]) and bool(torch.isfinite(y[rows]).all())


@pytest.mark.parametrize("T,k,E,d,F,bits", [(40, 1, 8, 512, 2112, 8), (1, 1, 3, 1024, 2112, 4), (256, 1, 16, 1024, 1088, 4), (100, 2, 12, 512, 2112, 8), (37, 2, 40, 2048, 1088, 4)])
@pytest.mark.parametrize("prune", [False, True])
def test_unsorted_call_that_streams_fc1_equals_the_gated_call(T, k, E, d, F, bits, prune):
    """Where the gated call runs fc1 in the streaming kernel and fc2 in row tiles: its bits, and with the un-permute those times the gate's scale."""
    print(f"unsorted, streaming T={T} k={k} E={E} d={d} F={F} bits={bits} pruned={prune}", flush=True)
    assert B.moe_grouped_ffn_wq_gated_supported(T, k, E, d, F, bits, 0, torch.float16) == 1 and B.moe_grouped_ffn_wq_gated_pays(T, k, E, d, F, bits, 0, torch.float16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + E)
    (s1, p1), (s2, p2) = _weights(gen, E, d, F, bits, 0), _weights(gen, E, F, d, bits, 0)
    x = torch.randn((T, d), generator=gen, device="cuda").half()
    idx = torch.randint(0, E, (T, k), generator=gen, device="cuda", dtype=torch.int32)
    if prune:
        idx[torch.rand(T, generator=gen, device="cuda") < 0.4] = E
    want = B.moe_grouped_ffn_wq_gated(x, idx, E, d, F, bits, 0, p1, s1, p2, s2, y_dtype=torch.float32)
    assert B.load().moe_last_ffn_kernels().decode().startswith("stream_unrolled_kernel grouped_gemm")
    got = B.moe_grouped_ffn_wq_unsorted(x, idx, E, d, F, bits, 0, p1, s1, p2, s2, out_dtype=torch.float32)
    assert B.load().moe_last_ffn_kernels().decode().startswith("stream_unrolled_kernel grouped_gemm")
    active = int(want[3][E])
    assert all(torch.equal(a, b) for a, b in zip(got[1:], want[1:])) and torch.equal(got[0][:active], want[0][:active])
    if k == 1:
        scale = torch.rand((T, 1), generator=gen, device="cuda")
        out = B.moe_grouped_ffn_wq_unsorted(x, idx, E, d, F, bits, 0, p1, s1, p2, s2, expert_scale=scale, out_dtype=torch.float32)[0]
        rows = want[1][:active].long()
        assert torch.equal(out[rows], want[0][:active] * scale[rows])
