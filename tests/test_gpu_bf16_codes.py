"""bf16 rows of channel-scaled layers that meet bf16 codes as they are: every kernel with row tiles against the oracle."""
import numpy as np
import pytest
import torch

import launches as L
from helpers import REL_L2_TOL, to_dev
from paper_2211_10017_amd import binding as B

# rows per expert, d, F, bits: 16-, 32- and 64-row blocks of the ring, the long ring, register-fed tiles of 32, 64 and 128 rows; partly filled tiles
# and last column blocks, odd numbers of K steps
CASES = [([16, 0, 17, 1, 2, 0, 33, 3, 5], 192, 576, 8), ([33, 32, 5, 0, 31], 704, 1216, 8), ([64, 65, 1, 128], 704, 1216, 8), ([50] * 32, 320, 1792, 8),
         ([20] * 40 + [0, 33], 192, 2688, 4), ([20] * 40 + [0, 33], 192, 5120, 8), ([60, 50, 33, 5] * 4, 192, 3392, 4), ([60, 50, 33, 5] * 4, 256, 3456, 8),
         ([270, 257, 130, 20], 2176, 4736, 4), ([300, 290, 270], 2112, 4224, 8), ([3, 9, 0, 17, 1], 1088, 704, 4), ([20, 40, 0, 33], 1088, 704, 4), ([60, 70, 1, 64], 1088, 704, 4)]


def test_cases_reach_every_kernel_without_a_conversion():
    ran = [[p.kernel for p in c.launches] for c in L.record([L.ffn(sum(r), len(r), d, F, bits, 0, B.MOE_BF16) for r, d, F, bits in CASES])]
    assert not any(k.startswith("rows_to_f16") for c in ran for k in c)
    built = {f"grouped_gemm_kernel<{b}, 4, {tm}>" for b in (4, 8) for tm in (1, 2, 4)} | {f"grouped_gemm_ring_kernel<{b}, 4, {bm}>" for b in (4, 8) for bm in (16, 32, 64)}
    built |= {"grouped_gemm_ring_long_kernel<8, 4, 64>"}
    assert built <= {k for c in ran for k in c}, built - {k for c in ran for k in c}


def test_conversion_where_matrix_work_is_the_larger_part():
    """Sizes on both sides of the rule."""
    sizes = [((1400, 32, 1024, 4096, 8), True), ((10000, 128, 1024, 4096, 4), True), ((8192, 16, 2048, 8192, 4), True), ((2000, 32, 2048, 8192, 8), True),
             ((2000, 32, 2048, 8192, 4), False), ((8192, 128, 2048, 8192, 8), True), ((4000, 16, 4096, 16384, 8), False), ((16384, 64, 4096, 16384, 4), False)]
    for (s, want), c in zip(sizes, L.record([L.ffn(*s, 0, B.MOE_BF16) for s, _ in sizes])):
        assert want != any(p.kernel.startswith("rows_to_f16") for p in c.launches), s
    assert any(p.kernel.startswith("rows_to_f16") for p in L.record([L.ffn(100, 8, 256, 512, 4, 64, B.MOE_BF16)])[0].launches)       # group scales always


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d,F,bits", CASES)
def test_bf16_codes_match_oracle(rows, d, F, bits):
    from test_gpu_ring import test_ring_gemm_matches_oracle as check
    check(rows, d, F, "bf16", bits, 0)


# Rows, d, F, bits of channel-scaled layers on the other side of the rule: FP16 kernels with a factor per row
CONVERTED = [([5, 1] * 8, 2048, 8192, 4), ([200, 130, 160, 70], 2048, 8192, 4), ([300, 220], 4096, 8192, 4), ([300, 270, 255, 215], 4096, 8192, 8), ([5, 1], 4096, 16384, 4),
             ([17, 7], 4096, 16384, 4), ([300, 220], 4096, 4096, 4)]


def test_converted_cases_are_converted():
    calls = L.record([L.ffn(sum(r), len(r), d, F, bits, 0, B.MOE_BF16) for r, d, F, bits in CONVERTED])
    assert all([p.kernel[:11] for p in c.launches][::2] == ["rows_to_f16"] * 2 for c in calls)
    ran = {p.kernel for c in calls for p in c.launches[1::2]}
    assert ran == {f"grouped_gemm_kernel<4, 0, {tm}>" for tm in (1, 2, 4)} | {"grouped_gemm_kernel<8, 0, 4>"} | {f"grouped_gemm_ring_kernel<4, 0, {bm}>" for bm in (16, 32, 64)}


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d,F,bits", CONVERTED)
def test_converted_rows_match_64_bits(rows, d, F, bits):
    print(f"converted bf16 rows={rows[:4]} d={d} F={F} bits={bits}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + F + bits)
    E, R = len(rows), sum(rows)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    quantised = [B.moe_quantize_experts(torch.randn((E, *s), generator=gen, device="cuda") * 0.05, bits, 0) for s in ((d, F), (F, d))]
    size = torch.exp2(torch.randint(-60, 60, (R, 1), generator=gen, device="cuda").float())
    x = (torch.randn((R, d), generator=gen, device="cuda") * size).bfloat16()
    (_, s1, p1), (_, s2, p2) = quantised
    y = B.moe_grouped_ffn_wq(x, to_dev(off, torch.int32), E, d, F, bits, 0, p1, s1, p2, s2, y_dtype=torch.float32).double()
    assert torch.isfinite(y).all()
    for e in range(E):
        lo, hi = int(off[e]), int(off[e + 1])
        v = x[lo:hi].double()
        for canon, s, _ in quantised:
            q = canon[e].to(torch.int32)
            if bits == 4:
                q = torch.stack([(q << 28) >> 28, (q << 24) >> 28], dim=-1).reshape(q.shape[0], -1)
            v = v @ (q.double() * s[e].reshape(1, -1).double())
            if s is s1:
                v = v.clamp(min=0).to(torch.bfloat16).double()
        rel = (y[lo:hi] - v).norm(dim=1) / v.norm(dim=1)
        # an element of h that rounds the other way is off by 2^-8 at most; the few that do are well below the acceptance bound
        assert float(rel.max()) <= REL_L2_TOL, (e, float(rel.max()))


def test_conversion_by_what_its_kernel_shows_of_it():
    """Sizes on both sides of the rule where one figure for all kernels answered wrongly."""
    sizes = [((713, 8, 4096, 16384, 4), False), ((490, 16, 2048, 8192, 4), False), ((3862, 8, 4096, 16384, 8), False), ((252, 8, 4096, 16384, 8), True), ((7, 8, 4096, 16384, 8), False), ((12, 32, 2048, 8192, 8), False), ((65, 8, 1024, 4096, 8), True),
             ((1218, 8, 768, 3072, 8), True), ((1906, 16, 768, 3072, 4), True)]
    for (s, want), c in zip(sizes, L.record([L.ffn(*s, 0, B.MOE_BF16) for s, _ in sizes])):
        assert want != any(p.kernel.startswith("rows_to_f16") for p in c.launches), s


def _masters(rng, E, d, F, bits, g):
    w = [(rng.standard_normal((E, *s)) * 0.05).astype(np.float32) for s in ((d, F), (F, d))]
    return [B.moe_quantize_experts(to_dev(m, torch.float32), bits, g, want_canon=False)[1:] for m in w]


# Without biases the layer commutes with powers of two: rows of any size give the same bits, scaled, as long as x, h and y stay in range (unscaled they are
# below 2^4; at 2^-100 the few elements of h below 2^-26 lose bits that bf16 does not have)
SCALES = [2.0 ** k for k in (-100, -60, 60, 100, 115, 119, 123)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d,F,bits", CASES)
def test_row_tiles_take_rows_of_any_size(rows, d, F, bits):
    print(f"bf16 row sizes rows={rows[:5]} d={d} F={F} bits={bits}", flush=True)
    rng = np.random.default_rng(d + F + bits)
    E, off = len(rows), to_dev(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32), torch.int32)
    (s1, p1), (s2, p2) = _masters(rng, E, d, F, bits, 0)
    x = to_dev(rng.standard_normal((sum(rows), d)).astype(np.float32), torch.bfloat16)
    ffn = lambda v: B.moe_grouped_ffn_wq(v, off, E, d, F, bits, 0, p1, s1, p2, s2, y_dtype=torch.float32).double()  # noqa: E731
    _compare_scaled(ffn, x)


@pytest.mark.gpu
@pytest.mark.parametrize("T,E,d,F,bits,g", [(40, 6, 192, 576, 4, 0), (40, 6, 192, 576, 8, 0), (40, 6, 192, 576, 4, 64), (40, 6, 192, 576, 8, 64), (90, 12, 256, 4096, 4, 0),
                                            (90, 12, 256, 4096, 8, 0), (90, 12, 256, 4096, 4, 128), (250, 8, 128, 2048, 4, 0), (250, 8, 128, 2048, 4, 64),
                                            (3, 5, 64, 2112, 4, 0), (3, 5, 1088, 576, 8, 0)])
def test_the_decode_kernel_takes_rows_of_any_size(T, E, d, F, bits, g):
    print(f"bf16 row sizes T={T} E={E} d={d} F={F} bits={bits} g={g}", flush=True)
    rng = np.random.default_rng(T + d + F + bits)
    (s1, p1), (s2, p2) = _masters(rng, E, d, F, bits, g)
    x = to_dev(rng.standard_normal((T, d)).astype(np.float32), torch.bfloat16)
    idx, one = to_dev(rng.integers(0, E, (T, 1)).astype(np.int32), torch.int32), torch.ones((T, 1), device="cuda")
    _compare_scaled(lambda v: B.moe_grouped_ffn_wq_sliced(v, idx, one, E, d, F, bits, g, p1, s1, p2, s2)[0].double(), x)


def _compare_scaled(ffn, x):
    want, size = ffn(x), torch.ones((len(x), 1), device="cuda", dtype=torch.float64)
    for i, s in enumerate(SCALES):
        size[i::len(SCALES)] = s                      # rows of very different sizes side by side
    got = ffn((x.double() * size).to(torch.bfloat16)) / size
    assert torch.isfinite(got).all() and (want.norm(dim=1) > 0).all()
    small = size[:, 0] < 2.0 ** -90
    assert torch.equal(got[~small], want[~small])
    assert ((got - want).norm(dim=1) <= 1e-6 * want.norm(dim=1)).all()
    # close to the smallest normal numbers h has units of 2^-133, 2^-13 unscaled: half of one lost in elements whose root mean square is 2^-2 at least, 2^-12; x
    # loses as much in its small elements; twice that for rows of few large elements
    tiny = ffn((x.double() * 2.0 ** -120).to(torch.bfloat16)) * 2.0 ** 120
    lost = ((tiny - want).norm(dim=1) / want.norm(dim=1)).max()
    print(f"   lost at 2^-120: {float(lost):.2e}", flush=True)
    assert lost <= 2.0 ** -10
