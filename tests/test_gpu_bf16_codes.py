"""bf16 rows of channel-scaled layers that meet bf16 codes as they are: every kernel with row tiles against the oracle."""
import pytest

import launches as L
from paper_2211_10017_amd import binding as B

# rows per expert, d, F, bits: 16-, 32- and 64-row blocks of the ring, the long ring, register-fed tiles of 32, 64 and 128 rows; partly filled tiles
# and last column blocks, odd numbers of K steps
CASES = [([16, 0, 17, 1, 2, 0, 33, 3, 5], 192, 576, 8), ([33, 32, 5, 0, 31], 704, 1216, 8), ([64, 65, 1, 128], 704, 1216, 8), ([50] * 32, 320, 1792, 8),
         ([20] * 40 + [0, 33], 192, 2688, 4), ([20] * 40 + [0, 33], 192, 5120, 8), ([60, 50, 33, 5] * 4, 192, 3392, 4), ([60, 50, 33, 5] * 4, 256, 3456, 8),
         ([270, 257, 130, 20], 2176, 4736, 4), ([300, 290, 270], 2112, 4224, 8)]


def test_cases_reach_every_kernel_without_a_conversion():
    ran = [[p.kernel for p in c.launches] for c in L.record([L.ffn(sum(r), len(r), d, F, bits, 0, B.MOE_BF16) for r, d, F, bits in CASES])]
    assert not any(k.startswith("rows_to_f16") for c in ran for k in c)
    built = {f"grouped_gemm_kernel<{b}, 0, {tm}>" for b in (4, 8) for tm in (1, 2, 4)} | {f"grouped_gemm_ring_kernel<8, 0, {bm}>" for bm in (16, 32, 64)}
    built |= {"grouped_gemm_ring_long_kernel<8, 0, 64>"}
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
