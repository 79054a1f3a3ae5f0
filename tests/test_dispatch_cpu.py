"""Which kernels the library launches for which sizes (launches.py: recorded on the CPU, nothing runs)."""
import pytest

import launches as L
from paper_2211_10017_amd import binding as B


@pytest.fixture(scope="module", autouse=True)
def _library():
    B.load()


@pytest.mark.parametrize("act", [B.MOE_F16, B.MOE_BF16])
def test_gate_of_few_tokens_by_many_experts_is_spread_over_the_chip(act):
    """Up to 512 tokens by 65 to 256 experts, odd counts included: a block per token or two.  (On the matrix cores sixteen
    tokens by all experts keep one compute unit busy: 64 tokens, 255 experts, d = 1024 77 us against 14.)"""
    sizes = [(T, d, E) for E in (65, 66, 99, 127, 128, 129, 130, 136, 250, 255, 256) for T in (1, 64, 256, 257, 512) for d in (512, 4096)]
    for (T, d, E), call in zip(sizes, L.record([L.gate(T, d, E, act) for T, d, E in sizes])):
        (launch,) = call.launches
        assert call.rc == 0 and launch.kernel.startswith("gate_lanes_kernel"), (T, d, E, launch)
        assert launch.grid[0] == (T if T <= 256 else (T + 1) // 2)
