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


def test_permute_shares_its_work_by_the_number_of_assignments():
    """One launch up to 4096 assignments: four, eight or sixteen wavefronts per block, and up to 64 blocks whatever their size where rows
    are copied.  (2000 rows of 4096 copied by a quarter of the blocks: 29 us against 13.)"""
    cases = [(1, 8, 4, 1), (256, 8, 4, 64), (257, 8, 8, 64), (512, 1000, 8, 64), (513, 8, 16, 64), (4096, 500, 16, 64), (4096, 1000, 8, 64)]
    for (R, E, waves, blocks), copies, index in zip(cases, L.record([L.permute(R, 1, E, 1024) for R, E, _, _ in cases]), L.record([L.permute(R, 1, E) for R, E, _, _ in cases])):
        assert [(p.block, p.grid[0]) for p in copies.launches] == [(64 * waves, blocks)], (R, E)
        assert [(p.block, p.grid[0]) for p in index.launches] == [(64 * waves, 1)] and index.launches[0].shared <= 64 * 1024
