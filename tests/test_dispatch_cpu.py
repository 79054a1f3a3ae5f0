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


def _kernels(call):
    return [p.kernel.split("<")[0] for p in call.launches if not p.kernel.startswith("rows_to_f16")]


def test_ffn_streams_where_streaming_is_the_faster_way():
    """The pair of GEMMs of permuted rows, several rows per expert: the streaming kernels for few row groups in all, few experts
    and small weights; row tiles where the experts' weights would be read more than once from memory or many tiles are there."""
    u, s, ring = "stream_unrolled_kernel", "stream_gemm_kernel", "grouped_gemm_ring_kernel"
    cases = [((40, 8, 1024, 4096, 4), [u, u]), ((40, 1, 1024, 4096, 4), [u, u]), ((64, 2, 512, 2048, 8), [u, u]), ((64, 1, 2048, 8192, 8), [u, s]),
             ((8, 1, 2048, 8192, 4), [u, s]), ((128, 4, 1024, 1024, 8), [u, u]), ((200, 128, 512, 512, 8), [u, u]),
             ((256, 16, 1024, 4096, 4), [ring, ring]), ((64, 32, 4096, 16384, 8), [ring, ring]), ((128, 32, 1024, 4096, 8), [u, ring]),
             ((128, 16, 2048, 8192, 4), [u, ring]),
             ((20, 32, 1024, 4096, 4), [u, u]), ((20, 32, 2048, 8192, 8), [u, s]), ((3, 4, 4096, 16384, 8), [s, s])]       # at most a row per expert: always
    for (sizes, want), call in zip(cases, L.record([L.ffn(*c) for c, _ in cases])):
        assert call.rc == 0 and _kernels(call) == want, (sizes, _kernels(call))


def test_layers_fetch_through_the_index_where_fc2_runs_in_row_tiles():
    lib = B.load()
    pays = lambda R, E, T, d, F, bits, g=0, act=B.MOE_F16: lib.moe_grouped_ffn_wq_indexed_pays(R, E, T, d, F, bits, g, act)  # noqa: E731
    assert pays(128, 32, 128, 1024, 4096, 8) and pays(384, 32, 192, 1024, 4096, 4) and pays(128, 64, 64, 4096, 16384, 4, 128)
    assert not pays(96, 2, 48, 2048, 2048, 8) and not pays(20, 32, 20, 1024, 4096, 8) and not pays(0, 32, 0, 1024, 4096, 8)
    assert pays(1, 32, 1, 1024, 4096, 8, 0, B.MOE_BF16)
    gated = lib.moe_grouped_ffn_wq_gated_pays
    assert gated(64, 2, 64, 1024, 4096, 8, 0, B.MOE_F16) and not gated(64, 2, 32, 2048, 8192, 4, 0, B.MOE_F16)


def _rows_of_tiles(call):
    """Rows per block of each GEMM in row tiles, negative in the register-fed kernel."""
    out = []
    for p in call.launches:
        name, args = p.kernel.split("<")[0], p.kernel.split("<")[1].rstrip(">").split(", ")
        if name == "grouped_gemm_ring_kernel":
            out.append(int(args[2]))
        elif name == "grouped_gemm_kernel":
            out.append(-32 * int(args[2]))
    return out


def test_register_fed_tiles_where_the_ring_unpacks_too_often():
    """4-bit weights, few rows per expert, many tiles; and 8-bit weights with 29 to 32 rows per expert."""
    cases = [((64, 32, 1024, 4096, 4, 128), [16, 16]), ((256, 32, 2048, 8192, 4, 128), [-32, 16]), ((256, 32, 4096, 16384, 4, 128), [-32, -32]),
             ((128, 64, 4096, 16384, 4, 128), [-32, 16]), ((512, 128, 1024, 4096, 4, 128), [-32, -32]), ((500, 128, 1024, 4096, 8, 128), [16, 16]),
             ((1024, 32, 2048, 8192, 8, 128), [-32, -32]), ((64, 2, 2048, 8192, 8, 128), [32, 32]), ((384, 16, 1024, 4096, 8, 128), [32, 32])]
    for (sizes, want), call in zip(cases, L.record([L.ffn(*c) for c, _ in cases])):
        assert _rows_of_tiles(call) == want, (sizes, call.launches)


def test_noted_kernels_are_the_ones_launched():
    """moe_last_ffn_kernels names every GEMM kernel that the call launches, in order, the two kinds of row tiles told apart."""
    cases = [L.ffn(64, 32, 1024, 4096, 8), L.ffn(2000, 8, 1024, 4096, 4), L.ffn(1024, 32, 2048, 8192, 8), L.ffn(250, 4, 512, 2048, 4, 128, B.MOE_BF16),
             L.ffn(40, 1, 2048, 8192, 8), L.indexed(500, 32, 1, 1024, 4096, 4), L.indexed(9000, 16, 2, 1024, 2048, 4, 128, B.MOE_BF16)]
    seen = set()
    for call in L.record(cases):
        assert call.rc == 0 and call.noted == " ".join(_kernels(call))
        seen |= set(_kernels(call))
    assert seen == {"stream_unrolled_kernel", "stream_gemm_kernel", "grouped_gemm_kernel", "grouped_gemm_ring_kernel"}


def test_lds_limits_are_raised_on_every_device():
    """A kernel that needs more than the default 64 KB of dynamic LDS asks for it once on each device that it runs on."""
    calls = [L.gate(9000, 512, 256), L.ffn(592, 4, 256, 320, 8), L.ffn(40, 1, 2048, 8192, 8)]
    rows = L.record([(*c, dev) for dev in (0, 1, 0, 5) for c in calls])
    for i in range(len(calls)):
        first, second, again, other = rows[i], rows[i + len(calls)], rows[i + 2 * len(calls)], rows[i + 3 * len(calls)]
        big = {p.kernel for p in first.launches if p.shared > 64 * 1024}
        assert big and big <= {k for k, _ in first.raised}
        assert [k for k, _ in second.raised] == [k for k, _ in first.raised] == [k for k, _ in other.raised] and not again.raised
        assert {d for _, d in second.raised} == {1} and {d for _, d in other.raised} == {5}


def test_every_form_of_the_row_tiles_is_in_the_two_build_comparison():
    """The cases of test_gpu_wait_guard.py and test_gpu_ring.py run the kernels they say, and together every instance the library has."""
    import torch

    from test_gpu_ring import RING
    from test_gpu_wait_guard import REGISTER_FED
    fed = L.record([L.ffn(sum(c[0]), len(c[0]), *c[1:5], B._DT[c[5]]) for c in REGISTER_FED])
    for case, call in zip(REGISTER_FED, fed):
        assert [p.kernel for p in call.launches if p.kernel.startswith("grouped")][0] == case[6], case
    ring = L.record([L.ffn(sum(c[0]), len(c[0]), *c[1:5], B._DT[{"f16": torch.float16, "bf16": torch.bfloat16}[c[5]]]) for c in RING])
    ran = {p.kernel for call in fed + ring for p in call.launches}
    modes, acc = (0, 1, 2, 4), 3                   # per channel, per group, two-term, per channel with bf16 rows; group sums
    built = {f"grouped_gemm_kernel<{b}, {m}, {t}>" for b in (4, 8) for m in modes for t in (1, 2, 4)} | {f"grouped_gemm_kernel<{b}, {acc}, {t}>" for b in (4, 8) for t in (1, 2)}
    built |= {f"grouped_gemm_ring_kernel<{b}, {m}, {bm}>" for b in (4, 8) for m in (0, 1, acc, 4) for bm in (16, 32, 64)}
    assert built <= ran, built - ran


def test_the_oracle_comparisons_reach_every_kernel():
    """Each GEMM kernel with its scale modes and tile heights is compared with the oracle, row by row, by some case of test_gpu_steps.py,
    test_gpu_ring.py or test_gpu_tile_end.py."""
    import test_gpu_ring
    import test_gpu_steps
    import test_gpu_tile_end

    def params(test, i=0):
        return test.pytestmark[i].args[1]
    bf = {"f16": B.MOE_F16, "bf16": B.MOE_BF16}
    calls = [L.ffn(sum(p[0]), len(p[0]), *p[1:5], bf[p[5]]) for p in params(test_gpu_steps.test_grouped_ffn_matches_oracle)]
    calls += [L.ffn(sum(p[0]), len(p[0]), *p[1:4], bound=max(p[0])) for p in params(test_gpu_steps.test_grouped_ffn_with_a_row_bound_matches_oracle)]
    calls += [L.ffn(sum(r[0]), len(r[0]), r[1], r[2], a[1], a[2], bf[a[0]]) for r in params(test_gpu_tile_end.test_tile_end_matches_oracle_in_every_output_type)
              for a in params(test_gpu_tile_end.test_tile_end_matches_oracle_in_every_output_type, 1)]
    ring = test_gpu_ring.test_ring_gemm_matches_oracle
    calls += [L.ffn(sum(r), len(r), *df, a[1], a[2], bf[a[0]]) for r in params(ring, 2) for df in params(ring, 1) for a in params(ring, 0)]
    launched = L.record(calls)
    assert all(c.rc == 0 for c in launched)
    ran = {p.kernel.split(", false")[0] for c in launched for p in c.launches}
    fed = {f"grouped_gemm_kernel<{b}, {m}, {t}>" for b, m, t in [(4, 0, 1), (4, 2, 1), (8, 1, 1), (8, 3, 1), (8, 0, 2), (4, 1, 2), (8, 2, 2), (4, 3, 2), (4, 0, 4), (4, 1, 4),
                                                                 (4, 2, 4), (8, 0, 4), (8, 1, 4), (8, 2, 4)]}
    ring = {f"grouped_gemm_ring_kernel<{b}, {m}, {bm}>" for b, m in [(4, 0), (8, 0), (4, 1), (8, 1), (8, 3), (4, 3)] for bm in (16, 32, 64)}
    stream = {"stream_gemm_kernel<4>", "stream_gemm_kernel<8>"} | {f"stream_unrolled_kernel<{b}, {kb}, {t}, {s}" for b in (4, 8) for kb, t, s in [(16, 1, 1), (32, 1, 1), (48, 1, 1), (64, 2, 4)]}
    assert fed | ring | stream <= ran, (fed | ring | stream) - ran


def test_long_rings_where_a_64_row_tile_has_its_compute_unit_to_itself():
    """8-bit weights of 18 MB and more and up to 240 tiles, as typical row counts make them."""
    cases = [((2000, 16, 3072, 768, 8), True), ((2000, 16, 3072, 768, 8, 128), True), ((600, 8, 768, 3072, 8, 128), False), ((600, 8, 512, 2048, 8, 64), False),
             ((2000, 16, 3072, 768, 4), False)]
    for (sizes, want), call in zip(cases, L.record([L.ffn(*c) for c, _ in cases])):
        ring = [p for p in call.launches if p.kernel.startswith("grouped_gemm_ring") and p.kernel.endswith("64>")]
        assert ring and (ring[0].shared > 80 * 1024) is want, (sizes, call.launches)


def test_decode_kernel_has_blocks_for_every_row_group_of_any_routing():
    """A block per slice and (expert, sixteen or thirty-two of its rows), however the rows fall: at most one item per assignment, and one per
    expert and for each further pass of rows.  (128 rows on two of 64 experts of 4096 x 16384, group scales: 383 us with the passes of an expert in one
    block, 8.2 ms for ... )"""
    cases = [((1, 2, 32, 1024, 4096, 4), 2, 64), ((64, 2, 64, 4096, 16384, 4, 128), 64 + 4, 32), ((192, 2, 32, 1024, 4096, 4), 32 + 352 // 32, 8),
             ((256, 2, 2, 64, 64, 8), 2 + 510 // 16, 1), ((256, 2, 2, 64, 64, 4), 2 + 510 // 32, 1), ((256, 2, 512, 64, 64, 4), 512, 1)]
    for (sizes, items, slices), call in zip(cases, L.record([L.sliced(*c[0]) for c in cases])):
        assert call.rc == 0 and call.launches[0].kernel.startswith("decode_ffn_kernel") and call.launches[0].grid[0] == 1 + items * slices, (sizes, call.launches)


def test_gated_call_cuts_d_ff_as_the_sliced_call_does():
    """The decode kernel in the gated call: slices as wide as the batch asks for, wider where the workspace holds no more, the workspace
    query large enough for them, and no room for partial sums where that kernel does not run."""
    lib = B.load()
    sizes = [(1, 2, 32, 1024, 4096, 4), (4, 2, 32, 1024, 4096, 4), (16, 2, 32, 1024, 4096, 4), (64, 2, 32, 1024, 4096, 4), (128, 2, 64, 1024, 4096, 4),
             (60, 1, 8, 1024, 4096, 4), (1, 1, 16, 512, 2048, 8), (128, 2, 128, 512, 2048, 8), (100, 1, 64, 1024, 1024, 4)]
    query = lambda T, k, E, d, F: lib.moe_grouped_ffn_wq_workspace_bytes(T * k, d, F, E, B.MOE_F16)  # noqa: E731
    own, sliced, tight = (L.record(c) for c in ([L.gated(*s, workspace=query(*s[:5])) for s in sizes], [L.sliced(*s) for s in sizes],
                                                [L.gated(*s, workspace=max(s[4] // 512 * s[0] * s[1] * s[3] * 4, 1 << 16)) for s in sizes]))
    for s, a, b, c in zip(sizes, own, sliced, tight):
        assert a.rc == b.rc == 0 and a.launches == b.launches and a.launches[0].kernel.startswith("decode_ffn_kernel"), (s, a.launches, b.launches)
        assert c.rc == 0 and c.launches[0].grid[0] <= a.launches[0].grid[0]
    assert tight[3].launches[0].kernel == "decode_ffn_kernel<4, false, false, 8, 1>" != own[3].launches[0].kernel
    assert L.record([L.gated(*sizes[3], workspace=8 * 128 * 1024 * 4 - 1)])[0].rc == 3
    assert query(128, 2, 64, 4096, 16384) == 256 * 16384 * 2              # h and nothing else
    assert L.record([("moe_grouped_ffn_wq_noalloc", [*L.ffn(120, 15, 1024, 4096, 4)[1][:-3], None])])[0].rc == 0    # (8 MiB hold its h, not the slices)


def _pays(T, k, E, d, F, bits, g=0, act=B.MOE_F16):
    return B.load().moe_grouped_ffn_wq_sliced_pays(T, k, E, d, F, bits, g, act)


def test_layers_are_not_cut_into_thousands_of_narrow_slices():
    assert not _pays(218, 1, 115, 256, 5312, 4, 64) and not _pays(139, 1, 131, 640, 4544, 4, 64) and not _pays(71, 2, 232, 576, 5952, 4, 0, B.MOE_BF16)
    assert not _pays(184, 2, 167, 1024, 4800, 8, 64)
    assert _pays(43, 1, 71, 448, 6720, 4) and _pays(236, 2, 78, 64, 7552, 8, 0, B.MOE_BF16) and _pays(218, 1, 115, 256, 5120, 4, 64)


def test_eight_bit_layers_are_sliced_unless_the_route_below_streams():
    """FP16 rows, channel scales, 140 to 300 MB of active weights: what decides is which kernel the layer would run otherwise."""
    assert all(_pays(*c, 8) for c in [(40, 2, 32, 1088, 4096), (60, 2, 32, 1088, 4096), (60, 2, 32, 960, 4096), (128, 2, 32, 960, 4096), (160, 2, 128, 512, 2048),
                                      (256, 2, 96, 512, 2560), (150, 2, 60, 768, 3072), (128, 2, 64, 512, 4096), (35, 1, 7, 2048, 8192)])
    assert not any(_pays(*c, 8) for c in [(40, 2, 32, 1024, 4096), (100, 1, 32, 1024, 4096), (128, 2, 32, 1024, 4096), (100, 1, 24, 2048, 2048),
                                          (64, 1, 8, 4096, 4096), (100, 2, 67, 512, 2112), (38, 2, 42, 1024, 2048)])
    assert _pays(28, 1, 32, 1024, 4096, 8) and _pays(40, 2, 32, 1024, 4096, 4) and _pays(40, 2, 32, 1024, 4096, 8, 0, B.MOE_BF16)


def test_both_calls_answer_alike_for_the_decode_kernel():
    """Where the gated call runs the decode kernel a layer takes the sliced call, whose launches are the same."""
    sizes = [(128, 2, 128, 1024, 4096, 4), (100, 2, 128, 1024, 4096, 4), (64, 2, 256, 1024, 4096, 4), (60, 1, 8, 1024, 4096, 4), (128, 2, 128, 512, 2048, 8),
             (64, 2, 32, 1024, 4096, 4), (128, 1, 16, 1024, 4096, 4), (128, 2, 256, 512, 2048, 8)]
    for s, a, b in zip(sizes, L.record([L.gated(*s) for s in sizes]), L.record([L.sliced(*s) for s in sizes])):
        assert a.launches[0].kernel.startswith("decode_ffn_kernel") and a.launches == b.launches and _pays(*s), s


def test_long_rings_only_where_one_round_of_blocks_is_expected():
    """64-row tiles as uniform routing makes them: 65 to 90 rows per expert are two tiles nearly everywhere."""
    cases = [((300, 4, 1280, 5120, 8), [False, True]), ((100, 1, 5120, 20480, 8), [False, True]), ((150, 2, 1280, 10240, 8), [False, True]),
             ((340, 4, 1280, 5120, 8), [False, True]), ((1994, 16, 768, 3072, 8), [False, True]), ((64, 1, 4096, 16384, 8), [True, True]), ((65, 1, 4096, 16384, 8), [True, True]), ((65, 1, 4096, 16448, 8), [False, True]),
             ((714, 26, 896, 2368, 8, 64), [False, False]), ((2046, 18, 7296, 832, 8, 64), [False, False]), ((722, 14, 3648, 1984, 8), [True, False])]
    for (sizes, want), call in zip(cases, L.record([L.ffn(*c) for c, _ in cases])):
        assert [p.shared > 80 * 1024 for p in call.launches if not p.kernel.startswith("rows")] == want, (sizes, call.launches)
        assert [p.kernel.startswith("grouped_gemm_ring_long") for p in call.launches if not p.kernel.startswith("rows")] == want      # its depth is a constant


def test_the_oracle_comparisons_reach_every_long_ring():
    import test_gpu_ring
    act = {"f16": B.MOE_F16, "bf16": B.MOE_BF16}
    (m_act, m_rows) = test_gpu_ring.test_long_rings_match_oracle_and_the_build_that_waits_for_all_loads.pytestmark
    ran = {p.kernel for rows, d, F in m_rows.args[1] for a, g in m_act.args[1] for p in L.record([L.ffn(sum(rows), len(rows), d, F, 8, g, act[a])])[0].launches}
    assert {f"grouped_gemm_ring_long_kernel<8, {m}, 64>" for m in (0, 1, 3, 4)} <= ran, ran


def test_the_oracle_comparisons_reach_every_form_of_the_decode_kernel():
    """Weight width, kind of scales, row type, slice width and sixteens of rows of the decode kernel, and the three reductions."""
    import test_gpu_sliced as t

    bf = {"f16": B.MOE_F16, "bf16": B.MOE_BF16}
    marks = lambda f: [m.args[1] for m in f.pytestmark]  # noqa: E731
    (loads, acts, sizes), (ts, wide_acts, wide), (rows, few) = (marks(f) for f in (t.test_sliced_ffn_matches_oracle, t.test_wide_slices_match_oracle,
                                                                                   t.test_few_rows_over_few_and_many_slices_match_oracle))
    calls = [L.sliced(T, k, E, d, F, b, g, bf[a]) for T, k, E, _ in loads for a, b, g in acts for d, F in sizes]
    calls += [L.sliced(T, 2, 34, d, F, b, g, bf[a]) for T in ts for a, b, g in wide_acts for d, F in wide]
    calls += [L.sliced(T, k, 5, d, F, 4) for T, k in rows for d, F in few]
    ran = {p.kernel for c in L.record(calls) for p in c.launches}
    flag = ("false", "true")
    built = {f"decode_ffn_kernel<{b}, {flag[g]}, {flag[f]}, {cw}, {rt}>" for b in (4, 8) for g in (0, 1) for f in (0, 1) for cw in (1, 2, 4, 8) for rt in (1, 2)
             if rt == 1 or b == 4}
    built |= {"decode_reduce_kernel<16, 4>", "decode_reduce_kernel<8, 4>", "decode_reduce_kernel<4, 2>"}
    assert built <= ran, built - ran
    reduced = {c.launches[1].kernel for c in L.record([L.sliced(T, k, 5, d, F, 4) for T, k in rows for d, F in few])}
    assert len(reduced) == 3
    (few_bf16,) = marks(t.test_few_bf16_rows_over_few_and_many_slices_match_oracle)
    codes = {c.launches[1].kernel for c in L.record([L.sliced(3, 2, 5, d, F, b, 0, B.MOE_BF16) for d, F, b in few_bf16])}
    assert codes == {k.replace("reduce", "reduce_codes") for k in reduced}


def test_large_group_scaled_experts_with_many_rows_stay_in_row_tiles():
    """Crowded routing would read their weights for every sixteen rows."""
    assert not _pays(256, 2, 64, 4096, 8192, 4, 128) and not _pays(256, 2, 64, 4096, 16384, 4, 128) and not _pays(192, 2, 64, 4096, 8192, 4, 128)
    assert _pays(160, 2, 64, 4096, 8192, 4, 128) and _pays(64, 2, 64, 4096, 16384, 4, 128) and _pays(256, 2, 64, 2048, 8192, 4, 128)


def test_the_conversion_of_bf16_rows_is_compared_in_every_form():
    """Each row length of test_gpu_indexed.py runs the form that it stands for, in calls that convert."""
    from test_gpu_indexed import LENGTHS
    converted = L.record([L.ffn(9, 2, 64, K, 8, 64, B.MOE_BF16) for K, _ in LENGTHS])
    assert [c.launches[2].kernel for c in converted] == [f"rows_to_f16_kernel<{256 if 4096 < K <= 16384 else 64}, {nv}>" for K, nv in LENGTHS]
    assert not any(p.kernel.startswith("rows_to_f16") for c in L.record([L.ffn(9, 2, 64, K, 8, 0, B.MOE_BF16) for K in (1024, 1088, 4096, 4160)]) for p in c.launches)


def test_the_unsorted_call_launches_what_the_indexed_call_does():
    """The same launches in the same order, for every form that it takes; what it does not take is refused; and it pays only where few blocks sort."""
    import itertools
    forms = [(T, k, E, d, F, bits, g, act, k == 1) for (T, k, E), (d, F), bits, g, act in itertools.product(
        [(1, 1, 1), (3, 2, 8), (64, 2, 32), (257, 1, 65), (2048, 2, 16), (4096, 1, 1024)], [(64, 128), (512, 2048), (4096, 1024)], (4, 8), (0, 64, 128), (B.MOE_F16, B.MOE_BF16))
        if not (g == 128 and d == 64)]
    here, there = L.record([L.unsorted(*f) for f in forms]), L.record([L.indexed(f[0] * f[1], f[2], f[1], *f[3:8], f[0], f[8]) for f in forms])
    for f, a, b in zip(forms, here, there):
        assert a.rc == b.rc == 0 and a.noted == b.noted, f
        tall, low = ("grouped_gemm_kernel<%d, 3, %d>" % (f[5], tm) for tm in (2, 1))
        if tall in [p.kernel for p in b.launches]:      # (fc1 in 64-row tiles of group sums, which do not sort: 32-row ones)
            assert [p.kernel for p in a.launches] == [p.kernel.replace(tall, low) for p in b.launches]
            assert not B.load().moe_grouped_ffn_wq_unsorted_pays(*f[:8]), f
        else:
            assert a.launches == b.launches, f
    refused = [L.unsorted(2049, 2, 8, 64, 64, 4), L.unsorted(4097, 1, 8, 64, 64, 4), L.unsorted(8, 1, 1025, 64, 64, 4), L.unsorted(0, 1, 8, 64, 64, 4), L.unsorted(8, 3, 8, 64, 64, 4),
               L.unsorted(8, 2, 8, 64, 64, 4, scale=True), L.unsorted(8, 1, 8, 96, 64, 4), L.unsorted(8, 1, 8, 64, 64, 5), L.unsorted(8, 1, 8, 64, 64, 4, 128),
               L.unsorted(8, 1, 8, 64, 64, 4, idx=None), L.unsorted(8, 1, 8, 64, 64, 4, act=B.MOE_F32)]
    assert all(c.rc in (1, 2) and not c.launches for c in L.record(refused))
    pays = lambda *a: B.load().moe_grouped_ffn_wq_unsorted_pays(*a)  # noqa: E731
    assert pays(683, 2, 32, 512, 2048, 4, 0, B.MOE_F16) and pays(1270, 2, 16, 1024, 4096, 8, 0, B.MOE_F16) and pays(31, 2, 64, 2048, 8192, 4, 128, B.MOE_BF16)
    assert not pays(1215, 2, 64, 2048, 8192, 4, 0, B.MOE_F16) and not pays(387, 2, 128, 1024, 4096, 8, 0, B.MOE_F16) and not pays(4097, 1, 8, 512, 2048, 4, 0, B.MOE_F16)


def test_small_and_few_experts_are_sliced_up_to_about_one_block_each():
    bf = B.MOE_BF16
    assert _pays(20, 2, 8, 512, 2048, 4, 0, bf) and _pays(141, 1, 16, 768, 3072, 4, 128) and _pays(149, 1, 8, 1024, 4096, 4) and _pays(82, 1, 8, 512, 2048, 8, 0, bf)
    assert _pays(229, 1, 128, 768, 3072, 8, 0, bf) and _pays(11, 2, 16, 4096, 16384, 4) and _pays(12, 1, 32, 2048, 8192, 8)
    assert not any(_pays(*c) for c in [(256, 1, 8, 512, 2048, 8), (113, 2, 8, 2048, 8192, 4), (238, 2, 8, 768, 3072, 4), (7, 1, 32, 4096, 16384, 8), (11, 1, 64, 4096, 16384, 4, 0, bf),
                                       (133, 1, 8, 4096, 16384, 8), (99, 2, 32, 4096, 16384, 4)])


def test_the_unsorted_call_streams_fc1_where_the_gated_call_does():
    """Level 1 of the gated call, where it pays: the same launches, fc2 in row tiles; a layer takes it with one expert per token."""
    lib = B.load()
    sizes = [(40, 1, 32, 1024, 4096, 8), (200, 1, 8, 1024, 4096, 8), (40, 1, 8, 512, 2112, 8), (100, 2, 12, 512, 2112, 8)]
    for s, a, b in zip(sizes, L.record([L.unsorted(*s) for s in sizes]), L.record([L.gated(*s, scale=False) for s in sizes])):
        assert a.rc == b.rc == 0 and a.launches == b.launches and _kernels(a)[0] == "stream_unrolled_kernel", (s, a.launches)
        assert bool(lib.moe_grouped_ffn_wq_unsorted_pays(*s, 0, B.MOE_F16)) == (s[1] == 1)
    assert not lib.moe_grouped_ffn_wq_unsorted_pays(256, 1, 8, 512, 2048, 8, 0, B.MOE_F16)      # level 2: everything fused in the gated call
    # level 1 that pays, but permuted rows would stream through fc2: both GEMMs in row tiles, and no layer takes it
    sizes = [(1, 1, 4, 1024, 4096, 8), (1, 1, 4, 1024, 3072, 8), (1, 1, 4, 2048, 8192, 4)]
    for s, call in zip(sizes, L.record([L.unsorted(*s) for s in sizes])):
        assert lib.moe_grouped_ffn_wq_gated_supported(*s, 0, B.MOE_F16) == 1 and lib.moe_grouped_ffn_wq_gated_pays(*s, 0, B.MOE_F16)
        assert call.rc == 0 and all(k.startswith("grouped_gemm") for k in _kernels(call)) and not lib.moe_grouped_ffn_wq_unsorted_pays(*s, 0, B.MOE_F16), (s, call.launches)


def test_layers_of_eight_experts_and_more_leave_the_ring_by_their_expected_tiles():
    """Rows through the routing index: short K in register-fed tiles once these fill most of the chip, long K of few 64-row blocks in 32-row ones, and
    what lies on the other side of each line as with permuted copies."""
    cases = [((892, 64, 2, 768, 3072, 4), [-32, 32]), ((470, 16, 1, 1024, 4096, 4), [-32, 32]), ((783, 16, 1, 512, 2048, 4, 128), [-32, 32]), ((705, 32, 1, 768, 3072, 8), [-32, 32]),
             ((382, 8, 1, 768, 3072, 4), [64, 32]), ((1318, 8, 2, 512, 2048, 4), [-64, 32]), ((840, 128, 2, 1024, 4096, 4), [-32, -32]), ((2368, 32, 1, 512, 2048, 4), [-64, 64]),
             ((320, 4, 1, 768, 3072, 4), [64, 64]), ((1000, 8, 2, 768, 3072, 8), [-64])]       # (the last: fc2 in the long ring)
    from test_gpu_indexed import TAKEN
    cases += TAKEN
    for (sizes, want), call in zip(cases, L.record([L.indexed(*c) for c, _ in cases])):
        assert call.rc == 0 and _rows_of_tiles(call) == want, (sizes, call.launches)


def test_two_term_weights_do_not_take_the_rings_place():
    """bf16 rows with groups other than 128: in register-fed tiles fc1's weights are two-term FP16 numbers, which end at weights of 256; what the ring takes of
    permuted copies it takes of rows through the index, in the same blocks."""
    from test_gpu_indexed import LARGE_WEIGHTS
    sizes = LARGE_WEIGHTS + [(892, 64, 2, 768, 3072, 4, 64), (470, 16, 1, 1024, 4096, 4, 256), (705, 32, 1, 768, 3072, 8, 64), (783, 16, 1, 512, 2048, 4, 64),
                             (840, 128, 2, 2048, 1024, 4, 64), (382, 8, 1, 3072, 768, 4, 64)]
    here = L.record([L.indexed(*s, B.MOE_BF16) for s in sizes])
    copies = L.record([L.ffn(s[0], s[1], *s[3:], B.MOE_BF16) for s in sizes])
    for s, a, b in zip(sizes, here, copies):
        fc1, permuted = ([p for p in c.launches if p.kernel.startswith("grouped")][0] for c in (a, b))
        assert a.rc == b.rc == 0 and fc1 == permuted and fc1.kernel.startswith("grouped_gemm_ring"), (s, fc1, permuted)


def test_bf16_rows_are_converted_by_what_the_launched_tiles_cost():
    """Rows through the index on both sides of the line, at sizes whose tiles are not those of permuted copies: (sizes, whether converted)."""
    cases = [((831, 64, 1, 1024, 4096, 4), False), ((610, 128, 2, 512, 2048, 4), False), ((1411, 128, 1, 1024, 2048, 4), False), ((592, 64, 2, 768, 3072, 4), False),
             ((327, 8, 1, 2048, 8192, 4), True), ((713, 8, 1, 4096, 16384, 4), True), ((609 * 2, 8, 2, 768, 3072, 8), False)]
    calls = L.record([L.indexed(*c, 0, B.MOE_BF16) for c, _ in cases])
    for (sizes, converted), call in zip(cases, calls):
        assert call.rc == 0 and any(p.kernel.startswith("rows_to_f16") for p in call.launches) == converted, (sizes, call.launches)


def test_partial_sums_of_few_experts_stay_within_their_weights_reach():
    """Sizes that a layer leaves to the other routes, timed there against the sliced call; and over the whole range, beyond 35 MB in all, partial sums are at
    most twice the active weights, or a fifth where the lines for larger layers take them."""
    import random
    assert not any(_pays(*c) for c in [(512, 1, 1, 2048, 2048, 4), (509, 1, 1, 3328, 3712, 4), (512, 1, 1, 2048, 8192, 4), (512, 1, 1, 1024, 4096, 4), (256, 2, 2, 1024, 4096, 4),
                                       (256, 2, 4, 1024, 4096, 4), (256, 1, 1, 512, 2048, 4), (43, 2, 5, 1024, 4096, 4), (161, 1, 8, 2048, 1024, 4), (16, 2, 48, 2048, 8192, 4, 0, B.MOE_BF16)])
    assert all(_pays(*c) for c in [(64, 1, 9, 1024, 1024, 4, 128), (23, 1, 7, 3904, 15616, 4), (49, 2, 16, 2048, 1024, 4, 64, B.MOE_BF16), (311, 1, 32, 448, 1792, 4, 64, B.MOE_BF16),
                                   (40, 1, 2, 1024, 4096, 4), (16, 1, 1, 2048, 8192, 8, 0, B.MOE_BF16)])
    rng, taken = random.Random(1), 0
    for _ in range(20000):
        E, k = rng.choice([1, 2, 3, 4, 6, 8, 16, 64]), rng.choice([1, 2])
        T, d, F, bits = int(2 ** rng.uniform(0, 9 if k == 1 else 8)), 64 * rng.randint(1, 64), 64 * rng.randint(1, 128), rng.choice([4, 8])
        sizes = (T, k, E, d, F, bits, rng.choice([0, 64]), rng.choice([B.MOE_F16, B.MOE_BF16]))
        if k > E or not _pays(*sizes):
            continue
        taken += 1
        partial, weights = B.load().moe_grouped_ffn_wq_sliced_workspace_bytes(*sizes), E * (1 - (1 - 1 / E) ** (T * k)) * 2 * d * F * bits / 8
        assert partial <= 2.01 * weights + 256 or 2 * partial + weights <= 35.1e6, sizes
    assert taken > 3000


def test_the_gates_chains_leave_what_other_forms_do_faster():
    """Many features past the last whole block of 128, long bf16 tokens on few experts, and tokens that the LDS does not hold."""
    bf = B.MOE_BF16
    cases = [((133, 112, 128), "gate_lanes_kernel<"), ((133, 248, 128), "gate_lanes_kernel<"), ((133, 192, 128), "gate_lanes_kernel_wide<"), ((133, 376, 128), "gate_lanes_kernel_wide<"),
             ((683, 1016, 60, bf), "gate_quad_kernel<"), ((683, 1032, 60, bf), "gate_token_kernel<"), ((683, 1016, 60), "gate_token_kernel<"), ((512, 1016, 60, bf), "gate_token_kernel<"),
             ((443, 5120, 8, bf), "gate_mfma_kernel<"), ((770, 4096, 12, bf), "gate_mfma_kernel<"), ((443, 4096, 8, bf), "gate_token_kernel<"), ((443, 8192, 8), "gate_token_kernel<"),
             ((768, 10240, 64, bf), "gate_token_kernel<true, 64, 3>"), ((769, 10240, 64, bf), "gate_quad_kernel<"), ((1024, 8192, 64, bf), "gate_token_kernel<true, 64, 4>"),
             ((592, 10240, 100, bf), "gate_mfma_kernel<")]
    for (sizes, want), call in zip(cases, L.record([L.gate(*c) for c, _ in cases])):
        assert call.rc == 0 and call.launches[0].kernel.startswith(want), (sizes, call.launches)
