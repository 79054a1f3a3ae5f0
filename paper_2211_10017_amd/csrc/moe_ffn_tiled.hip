// Host side of the LDS-tiled grouped GEMM: tile height, grid size, and the hand-over to the
// translation unit that holds the kernels of the weight width and activation dtype asked for.
#include <math.h>

#include "moe_ffn_common.h"

namespace moe {

// Rows per block of the kernel with the LDS ring, or 0 where register-fed tiles do as well or better (steps of a layer, register-fed
// tiles against the ring).  Few rows per expert: the launch streams weights, and what counts is how much of them is in flight.
// 16-row blocks up to ten rows per expert on average: 64 tokens, two of 32 experts, group scales: 1024 x 4096 84 and 60 us, 2048 x 8192
// 188 and 141; 500 tokens on 128 experts of 1024 x 4096 8-bit 260 and 228.  With 4-bit weights, which cost more to unpack than to
// read, only while there are too few tiles to hide that: 384 (a tile per expert and 256 channels), with one or two rows per expert
// 512, and 1024 for long K loops.  (Shares of a call that the ring gains, fc1 / fc2: 192 to 256 tiles 3-27 / 5-38 %, 384 tiles -2 to 9 /
// -3 to 19 %, 512 tiles and more than two rows per expert -7 to -3 / -6 to 2 %, skewed loads of 256 rows on 32 experts of 4096 x 16384, group
// scales, -18 % of the call.)
// 32-row blocks while the tiles alone do not fill the chip two to four times (240 tokens on 32 experts of 2048 x 8192: 201 and 154;
// 1900 tokens on 128 of them: 578 and 671), once with 8-bit weights and 29 to 32 rows per expert, where half of the experts take a second
// block (1024 rows on 32 experts of 2048 x 8192: 237 and 267; 64 on two: 85 and 60).  Beyond: only where 64-row tiles leave compute units without a block (fc2 of 500
// tokens on 32 experts of 1024 x 4096, 126 tiles: 41 and 28 us; with 264 tiles of 2048 x 8192 98 and 103).
static int ring_rows(const GemmArgs &p, int bits, int mean)
{
    const long experts = p.E < p.R ? p.E : p.R, ncol = (p.N + 255) / 256;
    if (mean <= 10 && bits == 8) return 16;
    if (mean <= 10 && p.R <= 512) return experts * ncol <= (mean > 2 ? 384 : p.K > 4096 ? 1024 : 512) ? 16 : 0;
    if (mean <= 32) return ((long)p.R / 32 + experts / 2) * ncol <= (mean <= 16 ? 1024 : mean > 28 && bits == 8 ? 256 : 512) ? 32 : 0;
    return ((long)p.R / 64 + experts / 2) * ncol <= 224 ? 64 : 0;
}

constexpr long kLongRingWeights = 18000000l;        // the fewest 8-bit weights for ring_long

// Row tiles that R rows make on E experts under uniform routing, an expert's rows taken as normally distributed.
double expected_row_tiles(long R, long E, int bm)
{
    const double mean = (double)R / E, sd = sqrt(mean * (1.0 - 1.0 / E));
    double tiles = floor(fmax(mean - 4 * sd, 0.0) / bm);       // (that all experts fill)
    for (double first = tiles * bm; first < mean + 4 * sd; first += bm)
        tiles += sd > 0 ? 0.5 * erfc((first + 0.5 - mean) / (sd * M_SQRT2)) : 1.0;
    return tiles * E;
}

// ring_rows for rows fetched through the routing index, as layers do (its own lines were drawn with permuted copies), of eight experts and more, by the
// tiles that uniform routing makes (350 drawn layers, both GEMMs in every form: 49 of 710 GEMMs change, 44 of them by more than 2 % of the step, 7 % on
// average, none to the worse; us a step below):
//  - K up to 1024, where a block's start and end are most of it and the ring is hardly full before it ends: register-fed tiles from 0.9 of 32 rows per
//    compute unit on, with 8-bit weights between 0.8 and 1.8 and 11 to 64 rows per expert.  (fc1 of 446 tokens, two of 64 experts of 768 x 3072, 62 -> 53;
//    470, one of 16 of 1024 x 4096, 46 -> 38; 783, one of 16 of 512 x 2048 with groups of 128, 34 -> 32.5; 8-bit, 705, one of 32 of 768 x 3072, 53.6 -> 49.6;
//    left out 382, one of 8 of 768 x 3072, 0.7 tiles, 35 and 34.5.)
//  - longer K in 64-row blocks: 32-row ones up to one of them per compute unit (fc2 of 382 tokens, one of 8 of 3072 x 768, 34.7 -> 31.6; 735, 38.5 -> 35.3; 1318, one
//    of 8 of 2048 x 512, fc1 in tiles as well, 31.9 -> 28.7; at 1.4 blocks, 74 rows on each of 32 of 2048 x 512, 38 -> 40), unless ring_long takes those of 64.
//  - up to eight rows per expert of 4-bit weights in 32-row blocks, from 3.9 of these per compute unit on: tiles, which unpack as much for twice the columns
//    (fc2 of 420 tokens, two of 128 experts of 4096 x 1024, 152 -> 138).
// Not for the two-term weights of register-fed tiles (bf16 rows, groups other than 128): 256 times code times scale overflows FP16 from weights of 256 on, where
// the ring keeps exact codes and folds the scales in fp32, at half the matrix instructions.
static int ring_rows_for(const GemmArgs &p, int bits, int smode, int mean)
{
    const int ring = ring_rows(p, bits, mean);
    if (!ring || p.E < 8 || !p.indexed || smode == SCALE_GROUP_SPLIT) return ring;
    const double tiles = expected_row_tiles(p.R, p.E, 32), fed = tiles * ((p.N + 255) / 256) / 256, blocks = tiles * ((p.N + 127) / 128) / 256;
    if (p.K <= 1024) return (bits == 4 ? fed >= 0.9 : mean > 10 && mean <= 64 && fed >= 0.8 && fed <= 1.8) ? 0 : ring;
    if (ring == 64 && blocks <= 1.0 && !(bits == 8 && (long)p.E * p.K * p.N >= kLongRingWeights)) return 32;
    return ring == 32 && bits == 4 && mean <= 8 && blocks >= 3.9 ? 0 : ring;
}

// Whether 64-row blocks of 8-bit weights take the whole LDS of a compute unit for their ring: uniform routing makes no more blocks
// than compute units, and the weights are many enough to come from memory, whose latency one stage in flight does not cover.
// A block more than that and the launch takes two rounds where two blocks per compute unit took one.  (244 GEMMs in 130 drawn layers: up to 250
// expected blocks 1 to 15 % of a step gained, five 1 % lost; from 256 on 4 to 22 % lost, two equal; the blocks of a lone expert are known.  300 tokens on 4 experts of 1280 x
// 5120: fc1, 307 blocks, 8 us lost of 64, fc2, 77, 5 gained; 100 on one of 5120 x 20480, 320 and 80 blocks, 18 lost and 25 gained of 197; 997 bf16 tokens, two
// of 16 of 768 x 3072, fc2, 227 blocks, 31.9 -> 27.3.  Below 18 MB of weights 0.92 to 1.0 times as fast a step: 300 tokens, two of 8 of 512 x
// 2048 36.1 -> 38.4.)
static bool ring_long(const GemmArgs &p, int bm)
{
    return (long)p.E * p.K * p.N >= kLongRingWeights && expected_row_tiles(p.R, p.E, bm) * ((p.N + 127) / 128) <= (p.E > 1 ? 250 : 256);
}

// 32-row tiles of a register-fed block.
// 64-row tiles also for taller experts where a third block per CU pays more than halving the
// dequantisation does: short K loops (the prologue and epilogue of a block then overlap the loops of
// two others, not of one), and 8-bit weights up to 256 rows per expert (their 128-row tile has
// registers for one set of weights in flight only)
static int tile_height(const GemmArgs &p, int bits, int mean)
{
    return mean <= 32 ? 1 : (mean <= 64 || p.K <= 2048 || (bits == 8 && mean <= 256)) ? 2 : 4;
}

// ... and of one that takes the ring's place (ring_rows_for): there are few tiles
static int tile_height_for(const GemmArgs &p, int bits, int mean)
{
    return p.indexed && mean <= 100 && ring_rows(p, bits, mean) ? 1 : tile_height(p, bits, mean);
}

// Whether bf16 rows of a channel-scaled layer meet bf16 codes as they are (codes_to_bf16) instead of being converted to scaled FP16 ahead of
// each GEMM.  Converting costs two launches and reads and writes x and h at 5 TB/s, of which 3 us and that much show; bf16 codes cost eight vector instructions more for
// eight of them every time a row tile converts them, and how much of that shows depends on what bounds the kernel (us per 1e9 codes over the chip): little in blocks of few rows,
// which wait for weights, least with 8-bit ones, of which there are twice as many bytes, unless a block has its compute unit to itself; most in 128-row tiles, where matrix and
// vector work share the chip's power.
// (9719 drawn layers, 100 to 16000 tokens: 0.11 % slower on average than the better way for each, at most 9 %; one figure for every kernel 0.23 % and 17 %; always converting
// 6.7 %, never 0.7 % and 17 %.  us a step, converted / as they are: 1906 tokens, one of 16 experts of 768 x 3072 57.1 / 50.5; 609, two of 8, 8-bit, 61.4 / 57.3; 10420, two of 64,
// 8-bit, 347 / 309; left to the conversion: 713, one of 8 of 4096 x 16384 267 / 312; 490, one of 16 of 2048 x 8192 97.7 / 111.2; 3862, one of 8 of 4096 x 16384, 8-bit, 1129 / 1211, 7 133 / 149.)
// indexed: as GemmArgs has it; the tiles are those that launch_tiled_gemm takes (with those of permuted copies for rows through the index, 831, one of 64 of 1024 x 4096 91.2,
// now 88.5; 1411, one of 128 of 1024 x 2048 103.9 / 98.3; 327, one of 8 of 2048 x 8192, converted now, 77.4 / 74.5; nineteen such layers, none slower).
bool bf16_codes_pay(int R, int tokens, int E, int d, int F, int bits, bool indexed)
{
    static const double ring_us[2][3] = {{16, 16, 24}, {0, 4, 0}}, tile_us[2][3] = {{7, 16, 27}, {0, 8, 21}};     // [8-bit][16, 32, 64 rows], [32, 64, 128 rows]
    GemmArgs p{};
    p.E = E, p.R = R, p.indexed = indexed;
    const int mean = (R + E - 1) / E;
    double us = 0;
    for (int fc = 0; fc < 2; ++fc) {
        p.K = fc ? F : d, p.N = fc ? d : F;
        const int ring = ring_rows_for(p, bits, SCALE_CHANNEL_BF16, mean), bm = ring ? ring : 32 * tile_height_for(p, bits, mean);
        const double tiles = expected_row_tiles(R, E, bm);
        us += tiles * p.K * p.N * 1e-9 * (ring ? ring_us[bits == 8][bm / 32] : tile_us[bits == 8][bm / 64]);
        if (bits == 8 && ring == 16 && tiles * ((p.N + 127) / 128) <= 256) us += p.K * 4e-4;      // nothing beside the lone block's chain
    }
    return us <= 3.0 + 4.0 * ((double)R * F + (double)tokens * d) / 5e6;
}

// Blocks that hold rows when launch_tiled_gemm takes this GEMM, under uniform routing; infinitely many where its tiles do not sort.
double row_tile_blocks(const GemmArgs &p, int bits, int smode)
{
    const int mean = (p.R + p.E - 1) / p.E, ring = ring_rows_for(p, bits, smode, mean), tm = tile_height_for(p, bits, mean);
    if (ring) return expected_row_tiles(p.R, p.E, ring) * ((p.N + 127) / 128);
    return smode == SCALE_GROUP_ACC && tm > 1 ? INFINITY : expected_row_tiles(p.R, p.E, 32 * tm) * ((p.N + 255) / 256);
}

int launch_tiled_gemm(const GemmArgs &p, int bits, int smode, hipStream_t s)
{
    // row-tile height from the mean rows per expert (the offsets themselves stay on the device)
    const int mean = (p.R + p.E - 1) / p.E;
    const int bm = ring_rows_for(p, bits, smode, mean);
    note_kernel(bm ? "grouped_gemm_ring_kernel" : "grouped_gemm_kernel");
    if (bm) {
        const long slots = (long)p.R / bm + (p.E < p.R ? p.E : p.R);
        const long wgs = (slots * ((p.N + 127) / 128) + kXcds - 1) / kXcds * kXcds;      // upper bound of the work items, whole rounds of XCDs
        if (wgs > 0x7fffffffL) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: %ld workgroups exceed one launch", wgs);
        GemmArgs q = p;
        q.ring_long = bits == 8 && bm == 64 && ring_long(p, bm);
        (bits == 4 ? launch_ring_4 : launch_ring_8)(q, smode, bm, dim3((unsigned)wgs), s);
        return check_launch("moe_grouped_ffn_wq (gemm)");
    }
    int tm = tile_height_for(p, bits, mean);
    if (smode == SCALE_GROUP_ACC && tm > 1) tm = p.gate_idx ? 1 : 2;         // (64-row tiles of group sums do not sort)
    const long most = p.R;                                      // experts that can hold rows
    const long ncol = (p.N + 255) / 256;
    // Tiles may be lower than the kernel's 32 * tm rows (it skips row tiles that hold no rows): with few
    // column blocks the launch is a handful of rounds of 512 blocks (two per CU), and 96-row tiles
    // can fill the last round better than 128-row tiles leave it.  Cost model: rounds x tile height,
    // lower tiles charged 6 % per step down for streaming the weights more often.
    int units = tm;
    if (tm == 4) {
        double best = 0;
        for (int u = 4; u >= 2; --u) {
            const long items = ((long)p.R / (32 * u) + (p.E < most ? p.E : most) / 2) * ncol;
            const double cost = (double)((items + 511) / 512) * u * (1.0 + 0.06 * (4 - u));
            if (u == 4 || cost < best) { best = cost; units = u; }
        }
    }
    GemmArgs q = p;
    q.tile_units = units;
    const long slots = (long)p.R / (32 * units) + (p.E < most ? p.E : most);
    if (slots == 0) return MOE_OK;
    const long wgs = (slots * ncol + kXcds - 1) / kXcds * kXcds;   // upper bound of the work items, whole rounds of XCDs
    if (wgs > 0x7fffffffL) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: %ld workgroups exceed one launch", wgs);
    dim3 grid((unsigned)wgs);
    const bool exact = smode == SCALE_GROUP_ACC || smode == SCALE_GROUP_SPLIT;
    if (bits == 4) (exact ? launch_tiled_4_exact : launch_tiled_4)(q, smode, tm, grid, s);
    else (exact ? launch_tiled_8_exact : launch_tiled_8)(q, smode, tm, grid, s);
    return check_launch("moe_grouped_ffn_wq (gemm)");
}

}  // namespace moe
