// Host-side planning arithmetic of libthi: how work is dealt to workgroups and how large the workspace
// regions are.  No kernels and no HIP calls here, so that this file and api.hip can also be built for the
// host alone (with stand-ins for the kernel launchers) and run under the sanitizers on a machine without
// a GPU.
#include "thi_internal.h"

namespace thi {

// ---- decode kernels ------------------------------------------------------------------------------
size_t skinny_handover_bytes() { return (size_t)SK_MAX_GRID * SK_SLOT_WORDS * sizeof(unsigned); }

// K < 1024, up to 32 tokens: slabs of 16 rows over all of K, or the stream-K kernel?  A compute unit takes its slabs one after the
// other, each with its own reduction and epilogue, the stream-K kernel 128 rows at a time and a hand-over: up to five slabs a CU,
// four behind an RMSNorm; with K <= 256, where there is little to stream, four and two (plain, others).  Slabs against stream-K over
// 420 calls of 1..32 tokens: 0.49-0.72 of its time with one or two slabs a CU and K > 256, 0.81-0.95 (up to 1.04) at the line; beyond
// it 1.02-1.4 (gate/up and RMSNorm kinds with K <= 256: 3 slabs 1.05, 4 1.22, 5 1.4).
bool rowslab_small_ok(int N, int K, int epilogue, int num_cus)
{
    if (K >= 1024) return false;
    const int rows = is_swiglu(epilogue) ? 8 : 16, most = K > 256 ? (is_rms(epilogue) ? 4 : 5) : epilogue == EPI_PLAIN ? 4 : 2;
    return ((long)N + rows - 1) / rows <= (long)most * num_cus;
}

// Row blocks: the outputs (rows of W, gate/up pairs for SwiGLU) are dealt to the workgroups in equal contiguous
// blocks; a block is T tiles of 16 rows in flight per pass over K (Sec. III-B.2: split the work along N).
RowBlockPlan plan_rowblock(int N, int epilogue, int num_cus, int ksplit)
{
    RowBlockPlan p;
    const int out_per_tile = is_swiglu(epilogue) ? 8 : 16;
    if (ksplit < 1) ksplit = 1;
    int groups = num_cus / ksplit;          // row blocks: ksplit workgroups each
    if (groups < 1) groups = 1;
    int per_wg = (N + groups - 1) / groups;
    if (!is_swiglu(epilogue)) per_wg = (per_wg + 1) & ~1;      // rotary pairs (n, n + 1) stay in one block
    p.per_wg = per_wg;
    p.ksplit = ksplit;
    p.grid = ((N + per_wg - 1) / per_wg) * ksplit;
    p.tiles = (per_wg + out_per_tile - 1) / out_per_tile;
    p.passes = (p.tiles + 5) / 6;
    const int per_pass = (p.tiles + p.passes - 1) / p.passes;
    p.T = per_pass < 2 ? 2 : per_pass;
    return p;
}

bool rowblock_split_ok(int N, int K, int epilogue, int num_cus, int ksplit)
{
    if (ksplit < 2 || ksplit > ROWBLOCK_MAX_SPLIT || epilogue != EPI_PLAIN) return false;
    if (((K + 127) >> 7) < 8 * ksplit) return false;           // every wave of every share gets k of its own
    const RowBlockPlan p = plan_rowblock(N, epilogue, num_cus, ksplit);
    // one pass (the hand-over happens once, at the end), one workgroup per compute unit at most, and a
    // slot / a counter per workgroup / block within the workspace
    return p.passes == 1 && p.grid <= num_cus && p.grid <= SK_MAX_GRID && p.T * 512 <= SK_SLOT_WORDS;
}

// The single-launch decode MLP: which shapes the one fused kernel that is built serves.
bool mlp_fused_ok(int M, int H, int I, int epilogue_up, int num_cus, int ksplit_down)
{
    if (M < MLP_FUSED_MIN_M || M > 32 || H < 1024 || H > ROWSLAB_MAX_K || I < 1024 || I > ROWSLAB_MAX_K) return false;
    if (epilogue_up != EPI_SWIGLU && epilogue_up != EPI_RMSNORM_SWIGLU) return false;
    if (epilogue_up == EPI_RMSNORM_SWIGLU && H > 24576) return false;      // gamma in LDS beside the two phases' ~104 KiB
    if (!rowblock_split_ok(H, I, EPI_PLAIN, num_cus, ksplit_down)) return false;
    const RowBlockPlan up = plan_rowblock(I, epilogue_up, num_cus, 1), down = plan_rowblock(H, EPI_PLAIN, num_cus, ksplit_down);
    // the one pair of block shapes that is built: six gate/up tiles and four down tiles in flight, one pass each
    return up.passes == 1 && up.T == 6 && up.grid <= num_cus && down.passes == 1 && down.T == 4 && down.grid <= num_cus &&
           num_cus <= MLP_MAX_GRID;
}

// ---- prefill GEMM ----------------------------------------------------------------------------------
size_t gemm_partial_bytes() { return (size_t)GEMM_MAX_GRID * 2 * 128 * 128 * sizeof(float); }

// The few-token kernel: BN rows per tile and S k ranges per tile, at most one workgroup per compute unit (a second round
// starts with an empty pipeline: 13B gate/up at 72 tokens as 432 tiles 68.8 us, the GEMM 63.8), not above K = 24576 (the
// 70B down projection measured 2-4 % behind the kernels it would replace).
//
// Which (BN, S): the smallest of a time in microseconds and KB per workgroup that was fitted to ~400 measured points with tiles of
// 32..96 rows: 4.2 us fixed, 24 ns a KB of weights, 13 ns a KB of activations, 93 ns a stage; sharing a tile 1 us, 32 ns a
// KB of its partial tiles and 2 / 3 us more with 80 / 96 rows.  On 304 problems (36000 x 128 .. 500 x 18400, 33..128 tokens, all
// seven heights, ~1750 points) the pick is 0.8 % slower than the best measured one on average, 3.5 % at the 95th percentile.
// What it takes, for the comparison with other kernels: that fit is 10 % low there (13 % with 80 and 96 rows, 17 % with 112), since
// it has no term for a tile's own work -- its MFMAs and LDS reads per stage, the meeting of the k groups, the
// epilogue -- so the price is a second fit to the 1750 points, within 9 % (rms) with no such trend: 2.8 us, 0.4 ns an element
// of the tile, 14 ns a KB of weights, 7 ns a KB of activations, 252 ns and 0.025 ns an element for each stage; sharing 1.6 us and 25 ns a KB
// of partial tiles.  (It picks no better: 1.0 %, 5.4 %.)
// Tiles of 80..144 rows are for shapes that smaller ones cut into more tiles than there are compute units, or into few
// enough that one more share would not fit (against the kernels that served them): 19968 x 6656 at 128 tokens 75.3 -> 62
// us (80 rows), 6656 x 17920 at 128 70.7 -> 59 (80, S = 3), gate/up 2 x 13824 x 5120 at 72 62.7 -> 55 (112), gate/up
// 2 x 17920 x 6656 at 64 107.7 -> 79 (144).  With more rows shared tiles only lose (15360 x 5120 at 72 tokens: 52 us with
// two shares of 144 rows, 35.5 with 64).
namespace {

// The same kernel with a token tile of 32, for up to MID_DECODE_M tokens.  S shares of K, so that there are num_cus / S tiles, each of
// equally many outputs (in fours), in the least tile that holds them; the S of the smallest modelled time: 4.15 us fixed,
// 19 ns a row of the tile; for each stage of 128 k 102 ns, 6.3 ns a row of weights and 2 ns a token, or what
// 8 TB/s give if that is longer; sharing 0.8 us and 0.117 ns a row, token and share.  Fitted to 430 points on 38 calls
// (4..32 tokens, 1536 x 4096 .. gate/up 2 x 28672 x 8192): the pick is 1.1 % slower than the best measured on average; the price is 7 % off (rms).  No tiles
// above 176 rows: those leave room for two stages, which left gate/up 2 x 28672 x 8192 at 147 us against 140 with the row blocks.
//
// rotate: workgroups that walk the same k at the same time ask for addresses a row's length apart, and where those agree in their low bits they
// fall on few of the memory's channels.  Spreading the tiles' starts over k costs what the L2 shared of the activations.  Tiles that have all of K and 48 rows
// or more: where rows are a multiple of 4 KiB or do not start on a line (at 20-32 tokens 12288 x 4096 19.4 -> 17.5 us, gate/up 2 x 11008 x 4096 36.5 -> 29.9,
// 19 x 2 x 13472 x 2336 28.8 -> 25.0, 10 x 2 x 6832 x 6560 34.0 -> 31.5; 2 x 13824 x 5120 44.5, 45.2; 2 x 12000 x 7168 52.6, 54.1).  The others: gate/up where rows are a
// multiple of 4 KiB; plain kinds by measurement from K = 8192 on, whatever the row's length (8192 x 8192 26.8 -> 24.1 with 32 rows; 4096 x 11008, rows of
// 21.5 KiB, 20.0 -> 18.7), and not below (6656 x 6656 with 32 rows 17.2, 18.6; 7136 x 1448 7.4, 7.8).
// alone: tiles that do, have all of K and rows that start on a line take less of a compute unit than the fit says (8192 x 8192 at 20 tokens: two shares of 64 rows
// 25.3, whole tiles of 32 rows 21.8; 10240 x 8192 29.5, 27.8).
MidPlan plan_mid_decode(int M, int N, int K, int epilogue, int num_cus)
{
    MidPlan best{0, 0, 0, 0.0, 0, false, 1, M};
    if (K > ROWSLAB_MAX_K || num_cus > SK_MAX_GRID) return best;
    const bool swiglu = is_swiglu(epilogue);
    const int rows_per = swiglu ? 2 : 1, ktiles = (K + 127) / 128;
    const double stream = (double)rows_per * N * K * 2.5e-7;      // (us: 8 TB/s)
    for (int S = 1; S <= 8 && (S == 1 || S * 4 <= ktiles); ++S) {
        const int groups = num_cus / S;
        if (groups < 1) break;
        const long per = ((long)N + 4L * groups - 1) / (4L * groups) * 4, rows = per * rows_per;
        int BN = 0;
        for (int b : {32, 48, 64, 80, 96, 112, 128, 144, 176})
            if (b >= rows) { BN = b; break; }
        if (!BN) continue;
        const int kt = (ktiles + S - 1) / S;
        const bool rotate = (S == 1 && BN >= 48 && (K % 2048 == 0 || K % 64 != 0)) || (swiglu ? K % 2048 == 0 : K >= 8192), alone = S == 1 && rotate && K % 64 == 0;
        const double cu = kt * (0.0063 * rows + (alone ? 0.0010 * M + 0.060 : 0.0020 * M + 0.102));
        const double us = 4.15 + (cu > stream ? cu : stream) + 0.019 * BN + (S > 1 ? 0.8 + 1.17e-4 * S * BN * (M > 8 ? M : 8) : 0.0);
        if (best.BN && us >= best.us) continue;
        best = MidPlan{BN, (int)((N + per - 1) / per), S, us, (int)per, rotate, 1, M};
    }
    return best;
}

}  // namespace

// rotate above 32 tokens: gate/up with K = 4096 at 72 tokens 41.2 -> 38.7 us; plain shapes lose (8192 x 8192 32.3 -> 34.6).
MidPlan plan_mid(int M, int N, int K, int epilogue, int num_cus)
{
    MidPlan best{0, 0, 0, 0.0, 0, false, 1, M};
    if (M <= MID_DECODE_M) return plan_mid_decode(M, N, K, epilogue, num_cus);
    if (M > 128 || K > 24576) return best;
    const long V = is_swiglu(epilogue) ? 2L * N : N;      // (more than an int holds from N = 2^30 on)
    const int ktiles = (K + 127) / 128, BM = M > 96 ? 128 : M > 64 ? 96 : 64;
    double least = 0.0;
    for (int BN : {32, 48, 64, 80, 96, 112, 144}) {
        if (BN > (M > 96 ? 80 : M > 64 ? 112 : 144)) continue;  // (more spill registers)
        const long tiles = (V + BN - 1) / BN;
        for (int S = 1; S <= (BN > 96 ? 1 : 16) && tiles * S <= num_cus && (S == 1 || S * 4 <= ktiles); ++S) {
            const int per = (ktiles + S - 1) / S;
            const double w = BN * per * 0.256, x = M * per * 0.256;
            const double us = 4.2 + 0.024 * w + 0.013 * x + 0.093 * per +
                              (S > 1 ? 1.0 + 0.032 * S * BN * M * 0.004 + (BN == 96 ? 3.0 : BN == 80 ? 2.0 : 0.0) : 0.0);
            if (best.BN != 0 && us >= least) continue;
            least = us;
            best = MidPlan{BN, (int)tiles, S, 2.83 + 4.0e-4 * BN * BM + 0.0139 * w + 0.0073 * x + per * (0.252 + 2.5e-5 * BN * BM) +
                                                  (S > 1 ? 1.6 + 1.0e-4 * S * BN * M : 0.0), is_swiglu(epilogue) ? BN / 2 : BN, is_swiglu(epilogue) && K % 2048 == 0, 1, M};
        }
    }
    // The outputs dealt evenly over the units that one round has (in fours), in the same tiles: fewer rows each, and none idle (gate/up 2 x 11008 x 4096 at
    // 72 tokens: 251 workgroups of 44 pairs, not 230 of 48).  Not where the tiles fill less than two thirds of them: each more reads the activations again (36 x 376 x
    // 2448 as 47 tiles of 8 rows in 5 ranges 7.7 us, as 12 of 32 rows 7.2; 39 x 352 x 7328 9.8, 9.2).
    if (best.BN && best.tiles * best.S * 3 >= num_cus * 2) {
        const int groups = num_cus / best.S;
        const long per = ((long)N + 4L * groups - 1) / (4L * groups) * 4;
        if (per < best.per) {
            best.per = (int)per;
            best.tiles = (int)((N + per - 1) / per);
        }
    }
    return best;
}

namespace {

// Time model (microseconds) of running `tiles` tiles of BN x BM on `grid` workgroups.
//   whole tiles only : ceil(tiles / grid) rounds;
//   shared remainder : floor(tiles / grid) whole rounds; the ragged remainder is cut along K and a second
//                      pass (one more launch, the partial tiles' round trip through memory) adds the parts.
// How the remainder is cut depends on what bounds the kernel.  With several token tiles it is the matrix
// cores, fed through the L2: workgroups on neighbouring tiles must walk the same k range at the same
// time or the panels they share are fetched once per workgroup (measured: a 30B-shaped down projection,
// 208 tiles of 256x256 on 256 workgroups in equal contiguous shares, ran HBM-bound at 585 us against 485
// us for whole tiles on 208 workgroups).  So every remainder tile is cut into the same `parts` = grid /
// remainder equal k ranges (whole tiles if that is 1) -- also with a single token tile of 256, whose
// activation panel is shared by every workgroup and too large for an L2 (measured on the 30B-shaped down
// projection at M = 256: 88 us against 97-113 us with contiguous shares), unless equal ranges would leave
// more than a tenth of the workgroups idle (7B-shaped gate/up at M = 160: 86 tiles x 2 ranges on 256
// workgroups, 81 against 75 us; 13B-shaped, 108 tiles x 2: 106 against 97 us).  The few-token configurations (one token tile of at most 128) are bound
// by their weight traffic, every weight panel is read exactly once whatever the cut, and equal contiguous
// shares (parts = 0) keep every workgroup busy.
// A workgroup's speed by configuration, fitted to measurements of every configuration and cut on projections of the
// 7B..70B shapes and some odd ones at M = 200..2048 (weight copies rotated so that they come from HBM): 256x256 tiles
// 5.4 TFLOP/s + 6 us per tile, 224 / 192 / 160 rows x 256 tokens 4.75 / 4.7 / 4.4 + 6 us, 128 rows x 256 tokens 4.6 TFLOP/s + 5 us, 128x128 tiles two per CU 1.95 TFLOP/s + 6 us,
// 128x128 one per CU (stages of 64 or 128 k) 3.6 TFLOP/s + 4 us; the second pass 8 us (a launch and its latencies: 5 us made
// 333 x 512 x 1376 cut 12 tiles in 21 ranges, 21.2 us against 16.1 whole) + its bytes at ~8 TB/s (they are still
// in the caches).  A share of a tile pays the fixed time in full, however small it is: priced by the share, as equal
// contiguous shares were, it made cut tiles look up to 5 us cheaper than they are (129 x 4096 x 11008 as 32 tiles of 128 rows x
// 256 tokens in 8 ranges 41.5 us, as 64 tiles of 128x128 in 4 ranges 36.6).  Tokens past M are loaded from one row, which the caches hold: tiles
// of 128 tokens save a tenth of the empty part's work (64 tiles in 4 ranges 36.3 us at 129 tokens, 38.7 at 203, 41.2 at 256;
// with a quarter, gate/up 300 x 11008 x 4096 goes to 128x128 tiles, 95 us against 86 with 192 rows).
// On 282 problems of 129..1500 tokens (the projections of the 7B..70B shapes and random ones), every configuration measured, the
// pick is 1.6 % slower than the best on average, 8 % at the 95th percentile.
struct Schedule {
    int sk_tiles;      // tiles cut along K (0: whole tiles only)
    int parts;         // equal k ranges per shared tile; 0 = equal contiguous shares across tile boundaries
    double us;
};

Schedule plan_schedule(int M, int tiles, int tiles_m, int grid, int BN, int BM, int ktiles, int K, double wg_tflops, double tile_fixed_us, bool cut, double second_pass_us)
{
    double work_us = 2.0 * BN * BM * (double)K / (wg_tflops * 1e6);
    if (BM == 128) work_us *= 1.0 - 0.1 * (1.0 - (double)M / ((double)tiles_m * BM));
    if (tiles_m == 1) {      // every weight panel is read by one workgroup only: its traffic is a second bound
        const double stream_us = (double)BN * K * 2.0 / (6.0e6 / grid);
        work_us = work_us > stream_us ? work_us : stream_us;
    }
    const double tile_us = tile_fixed_us + work_us;
    const int rem = tiles % grid, full = tiles / grid;
    const double tile_bytes = (double)BN * BM * 4.0;
    const double whole = (double)((tiles + grid - 1) / grid) * tile_us;
    if (rem == 0 || !cut) return Schedule{0, tiles_m == 1 ? 0 : 1, whole};
    int parts = grid / rem;
    if (parts > ktiles) parts = ktiles;
    // One token tile: equal contiguous shares for the few-token configurations, and for a 256-token tile
    // when equal ranges would leave more than a tenth of the workgroups idle.
    if (tiles_m == 1 && (BM <= 128 || (long)rem * parts * 10 < (long)grid * 9)) {
        const double shared = (double)full * tile_us + tile_fixed_us + (double)rem / grid * work_us + second_pass_us + (double)(grid + rem) * tile_bytes * 2.0 / 4.0e6;
        return shared < whole ? Schedule{rem, 0, shared} : Schedule{0, 0, whole};
    }
    if (parts < 2) return Schedule{0, 1, whole};
    // (a range takes 4 us at least: 554 x 512 x 1376 as 20 tiles in 11 ranges 17.7 us, whole 13.4; fewer than eight tiles'
    // worth of 128x128 are better cut in any case; counted in tiles of their own size, five of 256 tokens passed for few: gate/up 219 x 312 x 2304 24.8 us, 19.7
    // as ten of 128x128)
    const double range_us = full == 0 && (long)tiles * BN * BM >= 8L * 128 * 128 && work_us < 4.0 * parts ? 4.0 : work_us / parts;
    const double shared = (double)full * tile_us + tile_fixed_us + range_us + second_pass_us +
                          (double)rem * parts * tile_bytes * 2.0 / 8.0e6;
    return shared < whole ? Schedule{rem, parts, shared} : Schedule{0, 1, whole};
}

}  // namespace

// The configurations: tile, k per stage, cut along K?, ragged K?, workgroups per CU, TFLOP/s of a workgroup and fixed time per tile (us)
GemmTile gemm_tile(int config)
{
    switch (config) {
    case GEMM_FEW64: return GemmTile{128, 64, 128, true, false, 1, 900.0 / 256, 4.0};      // one token tile: bound by the weight stream anyway
    case GEMM_FEW128: return GemmTile{128, 128, 64, true, true, 1, 3.6, 4.0};      // (above 128 tokens too: plan_gemm)
    case GEMM_FEW256: return GemmTile{256, 128, 64, true, false, 1, 900.0 / 256, 4.0};
    case GEMM_ONE: return GemmTile{128, 256, 64, true, false, 1, 900.0 / 256, 4.0};        // (the kernel of GEMM_TALL)
    case GEMM_BIG: return GemmTile{256, 256, 64, true, true, 1, 5.4, 6.0};
    case GEMM_R224: return GemmTile{224, 256, 64, false, false, 1, 4.75, 6.0};
    case GEMM_R192: return GemmTile{192, 256, 64, true, false, 1, 4.7, 6.0};
    case GEMM_R160: return GemmTile{160, 256, 64, false, false, 1, 4.4, 6.0};
    case GEMM_TALL: return GemmTile{128, 256, 64, true, false, 1, 4.6, 5.0};
    case GEMM_DEEP: return GemmTile{128, 128, 128, true, true, 1, 3.6, 4.0};
    case GEMM_SMALL: return GemmTile{128, 128, 64, true, true, 2, 1.95, 6.0};
    default: return GemmTile{};
    }
}

namespace {

GemmPlan plan_config(int config, int M, int N, int K, int epilogue, int num_cus)
{
    const GemmTile t = gemm_tile(config);
    const int per_tile = is_swiglu(epilogue) ? t.BN / 2 : t.BN;
    GemmPlan p{};
    p.config = config;
    p.tiles_m = (M + t.BM - 1) / t.BM;
    p.tiles = (N + per_tile - 1) / per_tile * p.tiles_m;
    p.ktiles = (K + t.GK - 1) / t.GK;
    long grid = (long)num_cus * t.per_cu;        // workgroups that fit, and that the workspace has partial tiles for
    const long most = (long)GEMM_MAX_GRID * 128 * 128 / (t.BN * t.BM > 128 * 128 ? 256 * 256 : 128 * 128), units = (long)p.tiles * p.ktiles;
    if (grid > most) grid = most;
    if (grid > units) grid = units;
    p.grid = (int)grid;
    // The second pass of 128x128 tiles a shade less, above 128 tokens.  One per unit: 928 x 1073 x 3072 as 72 tiles in three ranges 18.9 us, whole 23.4; 465 x
    // 1057 x 2944 17.0, 21.8; gate/up 719 x 3872 x 4344 a round and 110 tiles in two ranges 76.9, two tiles per unit 91.7.  Two per unit: the price between
    // leaves 606 x 3961 x 5024 to whole tiles (41.2, in ranges 52.0) and 129 x 5603 x 5696 in five ranges.  With 7.85 for the larger tiles too, gate/up 204 x 12936 x
    // 9856 cut its 203 tiles of 256 tokens (172, whole 144) and 153 x 4474 x 6400 ran tiles of 256 tokens (39.2, here 30.4).
    const double second_pass_us = M <= 128 || t.BN != 128 || t.BM != 128 ? 8.0 : t.per_cu == 1 ? 7.85 : 7.92;
    const Schedule s = plan_schedule(M, p.tiles, p.tiles_m, p.grid, t.BN, t.BM, p.ktiles, K, t.wg_tflops, t.fixed_us, t.cut, second_pass_us);
    p.sk_tiles = s.sk_tiles;
    p.parts = s.parts;
    p.us = s.us;
    // No more workgroups than have work, and in whole rounds as many in each: consecutive workers share an XCD, so the ones without work
    // would be the last XCDs', whose L2 and whose way to memory then idle while the others queue (333 x 5001 x 1384 as 120 tiles: the first four
    // XCDs only).  203 x 12288 x 4096 41.5 -> 40.1 us, 333 x 5001 x 1384 22.4 -> 21.3, 1024 x 12288 x 4096 as 192 tiles of 256 rows 105 -> 98,
    // 1024 x 4096 x 4096 as 88 tiles of 192 rows in 2 ranges 57.7 -> 51.7, 512 x 27648 x 5120 as 432 tiles of 128 rows 149.6 -> 148.0.
    if (p.sk_tiles == 0 && p.tiles > 0) {
        const int rounds = (p.tiles + p.grid - 1) / p.grid;
        p.grid = (p.tiles + rounds - 1) / rounds;
    } else if (p.sk_tiles == p.tiles && p.parts >= 1) {
        p.grid = p.tiles * p.parts;
    }
    return p;
}

GemmPlan few_token_plan(const MidPlan& m)
{
    GemmPlan p{};
    p.config = GEMM_MID;
    p.mid = m;
    p.tiles = m.tiles;
    p.grid = m.tiles * m.S;
    p.us = m.us;
    return p;
}

}  // namespace

GemmPlan plan_gemm(int M, int N, int K, int epilogue, int num_cus)
{
    const bool even_k = K % 64 == 0;                 // else: the configurations that take a ragged K
    const int per128 = is_swiglu(epilogue) ? 64 : 128;
    const long t128 = ((long)N + per128 - 1) / per128;
    if (M <= 128) {
        // Few tokens: one token tile, the weights are read once and the kernel is bound by how many
        // bytes a CU keeps in flight: three stages of 128 rows x 128 k against 64 tokens (K a multiple of
        // 128), else four of 128 rows x 64 k against 128 tokens.  With far fewer tiles than workgroups every
        // tile is cut along K, and the second pass costs by the partial tiles' bytes, (workgroups +
        // tiles) x tile size: 128-row tiles halve them against 256-row tiles (7B-shaped O projection at
        // M = 128: 24.8 -> 18.5 us, gate/up 61 -> 53; second pass alone 8.5-9.7 us with 256 rows).  With
        // many more tiles than workgroups (70B-shaped gate/up: 448) the 256-row tile's smaller share of
        // activation staging wins instead (188 against 230 us), and with a ragged K two workgroups per CU (gate/up
        // 50 x 25832 x 176: 9.1 against 11.6 us; 100 x 40000 x 776 31.2 against 33.4).
        const int config = M <= 64 && K % 128 == 0 ? GEMM_FEW64 :
                           !even_k ? (t128 <= num_cus ? GEMM_FEW128 : GEMM_SMALL) :
                           t128 <= num_cus + num_cus / 8 ? GEMM_FEW128 : GEMM_FEW256;
        // The few-token kernel where its modelled time is the smaller one, or with tiles of up to 80 rows up to a fifth more: the
        // other model is low for large problems (10240 x 8192 at 128 tokens 55.8 us against 50.3 here), plan_mid's a little for
        // wide tiles and small K (61 x 28750 x 640 12.9 us, here 11.4).  On 813 problems of 33..128 tokens, both measured, the pick is
        // 0.2 % slower than the better one on average (one factor of 1.0 for all: 1.5 %).
        const MidPlan mp = plan_mid(M, N, K, epilogue, num_cus);
        if (mp.BN && (M <= MID_DECODE_M || mp.us < (mp.BN <= 80 ? 1.2 : 1.05) * plan_config(config == GEMM_FEW256 ? GEMM_FEW128 : config, M, N, K, epilogue, num_cus).us)) {
            return few_token_plan(mp);
        }
        return plan_config(config, M, N, K, epilogue, num_cus);
    }
    // 129..256 tokens and about as many 128-row tiles as workgroups (0.65..1.2 x: the gate/up shapes):
    // one token tile of 256 against 128 rows, so that the weights are read once and few tiles are cut
    // (7B-shaped gate/up at M = 192: 74.9 -> 67.4 us, 13B 98.9 -> 94.2, 30B 161 -> 152).  With fewer tiles
    // the 128 KiB partial tiles of the workgroups that share one cost more than reading the weights twice
    // (7B-shaped O projection 22.5 -> 31 us), with more the 256-row tile wins: both stay with the rule below.
    if (even_k && M <= 256 && t128 * 20 >= (long)num_cus * 13 && t128 * 5 <= (long)num_cus * 6)
        return plan_config(GEMM_ONE, M, N, K, epilogue, num_cus);
    // Several token tiles: the configuration with the smallest modelled time.  128 rows x 256 tokens halves the granularity
    // of the 256x256 tile where that leaves CUs idle (512 x 15360 x 5120: 120 tiles cut in two and a second pass 92.4
    // us, 240 whole tiles 87.8; 1500 x 4096 x 4096 68 -> 63), the four-stage 128x128 one where that still does
    // (300 x 12288 x 4096: a round and 32 tiles in 8 ranges 58 us, two per CU 70).  224, 192 and 160 rows x 256 tokens are
    // for the counts in between, where one of them nearly fills whole rounds (against the best of the others): 224 rows
    // 2048 x 6656 x 17920 437 -> 405 us, 2048 x 6656 x 6656 169 -> 160; 192 rows gate/up 512 x 22016 x 4096 107 -> 95.5,
    // 300 x 22016 x 4096 100 -> 85, 1024 x 12288 x 4096 110 -> 99; 160 rows 2048 x 5120 x 13824 286 -> 250, 2048 x 5120 x
    // 5120 118 -> 99, 512 x 19968 x 6656 150 -> 132, 1024 x 10240 x 8192 170 -> 152.  Not where the 256-row tile fills its
    // rounds as well: per flop they read more operand bytes (gate/up 2048 x 57344 x 8192 with 224 rows 1625 us, 1505).
    // 128x128 tiles, one workgroup per CU: stages of 64 k, four of them (FEW128), or of 128 k, three and two (DEEP)?  A load of 128 k
    // asks for pairs of lines, and where the rows do not start on a line (a ragged K) for three lines in the place of four; but K is
    // rounded up to 128, and its prologue is longer.  512 x 5120 x 5120 51.4 -> 45.6 us, 900 x 9000 x 8008 197 -> 174, 200 x 9000 x
    // 2008 28.7 -> 24.6, 587 x 4984 x 3352 42.5 -> 36.9, gate/up 366 x 11008 x 4096 101.5 -> 95.6; 471 x 404 x 1472 11.3 with 64 k (12.9), and
    // two token tiles start spread over k there: 203 x 12288 x 4096 38.4 (39.8).  Fewer than eight tiles are cut into many ranges
    // and take 128 k (247 x 173 x 2048 16.5 -> 12.0).  The shortest K go to SMALL, whose prologue is the shortest (300 x 1054 x 320 6.1, 64 k 6.3, 128 k 7.8).
    const int tiles_m = (M + 127) / 128;
    const bool deep = K % 64 || (tiles_m * t128 < 8 && K >= 1024) || (K % 128 == 0 && (K >= 8192 || (tiles_m >= 3 && K >= 1024)));
    const bool shortest = K < (K % 64 ? 448 : 384);
    GemmPlan best = plan_config(GEMM_BIG, M, N, K, epilogue, num_cus);
    for (int c = GEMM_BIG + 1; c <= GEMM_SMALL; ++c) {
        if (!even_k && !gemm_tile(c).ragged) continue;
        GemmPlan p = plan_config(c == GEMM_DEEP && !deep ? GEMM_FEW128 : c, M, N, K, epilogue, num_cus);
        // (their price is above what they take with few ranges: 731 x 1513 x 6592 in three 29.9 us, 256x256 tiles 35.9; 253 x 2890 x 10816 33.1, 39.1)
        if (c == GEMM_DEEP && p.sk_tiles == p.tiles && K >= (tiles_m > 2 ? 4096 : 8192) && K <= 16384) p.us *= p.parts <= 4 && tiles_m > 2 ? 0.87 : 0.95;
        if (c == GEMM_DEEP && shortest) {        // (priced as those: SMALL's own price is that of two workgroups on a CU)
            const double us = p.us;
            p = plan_config(GEMM_SMALL, M, N, K, epilogue, num_cus);
            p.us = us;
        }
        // (whole rounds and a cut rest are no better than larger tiles at the same price: gate/up 488 x 4144 x 6656 70.4 us cut as 256x256, here 80.9)
        const double shade = p.sk_tiles == 0 || p.sk_tiles == p.tiles ? 0.0 : c == GEMM_DEEP ? 0.15 : c == GEMM_SMALL ? 0.08 : 0.0;
        if (p.us + shade < best.us) best = p;
    }
    // 128x128 tiles, whole, with the compute units that get none touching the weights ahead: where that leaves 48 and more, and a tile takes
    // no longer than its ranges and their second pass would.  Its time was fitted to 300 products of 8..208 tiles (8 % rms); a cut
    // schedule's price is above what it takes with few ranges (530 x 2688 x 2511, two ranges: 27 for 20.2 us), hence the factors.  Not for two token
    // tiles in many tiles with a K that has them start spread over k (228 x 12288 x 4096 40.1, 39.3 without) or a long one (166 x 8192 x
    // 28672 250, 214 without): the touching units then lag behind the few that share a weight row.  Gate/up never has so few tiles but for toy sizes.
    const long whole = (long)tiles_m * t128;
    if (!is_swiglu(epilogue) && !shortest && whole >= 8 && whole <= num_cus - 48 && K <= 16384 &&
        (tiles_m > 2 || whole <= num_cus / 2 || (!even_k && K < 2048))) {
        const double slope = even_k ? 0.0042 + 1.6e-5 * whole : 0.0052 + 1.9e-5 * whole;
        const double us = 5.0 + K * slope * (tiles_m == 2 ? 1.12 : 1.0);
        // (128x128 tiles whole without the touching: never faster)
        auto takes = [&](const GemmPlan& p) {
            return p.us * (p.sk_tiles == 0 ? (p.tiles == whole ? 2.0 : 0.95) : p.parts == 2 ? 0.78 : p.parts <= 4 ? 0.87 : 0.95);
        };
        const double cut = takes(plan_config(deep ? GEMM_DEEP : GEMM_FEW128, M, N, K, epilogue, num_cus)), other = takes(best) < cut ? takes(best) : cut;
        if (us < other) {
            best = plan_config(!even_k || (K % 128 == 0 && K >= 4096) ? GEMM_DEEP : GEMM_FEW128, M, N, K, epilogue, num_cus);
            best.sk_tiles = 0;
            best.parts = 1;
            best.grid = (int)whole;
            best.us = us;
            // (a quarter of the units is enough, and more ask for the same lines as often as the others where the weights come from the
            // last-level cache: 333 x 5001 x 1384 cold / from there: none 19.2 / 14.7 us, 136 16.0 / 15.1, 64 15.9 / 14.5; 200 x 9000 x 2008 24.5 /
            // 18.3, 20.9 / 19.9, 20.7 / 18.6)
            best.helpers = (num_cus - (int)whole < num_cus / 4 ? num_cus - (int)whole : num_cus / 4) / 8 * 8;
        }
    }
    return best;
}

// Above 128 tokens: the few-token kernel with several token tiles of 44..128 tokens each, where it is priced below the GEMM.  It finishes shared tiles
// itself, where the GEMM's 128x128 tiles need a second pass, it reads half as much from LDS per product as those, tokens past the last are not
// loaded, and outputs and tokens are dealt evenly: one round of tiles in S ranges, tiles * S just below the number of CUs.  The least of a modelled time: 2.5 us, 0.58 ns an
// element of the tile, 13.2 ns a KB of weights and 10.7 of activations, 113 ns and 17.5 ps an element for each stage of 128 k, 0.15 ns an output; sharing 1.9 us and
// 22 ns a KB of partial tiles.  Fitted to 2565 points on 350 products (129..700 tokens, 300..14000 x 256..11200), 7 % off (rms); the pick is 0.9 % slower than the best
// measured on average.  Taken where it is below 0.92 of the GEMM's price (that one is 9 % off): 450 random calls of 129..700 tokens, all kinds, with
// and without this kernel in turn: 0.82 of the time on average, those that keep the GEMM among them, the worst 1.02.  (The points were measured with the weights
// loaded non-temporally and a longer set-up; the kernel is 1-9 % faster than that.)  150 x 4096 x 4096 23.0 -> 18.5 us, 175 x 5120 x 5120 26.2 -> 25.2, 159 x 10783 x 6384 67 -> 56, 300 x 512 x 1376 12.6 -> 7.2, 258 x 304 x
// 8480 21.1 -> 11.7, RMSNorm-QKV 256 x 1536 x 512 14.3 -> 8.2; beyond ~12000 x 203 or 4096 x 500 outputs a round no longer holds them.  With 80 MB of weights
// and more whose rows start on a line the GEMM's tiles are as fast or faster, both being bound by the way into LDS (168 x 6656 x 6656 38.2, 43.8; 174 x 12288 x
// 4096 35.6, 38.0; 144 x 5120 x 13824 48.3, 50.5; 135 x 10240 x 8192 54.3, 54.2).
// rotate: where rows are a multiple of 4 KiB (135 x 4096 x 4096 18.0, 17.6).
namespace {

// (gemm_us: the GEMM's price)
MidPlan plan_mid_tiles(int M, int N, int K, int epilogue, int num_cus, double gemm_us)
{
    MidPlan best{0, 0, 0, 0.0, 0, false, 1, M};
    const int rows_per = is_swiglu(epilogue) ? 2 : 1, ktiles = (K + 127) / 128;
    if (M <= 128 || M > 8 * 128 || K > 24576 || (K % 64 == 0 && (double)rows_per * N * K >= 4e7)) return best;
    for (int t = (M + 127) / 128; t <= 8; ++t) {
        const int per_m = ((M + t - 1) / t + 3) / 4 * 4;
        if (t > 2 && per_m < 44) break;
        for (int S = 1; S <= 16 && (S == 1 || S * 4 <= ktiles); ++S) {
            const int groups = num_cus / (S * t);
            if (groups < 1) break;
            const long per = ((long)N + 4L * groups - 1) / (4L * groups) * 4, rows = per * rows_per;
            int BN = 0;
            for (int b : {32, 48, 64, 80, 96, 112, 144})
                if (b >= rows) { BN = b; break; }
            const int BM = per_m <= 64 ? 64 : per_m <= 96 ? 96 : per_m <= 112 && (BN == 64 || BN == 96) ? 112 : 128;
            if (!BN || BN > (BM == 64 ? 144 : BM == 96 ? 112 : BM == 112 ? 96 : 80)) break;
            const int kt = (ktiles + S - 1) / S;
            const double us = 2.5 + 5.8e-4 * BN * BM + 0.256 * kt * (0.0132 * rows + 0.0107 * per_m) + kt * (0.113 + 1.75e-5 * BN * BM) + 1.5e-7 * M * N * rows_per +
                              (S > 1 ? 1.9 + 8.7e-5 * S * rows * per_m : 0.0);
            if (best.BN && us >= best.us) continue;
            best = MidPlan{BN, (int)((N + per - 1) / per) * t, S, us, (int)per, K % 2048 == 0, t, per_m};
        }
    }
    if (best.BN && best.us >= 0.92 * gemm_us) best.BN = 0;
    return best;
}

}  // namespace

// (the GEMM's plan is made once: it is 0.1-0.4 us of the call)
GemmPlan plan_product(int M, int N, int K, int epilogue, int num_cus, bool token_tiles)
{
    GemmPlan p = plan_gemm(M, N, K, epilogue, num_cus);
    if (!token_tiles) return p;
    const MidPlan m = plan_mid_tiles(M, N, K, epilogue, num_cus, p.us);
    return m.BN ? few_token_plan(m) : p;
}

// ---- decode attention ------------------------------------------------------------------------------
// query heads that share a pass over their cache head: 16 on the matrix cores (D = 128, groups of four and more)
int attention_heads_per_workgroup(int D, int group)
{
    if (group >= 4 && D == 128) return 16;
    return group >= 8 ? 8 : group >= 4 ? 4 : group >= 2 ? 2 : 1;
}

// Chunks per request, at most; 1 = requests are not cut: enough workgroups without, or caches of at most one chunk.  One
// workgroup per compute unit while that leaves a request four chunks and more (6 requests x 8 cache heads of 8192 positions: 5 chunks
// 28.9 us, 10 chunks 29.6; 218 calls with up to 64 pairs and grouped heads 2-4 % slower with two), else two: with fewer chunks
// it is a request's length that decides how long a workgroup takes, and a second one on a unit fills the gaps (217 calls with 65..255
// pairs and caches above 512 positions: 0.96 of the time with one per unit, rounded up).  Long requests cut into 512..2048
// positions whatever the rule says were 1-3 % slower on average over 300 calls and up to twice as fast where one request
// is much longer than all others.
//
// Requests of up to 512 positions are one chunk with half as many (request, cache head) pairs as compute units and more: so many
// workgroups draw almost what memory gives, and a short request cut gains less than the second launch costs (69 calls with 128..255
// pairs and caches of up to 512 positions: 0.71 of the time they take cut; up to 1024 positions, batches of unequal lengths lost).
AttnSplit attention_split(int B, int heads, int S_max, int num_cus)
{
    const long base = (long)B * heads;
    const int whole = 2 * base >= num_cus ? AT_WHOLE : AT_MIN_CHUNK;
    if (base >= num_cus || S_max <= whole) return AttnSplit{1, whole};
    long want = num_cus / base;
    if (want < 4) want = 2L * num_cus / base;
    if (want > AT_MAX_SPLIT) want = AT_MAX_SPLIT;
    const int most = (S_max - 1) / AT_MIN_CHUNK + 1;
    return AttnSplit{(int)(want < most ? want : most), whole};
}

}  // namespace thi
