// Host-side planning arithmetic of libthi: how work is dealt to workgroups and how large the workspace
// regions are.  No kernels and no HIP calls here, so that this file and api.hip can also be built for the
// host alone (with stand-ins for the kernel launchers) and run under the sanitizers on a machine without
// a GPU.
#include "thi_internal.h"

namespace thi {

// ---- decode kernels ------------------------------------------------------------------------------
size_t skinny_handover_bytes() { return (size_t)SK_MAX_GRID * SK_SLOT_WORDS * sizeof(unsigned); }

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
    if (M <= 16 || M > 32 || H < 1024 || H > ROWSLAB_MAX_K || I < 1024 || I > ROWSLAB_MAX_K) return false;
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

// The few-token kernel: BN rows per tile and S k ranges per tile with the smallest modelled time, at most one workgroup per
// compute unit (a second round starts with an empty pipeline: 13B gate/up at 72 tokens as 432 tiles 68.8 us, the GEMM
// 63.8), not above K = 24576 (the 70B down projection measured 2-4 % behind the kernels it would replace).  The
// constants, in microseconds and KB per workgroup, are fitted to ~400 measured (shape, M, BN, S) points, 17 shapes x
// M = 40..128: 4.2 us fixed, 24 ns a KB of weights, 13 ns a KB of activations, 93 ns a stage; sharing a tile 1 us, 32 ns a
// KB of its partial tiles and 2 / 3 us more with 80 / 96 rows.  The pick is 1 % slower than the best measured one on
// average, 16 % at worst (on problems of 5 us); on 20 further points with the wide tiles it was the best one each time.
// Tiles of 80..144 rows are for shapes that smaller ones cut into more tiles than there are compute units, or into few
// enough that one more share would not fit (against the kernels that served them): 19968 x 6656 at 128 tokens 75.3 -> 62
// us (80 rows), 6656 x 17920 at 128 70.7 -> 59 (80, S = 3), gate/up 2 x 13824 x 5120 at 72 62.7 -> 55 (112), gate/up
// 2 x 17920 x 6656 at 64 107.7 -> 79 (144).  With more rows shared tiles only lose (15360 x 5120 at 72 tokens: 52 us with
// two shares of 144 rows, 35.5 with 64).
MidPlan plan_mid(int M, int N, int K, int epilogue, int num_cus)
{
    MidPlan best{0, 0, 0, 0.0};
    if (M > 128 || K > 24576) return best;
    const int V = is_swiglu(epilogue) ? 2 * N : N;
    const int ktiles = (K + 127) / 128;
    for (int BN : {32, 48, 64, 80, 96, 112, 144}) {
        if (BN > (M > 96 ? 80 : M > 64 ? 112 : 144)) continue;  // (more spill registers)
        const int tiles = (V + BN - 1) / BN;
        for (int S = 1; S <= (BN > 96 ? 1 : 16) && tiles * S <= num_cus && (S == 1 || S * 4 <= ktiles); ++S) {
            const int per = (ktiles + S - 1) / S;
            const double w = BN * per * 0.256, x = M * per * 0.256;
            const double us = 4.2 + 0.024 * w + 0.013 * x + 0.093 * per +
                              (S > 1 ? 1.0 + 0.032 * S * BN * M * 0.004 + (BN == 96 ? 3.0 : BN == 80 ? 2.0 : 0.0) : 0.0);
            if (best.BN == 0 || us < best.us) best = MidPlan{BN, tiles, S, us};
        }
    }
    return best;
}

// ---- decode attention ------------------------------------------------------------------------------
// query heads that share a pass over their cache head: 16 on the matrix cores (D = 128, groups of four and more)
int attention_heads_per_workgroup(int D, int group)
{
    if (group >= 4 && D == 128) return 16;
    return group >= 8 ? 8 : group >= 4 ? 4 : group >= 2 ? 2 : 1;
}

// Chunks per request, at most; 1 = requests are not cut: enough workgroups without, or caches of at most one chunk.  One
// workgroup per compute unit, and no more than that while it leaves a request four chunks or more (6 requests x 8 cache
// heads of 8192 positions: 5 chunks 28.5 us, 6 chunks and 32 compute units with two of them 31); below that the chunks a
// request would lose weigh more than the second workgroup on some units (3 x 40 heads, one request of 13078 positions among short
// ones: 3 chunks 66 us, 2 chunks 89).  Two to four workgroups per unit, or long requests cut into 512..2048 positions
// whatever the rule says, were 1-3 % slower on average over 300 calls and up to twice as fast where one request is much
// longer than all others.
int attention_split(int B, int heads, int S_max, int num_cus)
{
    const long base = (long)B * heads;
    if (base >= num_cus || S_max <= AT_MIN_CHUNK) return 1;
    long want = num_cus / base;
    if (want < 4) want = (num_cus + base - 1) / base;
    if (want > AT_MAX_SPLIT) want = AT_MAX_SPLIT;
    const int most = (S_max - 1) / AT_MIN_CHUNK + 1;
    return (int)(want < most ? want : most);
}

}  // namespace thi
