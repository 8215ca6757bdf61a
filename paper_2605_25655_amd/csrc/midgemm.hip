// fp16 MFMA GEMM for few tokens on gfx950, bound by the way into LDS.  Up to 128 tokens one token tile, and the weights are read once; above, several where they
// are faster (plan_product), neighbours on an XCD that read their weights once each.
//
// Between decode and prefill the weights still stream by once, but every compute unit also needs the activations, and the
// way into LDS is what is short.  Measured with the loads alone: a CU brings in ~120 GB/s of what its L2 holds, but ~60 GB/s (27 GB/s when all
// 256 share the HBM) as soon as some of it comes from memory, whatever the number of stages: the loads return in order, and 256 lines (32 KiB) are
// in flight per CU.  So
//   - every CU takes part, and with one token tile, which holds all tokens, a weight row is read by one workgroup only;
//   - a workgroup reads its rows' K / S weights and M * K / S activations: outputs dealt evenly (in fours) over tiles in S k ranges, tiles * S
//     just below the number of CUs; rows that no output needs and tokens past M are not asked for (time goes by the number of loads:
//     21-25 ns each, 8.8 where the L2 holds everything);
//   - the token tile is no larger than it must be (64, 96, 112 with 64 or 96 rows, or 128): what it does not take deepens the pipeline
//     (72 x 12288 x 4096: 29.1 us with a tile of 128 and three stages, 25.3 with 96 and four);
//   - a stage is 128 k (256 bytes of a row, half the barriers of 64 k), the eight waves are two token groups x the four
//     k-steps of a stage (with 112 tokens two row groups instead): a fragment of weights is read from LDS twice and one of activations once, where eight waves
//     along the tokens read the weights eight times.  The four k groups' sums meet in LDS at the end;
//   - a k-tile's loads go out right behind its barrier, with next to no scalar work around them: the address of each is a pointer that
//     advances, what the wave waits for is a constant (two copies of the loop, by the loads per wave).  With addresses
//     computed per load, a branch tree for the wait and the loads spread between the MFMAs, gate/up 2 x 11008 x 4096 at 72 tokens took 37.7 us (now 35.2),
//     72 x 12288 x 4096 26.2 (24.1), 128 x 4096 x 11008 31.1 (29.1), 128 x 19968 x 6656 64.8 (61.0), 38 x 11488 x 2368, which 180 of 256 CUs did, 16.3 (13.8);
//   - plain shapes ask for a k-tile's weights and activations in one order and for the next one's in the other: longer runs of loads that the L2
//     holds, which come at its rate (128 x 12288 x 4096 30.6 -> 29.3 us; where starts are spread over k it loses 1-3 %).
// Two workgroups per CU with half the stages each, and waves that do nothing but load, were both slower.
//
// S > 1 hands over fp32 partial tiles inside the kernel: every workgroup of a tile stores its partial tile with
// device-scope stores, waits for the acknowledgements and counts its arrival; the one that arrives last adds the
// others' in share order (its own in its place, so the result does not depend on who that is) and runs the epilogue.
// Nobody waits for anybody.
//
// Up to 32 tokens (a tile of 32) it takes RMSNorm along: gamma is one more row of a stage, a wave multiplies its activation fragments by
// it in front of their MFMAs (one fp16 rounding, as in the decode kernels) and adds the squares, 1 / rms scales the finished
// sums.  Gate/up at 32 tokens against the row blocks 2 x 13824 x 5120 51.6 -> 44.2 us, 2 x 17920 x 6656 83.1 -> 72.7 (5.7 and 6.6 TB/s; with RMSNorm 0.8 us
// more), 2 x 11008 x 4096 31.6 -> 29.4 (forced: the MLP it belongs to keeps the row blocks, api.hip); 4096 x 11008 21.8 -> 19.0, 8192 x 8192 26.2 -> 23.5,
// 12288 x 4096 21.0 -> 17.8.
//
// Against the GEMM's few-token configurations and their second pass, or the stream-K decode kernel where that ran (same
// box, rotated weights), N x K: 40 tokens 4096 x 4096 16.3 -> 12.4 us, 4096 x 11008 26.6 -> 21.8, 15360 x 5120 38 -> 30;
// 72 tokens 4096 x 4096 18.3 -> 15.6, 4096 x 11008 32.2 -> 24.6, 12288 x 4096 33.6 -> 24.1, 19968 x 6656 71 -> 54,
// gate/up 2 x 11008 x 4096 49.5 -> 35, 2 x 13824 x 5120 62.7 -> 55; 128 tokens 6656 x 17920 70.7 -> 59, 4096 x 11008
// 35.6 -> 29, 12288 x 4096 35.6 -> 29.
#include "thi_internal.h"

#include <mutex>
#include <type_traits>

namespace thi {

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int MID_THREADS = 64 * MID_WAVES, MID_GK = 128, MID_P = MID_GK / 8;      // 16-byte pieces per staged row
constexpr int MID_KG = 4;                            // the waves: the four k-steps of a stage x ...
constexpr int mid_tg(int BM) { return BM / 16 % 2 ? 1 : 2; }      // ... two token groups, or two row groups where the token fragments are odd in number
constexpr int MID_LDS = 160 * 1024;

__device__ __forceinline__ void mid_dma(bool nt, const void* base_uniform, unsigned lane_byte_offset, unsigned lds_addr)
{
    if (nt)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr) : "memory");
}

// rows of a stage: weights, tokens, and with RMSNorm gamma (a load brings four rows)
template <int BN, int BM, bool RMS>
constexpr int mid_rows() { return BN + BM + (RMS ? 4 : 0); }

template <int BN, int BM, bool RMS>
constexpr int mid_stages()
{
    constexpr int n = MID_LDS / (mid_rows<BN, BM, RMS>() * MID_GK * 2);
    return n > 5 ? 5 : n;
}

// the k groups' partial fragments meet in LDS: all at once where they fit, else in two rounds of a multiple of four
template <int BN, int BM>
constexpr int mid_round()
{
    constexpr int F = BN * mid_tg(BM) * MID_KG / (16 * MID_WAVES) * (BM / (16 * mid_tg(BM)));
    return MID_WAVES * F * 1024 <= MID_LDS ? F : (F / 2 + 3) / 4 * 4;
}

template <int BN, int BM, bool RMS>
constexpr int mid_lds()
{
    constexpr int F = BN * mid_tg(BM) * MID_KG / (16 * MID_WAVES) * (BM / (16 * mid_tg(BM))), R = mid_round<BN, BM>();
    constexpr int stages = mid_stages<BN, BM, RMS>() * mid_rows<BN, BM, RMS>() * MID_GK * 2, parts = MID_WAVES * R * 1024;
    static_assert(parts <= MID_LDS && F <= 2 * R, "the k groups' partial fragments");
    return stages > parts ? stages : parts;
}

template <int BN, int BM, int EPI, bool RMS>
__global__ __launch_bounds__(MID_THREADS) void gemm_mid(GemmArgs a, int tiles, int S, int ktiles, int per, int rotate, int tiles_m, int per_m,
                                                     unsigned by_tiles, unsigned by_S, unsigned by_tiles_m)
{
    constexpr int TG = mid_tg(BM), NG = MID_WAVES / (TG * MID_KG);       // groups of waves along the tokens and along the rows
    constexpr int TN = BN / (16 * NG), TM = BM / (16 * TG), F = TN * TM;
    constexpr int NS = mid_stages<BN, BM, RMS>();
    constexpr int STAGE = mid_rows<BN, BM, RMS>() * MID_P;   // 16-byte units: weight rows, token rows, gamma
    constexpr int CMAX = ((BN + BM) / 4 + RMS + MID_WAVES - 1) / MID_WAVES, CMIN = CMAX > 1 ? CMAX - 1 : 1;   // loads per k-tile and wave
    static_assert(NS >= 2 && BN % (16 * NG) == 0, "pipeline shape");
    constexpr bool AHEAD = 4 * F + 8 * (TN + TM) <= 130;      // (in registers)
    constexpr int OWN = (F + MID_KG - 1) / MID_KG;           // fragments a wave finishes, at most
    extern __shared__ uintx4 smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = wv % TG, wn = wv / TG % NG, kg = wv / (TG * NG);
    const int lr = lane & 15, hi = lane >> 4;
    const int K = a.K;

    // consecutive workers on one XCD (hardware deals workgroup ids round-robin to the eight); a share's workers are
    // consecutive, so that the workgroups of an XCD walk the same slice of the activations together
    const unsigned G = gridDim.x, bid = blockIdx.x, xcd = bid % 8;
    const unsigned worker = xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8) + bid / 8;
    // Every instruction from here to the first load is time in which nothing is in flight, ~1.4 ns each.  So quotients are products (mid_quotient) and
    // a load's operand is chosen among pointers made once: 463..865 instructions -> 190..547, 49 x 768 x 256 4.2 -> 3.8 us, 54 x 512 x 1376 7.7 -> 7.4,
    // gate/up 54 x 2 x 1376 x 512 and its down projection 14.0 -> 13.1, 110 x 4096 x 4096 16.9 -> 16.5.
    const int share = (int)mid_quotient(worker, tiles, by_tiles), tile = (int)worker - share * tiles;
    const int tile_n = (int)mid_quotient(tile, tiles_m, by_tiles_m);
    const int m0 = (tile - tile_n * tiles_m) * per_m;        // this tile's tokens
    const int M = a.M - m0 < per_m ? a.M - m0 : per_m;
    const int kb = (int)mid_quotient(share * ktiles, S, by_S), ke = (int)mid_quotient((share + 1) * ktiles, S, by_S), nk = ke - kb;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
    // rotate: the tiles of a share start spread over its k-tiles and wrap round (the ranges of an XCD's tiles stay close)
    const int rot = rotate ? (int)mid_quotient(tile * nk, tiles, by_tiles) : 0;      // (a row tile's token tiles are neighbours)

    // A k-tile's loads: T_W of the weights, then T_M of the activations, then gamma, each of four stage rows; the wave takes numbers wv, wv + 8, ...: C or
    // C - 1 of them (a number past the end among the first C - 1 repeats an earlier load: the same bytes to the same place).  Lane L brings the 16-byte unit L
    // of a load: row L / 16, physical piece L % 16, logical piece (L % 16) ^ (row % 16).  Rows that no output of the tile needs are not asked for.
    const int first = tile_n * per, stop = first + per < a.N ? first + per : a.N;      // this tile's outputs (gate/up pairs for SwiGLU)
    const int T_W = (is_swiglu(EPI) ? 2 * per : per) / 4;
    const int T_M = (M + 3) / 4, T = T_W + T_M + (RMS ? 1 : 0);
    const size_t k0 = (size_t)(unsigned)(kb + rot) * MID_GK;
    const uint16_t* const w_first = a.w0 + (size_t)(unsigned)first * (unsigned)K + k0;
    const uint16_t* const u_first = is_swiglu(EPI) ? a.w1 + (size_t)(unsigned)first * (unsigned)K + k0 : w_first;
    const uint16_t* const x_first = a.x + (size_t)(unsigned)m0 * (unsigned)K + k0;
    const uint16_t* const g_first = RMS ? a.gamma + k0 : x_first;
    const uint16_t* src[CMAX];                               // (uniform) where the load's operand starts
    unsigned off[CMAX], tail_off[CMAX], dst[CMAX];           // the lane's byte offset, and that in the last k-tile; (uniform) its place in the stage
    const int pieces = (K - (ktiles - 1) * MID_GK) / 8;      // of the last k-tile: what lies past them is loaded from its first and zeroed once it has landed
#pragma unroll
    for (int i = 0; i < CMAX; ++i) {
        int n = wv + MID_WAVES * i;
        n = n < T ? n : T - 1;
        const bool weights = MID_WAVES * i < BN / 4 && n < T_W, tokens = !RMS || n < T_W + T_M;
        // (gate/up pairs, an odd number of fours: the last four up rows lie behind four gate rows that do not exist)
        const int block = weights ? (is_swiglu(EPI) && (per & 7) == 4 && n == T_W - 1 ? n + 1 : n) : tokens ? BN / 4 + n - T_W : (BN + BM) / 4;
        // row within the stage, and from the start of its operand's tile; rows that do not exist: a valid one
        const int v = block * 4 + hi, r = weights ? (is_swiglu(EPI) ? (v >> 4) * 8 + (v & 7) : v) : v - BN;      // 8 gate rows, the 8 matching up rows, ...
        const int last = weights ? stop - 1 - first : tokens ? M - 1 : 0;
        off[i] = ((unsigned)(r < last ? r : last) * (unsigned)K + (unsigned)(lr ^ (v & 15)) * 8u) * 2u;
        tail_off[i] = (lr ^ (v & 15)) < pieces ? off[i] : off[i] - (unsigned)(lr ^ (v & 15)) * 16u;
        dst[i] = lds0 + (unsigned)block * 1024u;
        src[i] = weights ? (is_swiglu(EPI) && ((block >> 1) & 1) ? u_first : w_first) : tokens ? x_first : g_first;
    }
    // Which loads are non-temporal: the weights, unless other token tiles read them too (mid_streams).  234 x 5907 x 3272 on three token tiles 28.2 -> 26.4 us
    // with their weights left in the caches, gate/up 163 x 2 x 2056 x 5896 29.9 -> 29.2.  (Where a tile is full, most are known beforehand and have no branch.)
    const bool full_tile = T_W == BN / 4 && tiles_m == 1;
    const unsigned streams = (unsigned)__builtin_amdgcn_readfirstlane((int)mid_streams(wv, T_W, tiles_m));
    const int c_loads = (T + MID_WAVES - 1) / MID_WAVES < CMIN ? CMIN : (T + MID_WAVES - 1) / MID_WAVES;
    const int it_tail = (K & (MID_GK - 1)) != 0 && ke == ktiles ? nk - 1 - rot : -1;      // the turn of a ragged K's last k-tile

    floatx4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    half8 wa[AHEAD ? 2 : 1][TN], xb[AHEAD ? 2 : 1][TM], gm[AHEAD ? 2 : 1];
    float ssq[TM];                               // RMSNorm: of token lr of a fragment, over this lane's k
#pragma unroll
    for (int j = 0; j < TM; ++j) ssq[j] = 0.f;
    const int fpos = lr * MID_P + ((4 * kg + hi) ^ lr);      // every fragment starts on a multiple of 16 rows
    auto frags = [&](int buf, int fs) __attribute__((always_inline)) {
        const uintx4* base = smem + buf * STAGE + fpos;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) wa[fs][tn] = __builtin_bit_cast(half8, base[(wn * (BN / NG) + tn * 16) * MID_P]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xb[fs][tm] = __builtin_bit_cast(half8, base[(BN + tg * (BM / TG) + tm * 16) * MID_P]);
        if constexpr (RMS) gm[fs] = __builtin_bit_cast(half8, smem[buf * STAGE + (BN + BM) * MID_P + (4 * kg + hi)]);
    };
    // RMSNorm: the squares of a k-tile's activations, then x * gamma in one rounding
    auto norm = [&](int fs) __attribute__((always_inline)) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const half2_t h2 = {xb[fs][tm][e], xb[fs][tm][e + 1]};
                ssq[tm] = __builtin_amdgcn_fdot2(h2, h2, ssq[tm], false);
            }
            xb[fs][tm] *= gm[fs];
        }
    };
    auto multiply = [&](int fs) __attribute__((always_inline)) {
        if constexpr (RMS) norm(fs);
#pragma unroll
        for (int q = 0; q < F; ++q)
            acc[q / TM][q % TM] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[fs][q / TM], xb[fs][q % TM], acc[q / TM][q % TM], 0, 0, 0);
    };
    auto run = [&](auto count) __attribute__((always_inline)) {
        constexpr int C = decltype(count)::value;
        static_assert(C * (NS - 2) < 64, "wait count out of range");
        const bool full = wv + MID_WAVES * (C - 1) < T;      // (the others have one load less)
        int next = 0, kt_next = rot;                         // the k-tile that is loaded next: which turn, and its place in the range
        unsigned stage = 0;                                  // ... and the stage it goes to (bytes)
        auto nt = [&](int i) __attribute__((always_inline)) {
            return ((i + 1) * MID_WAVES <= BN / 4 && full_tile) || (i * MID_WAVES < BN / 4 && (streams >> i & 1));
        };
        // The loads up front are code that runs once: a select for the tail, where a branch per load is one more place to fetch instructions from
        // (45 x 9752 x 344 6.5 -> 6.0 us, 56 x 13913 x 264 7.3 -> 6.7).  Those in the loop are not: there the branch keeps them apart, and with
        // one question per k-tile 128 x 8192 x 8192 took 39.3 us for 37.9, 90 x 15360 x 5120 38.2 for 35.9.
        auto up_front = [&](int i) __attribute__((always_inline)) {
            if (i == C - 1 && !full) return;
            mid_dma(nt(i), src[i], next == it_tail ? tail_off[i] : off[i], dst[i] + stage);
        };
        auto in_the_loop = [&](int i) __attribute__((always_inline)) {
            if (i == C - 1 && !full) return;
            if (next != it_tail) mid_dma(nt(i), src[i], off[i], dst[i] + stage);
            else mid_dma(false, src[i], tail_off[i], dst[i] + stage);
        };
        auto advance = [&]() __attribute__((always_inline)) {
            ++next;
            stage = stage + STAGE * 16 == NS * STAGE * 16 ? 0 : stage + STAGE * 16;
            if (++kt_next == nk) {                           // wraps round
                kt_next = 0;
#pragma unroll
                for (int i = 0; i < C; ++i) src[i] -= (size_t)(nk - 1) * MID_GK;
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i) src[i] += MID_GK;
            }
        };
        auto load = [&](auto one) __attribute__((always_inline)) {
            if (BM >= 64 && !rotate && (next & 1)) {
#pragma unroll
                for (int i = C - 1; i >= 0; --i) one(i);
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i) one(i);
            }
            advance();
        };
        auto zero_tail = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < C; ++i)
                if ((i < C - 1 || full) && tail_off[i] != off[i]) smem[buf * STAGE + (int)((dst[i] - lds0) / 16u) + lane] = uintx4{0u, 0u, 0u, 0u};
        };
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s < nk) load(up_front);
        // One k-tile: it must have landed (the ones behind it, up to NS - 2, may be in flight), and every wave has read its fragments of the
        // one in front, whose stage is free.  The loads come first: what a compute unit has in flight is what bounds the kernel.
        int st = 0;
        auto step = [&](int it, int fs) __attribute__((always_inline)) {
            const bool more = it + NS - 2 < nk;              // (step 0, with NS k-tiles on their way, could leave NS - 1: its wait is a little early)
            if (more && full) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C * (NS - 2)) : "memory");
            else if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((C - 1) * (NS - 2)) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (it == it_tail) zero_tail(st);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            if (it > 0 && next < nk) load(in_the_loop);
            __builtin_amdgcn_sched_barrier(0);
            frags(st, fs);
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
            st = st + 1 == NS ? 0 : st + 1;
        };
        if constexpr (AHEAD) {                               // a k-tile is multiplied while the next one's fragments are read
            step(0, 0);
            int it = 1;
            for (; it + 1 < nk; it += 2) {
                step(it, 1);
                multiply(0);
                __builtin_amdgcn_sched_barrier(0);
                step(it + 1, 0);
                multiply(1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (it < nk) {
                step(it, 1);
                multiply(0);
                multiply(1);
            } else {
                multiply(0);
            }
        } else {
            for (int it = 0; it < nk; ++it) {
                step(it, 0);
                multiply(0);
            }
        }
    };
    if (c_loads == CMIN) run(std::integral_constant<int, CMIN>{});
    else run(std::integral_constant<int, CMAX>{});

    // ---- the four k groups meet in LDS: group g finishes the fragments f % 4 == g of its token group ----------------
    constexpr int FR = mid_round<BN, BM>();                       // fragments per round
    floatx4* const part = reinterpret_cast<floatx4*>(smem);      // [token group][source k group][fragment of the round][lane]
    floatx4 mine[OWN];
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += FR) {
        __syncthreads();
#pragma unroll
        for (int f = f0; f < F && f < f0 + FR; ++f)
            if (f % MID_KG != kg) part[(((wn * TG + tg) * MID_KG + kg) * FR + f - f0) * 64 + lane] = acc[f / TM][f % TM];
        __syncthreads();
#pragma unroll
        for (int o = f0 / MID_KG; o < OWN && MID_KG * o < f0 + FR; ++o) {
            mine[o] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (MID_KG * o + kg >= F) continue;
            floatx4 own = acc[(MID_KG * o) / TM][(MID_KG * o) % TM];
#pragma unroll
            for (int g = 1; g < MID_KG; ++g)
                if (MID_KG * o + g < F && kg == g) own = acc[(MID_KG * o + g < F ? MID_KG * o + g : 0) / TM][(MID_KG * o + g < F ? MID_KG * o + g : 0) % TM];
#pragma unroll
            for (int g = 0; g < MID_KG; ++g)                     // in k order
                mine[o] += g == kg ? own : part[(((wn * TG + tg) * MID_KG + g) * FR + MID_KG * o + kg - f0) * 64 + lane];
        }
    }

    const int m_wave = tg * (BM / TG);
    // RMSNorm: the tokens' sums of squares over this workgroup's k range, k groups in order
    float* const s_ssq = reinterpret_cast<float*>(smem);
    if constexpr (RMS) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            ssq[tm] += __shfl_xor(ssq[tm], 16);
            ssq[tm] += __shfl_xor(ssq[tm], 32);
        }
        __syncthreads();                                     // everybody has read the partial fragments
        if (hi == 0) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) s_ssq[kg * BM + m_wave + tm * 16 + lr] = ssq[tm];
        }
        __syncthreads();
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const float* const q = s_ssq + m_wave + tm * 16 + lr;
            ssq[tm] = ((q[0] + q[BM]) + q[2 * BM]) + q[3 * BM];
        }
    }
    if (S > 1) {
        constexpr size_t frags_of = mid_slot_floats(BN, BM, false);        // floats: [wave][finished fragment][lane][4]
        constexpr size_t slot = mid_slot_floats(BN, BM, RMS);              // ... then the sums of squares
        static_assert(frags_of == (size_t)MID_WAVES * OWN * 64 * 4, "a workgroup's partial tile");
        static_assert(BM > MID_DECODE_M || slot <= SK_SLOT_WORDS, "at decode sizes it lies in the decode kernels' slots");
        float* const ps = a.partials + ((size_t)tile * S + share) * slot + (size_t)(wv * OWN * 64 + lane) * 4;
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            if (MID_KG * o + kg < F && m_wave + ((MID_KG * o + kg) % TM) * 16 < M)
                // (the no-op keeps the next instruction off the data registers: the compiler does not know this store)
                asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(ps + o * 256), "v"(mine[o]) : "memory");
        if constexpr (RMS) {
            float* const pq = a.partials + ((size_t)tile * S + share) * slot + frags_of + m_wave + lr;
            if (kg == 0 && hi == 0) {
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) __hip_atomic_store(pq + tm * 16, ssq[tm], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // acknowledged by the memory system ...
        __syncthreads();                                     // ... for every thread, before the arrival is counted
        unsigned* const flag = reinterpret_cast<unsigned*>(smem);
        if (tid == 0) {
            const unsigned before = __hip_atomic_fetch_add(a.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned is_last = before + 1u == (unsigned)S;
            if (is_last) __hip_atomic_store(a.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // zero between calls
            *flag = is_last;
        }
        __syncthreads();
        if (*flag == 0u) return;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(a.partials + (size_t)tile * S * slot, 0, (int)(S * slot * 4), 0x00020000);
        floatx4 v[OWN];
#pragma unroll
        for (int o = 0; o < OWN; ++o) v[o] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < S; s0 += 4) {
            floatx4 q[4][OWN];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int o = 0; o < OWN; ++o) q[b][o] = mine[o];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if (s0 + b >= S || s0 + b == share) continue;    // (uniform)
#pragma unroll
                for (int o = 0; o < OWN; ++o)
                    q[b][o] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (wv * OWN * 64 + lane) * 16,
                                                                                                (int)((s0 + b) * slot * 4) + o * 1024, 16));
            }
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (s0 + b < S) {
#pragma unroll
                    for (int o = 0; o < OWN; ++o) v[o] += q[b][o];
                }
        }
#pragma unroll
        for (int o = 0; o < OWN; ++o) mine[o] = v[o];
        if constexpr (RMS) {                                 // in share order
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) ssq[tm] = 0.f;
            for (int s = 0; s < S; ++s) {
                const float* const pq = a.partials + ((size_t)tile * S + s) * slot + frags_of + m_wave + lr;
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) ssq[tm] += __hip_atomic_load(pq + tm * 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }

#pragma unroll
    for (int o = 0; o < OWN; ++o) {
        const int f = MID_KG * o + kg, tn = wn * TN + f / TM, tm = f % TM;
        if (f >= F) continue;
        const int m = m_wave + tm * 16 + lr;
        if constexpr (RMS) {
            float q = ssq[0];
#pragma unroll
            for (int t = 1; t < TM; ++t) q = tm == t ? ssq[t] : q;
            mine[o] *= 1.0f / __builtin_sqrtf(q / (float)K + a.eps);
        }
        uint16_t* const orow = a.out + (size_t)(m0 + (m < M ? m : 0)) * a.ldo;
        if (is_swiglu(EPI)) {
            // rows 0..7 of a fragment are gate rows, 8..15 the matching up rows: exchanged between the wave's halves
            floatx4 up;
#pragma unroll
            for (int c = 0; c < 4; ++c) up[c] = __shfl_xor(mine[o][c], 32);
            const int j = first + tn * 8 + 4 * hi;
            if (hi < 2 && m < M) {
                half4 hv;
#pragma unroll
                for (int c = 0; c < 4; ++c) hv[c] = (_Float16)silu_mul(mine[o][c], up[c]);
                if (j + 3 < stop) {
                    *reinterpret_cast<half4_any*>(orow + j) = hv;
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (j + c < stop) orow[j + c] = __builtin_bit_cast(uint16_t, hv[c]);
                }
            }
        } else if (m < M) {
            const int n = first + tn * 16 + 4 * hi;
            float y[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) y[c] = mine[o][c];
            if constexpr (has_rope(EPI) && RMS) {                // no pass in front that leaves a table
                rope_pair(a.rope, a.rope.pos[m0 + m], n, y[0], y[1]);
                rope_pair(a.rope, a.rope.pos[m0 + m], n + 2, y[2], y[3]);
            } else if (has_rope(EPI)) {
                rope_pair_table(a.rope, m0 + m, n, y[0], y[1]);
                rope_pair_table(a.rope, m0 + m, n + 2, y[2], y[3]);
            }
            if (n + 3 < stop) {
                half4 hv;
                if (a.residual) {
                    const half4 rv = *reinterpret_cast<const half4_any*>(a.residual + (size_t)(m0 + m) * a.ldo + n);
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] += (float)rv[c];
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) hv[c] = (_Float16)y[c];
                *reinterpret_cast<half4_any*>(orow + n) = hv;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (n + c < stop) {
                        if (a.residual) y[c] += half_bits_to_float(a.residual[(size_t)(m0 + m) * a.ldo + n + c]);
                        orow[n + c] = to_half_bits(y[c]);
                    }
            }
        }
    }
}

template <int BN, int BM, bool RMS>
hipError_t launch_mid_cfg(const GemmArgs& a, int epilogue, const MidPlan& p, hipStream_t stream)
{
    const size_t lds = mid_lds<BN, BM, RMS>();
    const int ktiles = (a.K + MID_GK - 1) / MID_GK;
#define THI_LAUNCH(E)                                                                                        \
    do {                                                                                                     \
        auto kern = gemm_mid<BN, BM, E, RMS>;                                                                \
        static std::once_flag attr_once;      /* one opt-in per kernel variant, safe from several threads */ \
        std::call_once(attr_once, [&] {                                                                      \
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                   \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                 \
        });                                                                                                  \
        hipLaunchKernelGGL(kern, dim3(p.tiles * p.S), dim3(MID_THREADS), lds, stream, a, p.tiles, p.S, ktiles, p.per, (int)p.rotate, p.tiles_m, p.per_m, \
                           mid_divisor(p.tiles), mid_divisor(p.S), mid_divisor(p.tiles_m));                   \
    } while (0)
    switch (epilogue) {
    case EPI_PLAIN: THI_LAUNCH(EPI_PLAIN); break;
    case EPI_ROPE:                             // up to MID_DECODE_M tokens always behind RMSNorm
        if constexpr (BM > MID_DECODE_M || RMS) THI_LAUNCH(EPI_ROPE);
        else return hipErrorInvalidValue;
        break;
    case EPI_SWIGLU: THI_LAUNCH(EPI_SWIGLU); break;
    default: return hipErrorInvalidValue;      // RMSNorm: by a.gamma
    }
#undef THI_LAUNCH
    return hipGetLastError();
}

template <int BM, bool RMS>
hipError_t launch_mid_bm(const GemmArgs& a, int epilogue, const MidPlan& p, hipStream_t stream)
{
    switch (p.BN) {
    case 32: if constexpr (BM != 112) return launch_mid_cfg<32, BM, RMS>(a, epilogue, p, stream); else break;
    case 112: if constexpr (BM <= 96) return launch_mid_cfg<112, BM, RMS>(a, epilogue, p, stream); else break;
    case 128: if constexpr (BM <= 32) return launch_mid_cfg<128, BM, RMS>(a, epilogue, p, stream); else break;
    case 144: if constexpr (BM <= 64) return launch_mid_cfg<144, BM, RMS>(a, epilogue, p, stream); else break;
    case 176: if constexpr (BM <= 32) return launch_mid_cfg<176, BM, RMS>(a, epilogue, p, stream); else break;
    case 48: if constexpr (BM != 112) return launch_mid_cfg<48, BM, RMS>(a, epilogue, p, stream); else break;
    case 64: return launch_mid_cfg<64, BM, RMS>(a, epilogue, p, stream);
    case 80: if constexpr (BM != 112) return launch_mid_cfg<80, BM, RMS>(a, epilogue, p, stream); else break;
    case 96: if constexpr (BM <= 112) return launch_mid_cfg<96, BM, RMS>(a, epilogue, p, stream); else break;
    default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_mid(const GemmArgs& a, int epilogue, const MidPlan& p, hipStream_t stream)
{
    if (a.M <= MID_DECODE_M) return a.gamma ? launch_mid_bm<32, true>(a, epilogue, p, stream) : launch_mid_bm<32, false>(a, epilogue, p, stream);
    if (a.gamma) return hipErrorInvalidValue;                // RMSNorm runs as a pass of its own in front
    if (p.per_m <= 64) return launch_mid_bm<64, false>(a, epilogue, p, stream);
    if (p.per_m <= 96) return launch_mid_bm<96, false>(a, epilogue, p, stream);
    if (p.per_m <= 112 && (p.BN == 64 || p.BN == 96)) return launch_mid_bm<112, false>(a, epilogue, p, stream);
    if (p.per_m <= 128) return launch_mid_bm<128, false>(a, epilogue, p, stream);
    return hipErrorInvalidValue;
}

}  // namespace thi
