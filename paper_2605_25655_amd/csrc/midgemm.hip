// fp16 MFMA GEMM for few tokens (up to 128) on gfx950: one token tile, weights read once, bound by memory.
//
// Between decode and prefill the weights still stream by once, but every compute unit also needs the activations, and the
// way into LDS is what is short: measured with the loads alone, a CU brings in 27 GB/s of an HBM stream that all 256
// share (7 TB/s), ~120 GB/s of what its L2 holds, and ~60 GB/s of a mixture whatever the number of stages (64 KiB are
// in flight, the loads return in order, so the activations wait behind the weights' HBM latency).  So
//   - every CU takes part, and a weight row is read by one workgroup only (the token tile holds all tokens);
//   - a workgroup reads BN * K / S weights and M * K / S activations: BN rows per tile, S k ranges per tile, tiles * S
//     just below the number of CUs (tiles of 32..144 rows, so that most shapes come close); tokens past M are not loaded;
//   - the token tile is no larger than it must be (64, 96 or 128): what it does not take deepens the pipeline
//     (72 x 12288 x 4096: 29.1 us with a tile of 128 and three stages, 25.3 with 96 and four);
//   - a stage is 128 k (256 bytes of a row, half the barriers of 64 k), the eight waves are two token groups x the four
//     k-steps of a stage: a fragment of weights is read from LDS twice and one of activations once, where eight waves
//     along the tokens read the weights eight times.  The four k groups' sums meet in LDS at the end.
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
// more), 2 x 11008 x 4096 31.6 -> 29.4 (forced: the MLP it belongs to keeps the row blocks, api.hip); 4096 x 11008 21.8 -> 19.0, 8192 x 8192 26.2 -> 24.5.
//
// Against the GEMM's few-token configurations and their second pass, or the stream-K decode kernel where that ran (same
// box, rotated weights), N x K: 40 tokens 4096 x 4096 16.3 -> 12.6 us, 4096 x 11008 26.6 -> 21.8, 15360 x 5120 38 -> 31;
// 72 tokens 4096 x 4096 18.3 -> 15.6, 4096 x 11008 32.2 -> 25.2, 12288 x 4096 33.6 -> 25.6, 19968 x 6656 71 -> 54,
// gate/up 2 x 11008 x 4096 49.5 -> 40, 2 x 13824 x 5120 62.7 -> 55; 128 tokens 6656 x 17920 70.7 -> 59, 4096 x 11008
// 35.6 -> 30.8, 12288 x 4096 35.6 -> 32.
#include "thi_internal.h"

#include <mutex>
#include <type_traits>

namespace thi {

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int MID_THREADS = 512, MID_WAVES = 8, MID_GK = 128, MID_P = MID_GK / 8;      // 16-byte pieces per staged row
constexpr int MID_TG = 2, MID_KG = 4;                // the waves: two token groups x the four k-steps of a stage
constexpr int MID_LDS = 160 * 1024;

template <bool NT>
__device__ __forceinline__ void mid_dma(const void* base_uniform, unsigned lane_byte_offset, unsigned lds_addr)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr) : "memory");
}

// at most n * PER loads of this wave still in flight (n uniform, 1..12)
template <int PER>
__device__ __forceinline__ void wait_loads(int n)
{
    static_assert(PER * 12 < 64, "wait count out of range");
    switch (n) {
    case 1: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * PER) : "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * PER) : "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(5 * PER) : "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(6 * PER) : "memory"); break;
    case 7: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(7 * PER) : "memory"); break;
    case 8: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * PER) : "memory"); break;
    case 9: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 * PER) : "memory"); break;
    case 10: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(10 * PER) : "memory"); break;
    case 11: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(11 * PER) : "memory"); break;
    case 12: asm volatile("s_waitcnt vmcnt(%0)" ::"n"(12 * PER) : "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
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
    constexpr int F = (BN / 16) * (BM / (16 * MID_TG));
    return MID_WAVES * F * 1024 <= MID_LDS ? F : (F / 2 + 3) / 4 * 4;
}

template <int BN, int BM, bool RMS>
constexpr int mid_lds()
{
    constexpr int F = (BN / 16) * (BM / (16 * MID_TG)), R = mid_round<BN, BM>();
    constexpr int stages = mid_stages<BN, BM, RMS>() * mid_rows<BN, BM, RMS>() * MID_GK * 2, parts = MID_WAVES * R * 1024;
    static_assert(parts <= MID_LDS && F <= 2 * R, "the k groups' partial fragments");
    return stages > parts ? stages : parts;
}

template <int BN, int BM, int EPI, bool RMS>
__global__ __launch_bounds__(MID_THREADS) void gemm_mid(GemmArgs a, int tiles, int S, int ktiles, int per, int rotate)
{
    constexpr int TN = BN / 16, TM = BM / (16 * MID_TG), F = TN * TM;
    constexpr int NS = mid_stages<BN, BM, RMS>();
    constexpr int STAGE = mid_rows<BN, BM, RMS>() * MID_P;   // 16-byte units: weight rows, token rows, gamma
    constexpr int T_W = BN / 4;                              // wave-wide loads of the weights per k-tile (four rows each)
    constexpr int NI = (mid_rows<BN, BM, RMS>() / 4 + MID_WAVES - 1) / MID_WAVES;   // loads per k-tile and wave, at most
    static_assert(NS >= 2 && NI <= 12 && BN % 16 == 0, "pipeline shape");
    constexpr int OWN = (F + MID_KG - 1) / MID_KG;           // fragments a wave finishes, at most
    extern __shared__ uintx4 smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = wv & 1, kg = wv >> 1;
    const int lr = lane & 15, hi = lane >> 4;
    const int K = a.K, M = a.M;

    // consecutive workers on one XCD (hardware deals workgroup ids round-robin to the eight); a share's workers are
    // consecutive, so that the workgroups of an XCD walk the same slice of the activations together
    int worker;
    {
        const int G = gridDim.x, bid = blockIdx.x, per = G / 8, rem = G % 8, xcd = bid % 8, local = bid / 8;
        worker = xcd * per + (xcd < rem ? xcd : rem) + local;
    }
    const int share = worker / tiles, tile = worker % tiles;
    const int kb = share * ktiles / S, ke = (share + 1) * ktiles / S, nk = ke - kb;
    const bool ragged = (K & (MID_GK - 1)) != 0;
    // rotate: the tiles of a share start spread over its k-tiles and wrap round (the ranges of an XCD's tiles stay close)
    const int rot = rotate ? (int)((long)tile * nk / tiles) : 0;
    auto k_tile = [&](int it) __attribute__((always_inline)) { const int k = it + rot; return kb + (k < nk ? k : k - nk); };

    // This wave's loads: number wv + 8 i covers four stage rows (weights first, then tokens); lane L brings the 16-byte
    // unit L of it: row L / 16, physical piece L % 16, logical piece (L % 16) ^ (row % 16).
    const int T_X = T_W + ((M + 3) >> 2), T = T_X + (RMS ? 1 : 0);
    const int cnt = (T - wv + MID_WAVES - 1) / MID_WAVES;
    const int first = tile * per, stop = first + per < a.N ? first + per : a.N;      // this tile's outputs (gate/up pairs for SwiGLU)
    const uint16_t* const wbase = a.w0 + (size_t)first * K;
    const uint16_t* const ubase = is_swiglu(EPI) ? a.w1 + (size_t)first * K : nullptr;
    // four stage rows each: where load idx goes
    auto block = [&](int idx) __attribute__((always_inline)) { return !RMS || idx < T_X ? idx : (BN + BM) / 4; };
    unsigned off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int idx = wv + MID_WAVES * i;
        const int v = block(idx) * 4 + hi;                   // row within the stage
        int row;                                             // ... and from the start of its operand's tile; rows that do not exist: a valid one
        if (idx < T_W) {
            row = is_swiglu(EPI) ? (v >> 4) * 8 + (v & 7) : v;       // 8 gate rows, the 8 matching up rows, ...
            row = first + row < stop ? row : stop - 1 - first;
        } else if (!RMS || idx < T_X) {
            row = v - BN < M ? v - BN : M - 1;
        } else {
            row = 0;
        }
        off[i] = (unsigned)(row * K + (lr ^ (v & 15)) * 8) * 2u;
    }
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
    // pieces past K (last k-tile of a ragged K): loaded from the k-tile's first piece, zeroed once they have landed
    auto past_k = [&](int idx, int kt) __attribute__((always_inline)) {
        const int p = lr ^ ((block(idx) * 4 + hi) & 15);
        return kt * MID_GK + p * 8 >= K ? p : 0;
    };
    auto load1 = [&](int i, int kt, int buf) __attribute__((always_inline)) {
        if (i >= cnt) return;
        const int idx = wv + MID_WAVES * i;
        unsigned o = off[i];
        if (ragged && kt == ktiles - 1) o -= 16u * (unsigned)past_k(idx, kt);
        const unsigned dst = lds0 + (unsigned)(buf * STAGE + block(idx) * 64) * 16u;
        if (idx < T_W) mid_dma<true>((is_swiglu(EPI) && ((idx >> 1) & 1) ? ubase : wbase) + (size_t)kt * MID_GK, o, dst);
        else mid_dma<false>((!RMS || idx < T_X ? a.x : a.gamma) + (size_t)kt * MID_GK, o, dst);
    };
    auto load = [&](int kt, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) load1(i, kt, buf);
    };
    auto zero_tail = [&](int kt, int buf) __attribute__((always_inline)) {
        if (!ragged || kt != ktiles - 1) return;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (i >= cnt) break;
            const int idx = wv + MID_WAVES * i;
            if (past_k(idx, kt)) smem[buf * STAGE + block(idx) * 64 + lane] = uintx4{0u, 0u, 0u, 0u};
        }
    };

    floatx4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    half8 wa[2][TN], xb[2][TM], gm[2];
    float ssq[TM];                               // RMSNorm: of token lr of a fragment, over this lane's k
#pragma unroll
    for (int j = 0; j < TM; ++j) ssq[j] = 0.f;
    const int fpos = lr * MID_P + ((4 * kg + hi) ^ lr);      // every fragment starts on a multiple of 16 rows
    auto frags = [&](int buf, int fs) __attribute__((always_inline)) {
        const uintx4* base = smem + buf * STAGE + fpos;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) wa[fs][tn] = __builtin_bit_cast(half8, base[tn * 16 * MID_P]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) xb[fs][tm] = __builtin_bit_cast(half8, base[(BN + tg * (BM / MID_TG) + tm * 16) * MID_P]);
        if constexpr (RMS) gm[fs] = __builtin_bit_cast(half8, smem[buf * STAGE + (BN + BM) * MID_P + 4 * kg + hi]);
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
    // one k-tile: it must have landed (the ones behind it, up to NS - 2, may be in flight) and its predecessor's
    // fragments have been read; then the predecessor's stage is free, and the predecessor is multiplied while this one's
    // fragments are read.
    auto step = [&](auto par, int it, int st, int free_st) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        if (it + NS - 2 < nk) wait_loads<NS - 2>(cnt);
        else wait_loads<0>(0);
        zero_tail(k_tile(it), st);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        frags(st, P);
        __builtin_amdgcn_sched_barrier(0);
        const bool more = it > 0 && it + NS - 1 < nk;
        if constexpr (RMS) {
            if (it > 0) norm(1 - P);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (it > 0) {
#pragma unroll
                for (int q = F * i / NI; q < F * (i + 1) / NI; ++q)
                    acc[q / TM][q % TM] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[1 - P][q / TM], xb[1 - P][q % TM], acc[q / TM][q % TM], 0, 0, 0);
            }
            if (more) load1(i, k_tile(it + NS - 1), free_st);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto last = [&](auto par) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        if constexpr (RMS) norm(P);
#pragma unroll
        for (int q = 0; q < F; ++q)
            acc[q / TM][q % TM] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[P][q / TM], xb[P][q % TM], acc[q / TM][q % TM], 0, 0, 0);
    };

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nk) load(k_tile(s), s);
    // (the last stage is filled by step 0 too: nothing has been read from it)
    if (NS - 1 < nk) load(k_tile(NS - 1), NS - 1);
    // with NS loads issued up front, step 0 may leave NS - 1 k-tiles in flight; its wait for NS - 2 is a little early
    int st = 0, prev = NS - 1;
    for (int it = 0; it < nk; it += 2) {
        step(std::integral_constant<int, 0>{}, it, st, prev);
        prev = st; st = st + 1 == NS ? 0 : st + 1;
        if (it + 1 < nk) {
            step(std::integral_constant<int, 1>{}, it + 1, st, prev);
            prev = st; st = st + 1 == NS ? 0 : st + 1;
        }
    }
    if (nk & 1) last(std::integral_constant<int, 0>{});
    else last(std::integral_constant<int, 1>{});

    // ---- the four k groups meet in LDS: group g finishes the fragments f % 4 == g of its token group ----------------
    constexpr int R = mid_round<BN, BM>();                       // fragments per round
    floatx4* const part = reinterpret_cast<floatx4*>(smem);      // [token group][source k group][fragment of the round][lane]
    floatx4 mine[OWN];
#pragma unroll
    for (int f0 = 0; f0 < F; f0 += R) {
        __syncthreads();
#pragma unroll
        for (int f = f0; f < F && f < f0 + R; ++f)
            if (f % MID_KG != kg) part[((tg * MID_KG + kg) * R + f - f0) * 64 + lane] = acc[f / TM][f % TM];
        __syncthreads();
#pragma unroll
        for (int o = f0 / MID_KG; o < OWN && MID_KG * o < f0 + R; ++o) {
            mine[o] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (MID_KG * o + kg >= F) continue;
            floatx4 own = acc[(4 * o) / TM][(4 * o) % TM];
#pragma unroll
            for (int g = 1; g < MID_KG; ++g)
                if (4 * o + g < F && kg == g) own = acc[(4 * o + g < F ? 4 * o + g : 0) / TM][(4 * o + g < F ? 4 * o + g : 0) % TM];
#pragma unroll
            for (int g = 0; g < MID_KG; ++g)                     // in k order
                mine[o] += g == kg ? own : part[((tg * MID_KG + g) * R + 4 * o + kg - f0) * 64 + lane];
        }
    }

    const int m_wave = tg * (BM / MID_TG);
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
        static_assert(MID_KG == 4, "four k groups");
    }
    if (S > 1) {
        constexpr size_t frags_of = mid_slot_floats(BN, BM, false);        // floats: [wave][finished fragment][lane][4]
        constexpr size_t slot = mid_slot_floats(BN, BM, RMS);              // ... then the sums of squares
        static_assert(frags_of == (size_t)MID_WAVES * OWN * 64 * 4, "a workgroup's partial tile");
        static_assert(BM > MID_DECODE_M || slot <= SK_SLOT_WORDS, "at decode sizes it lies in the decode kernels' slots");
        float* const ps = a.partials + ((size_t)tile * S + share) * slot + (size_t)(wv * OWN * 64 + lane) * 4;
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            if (4 * o + kg < F && m_wave + ((4 * o + kg) % TM) * 16 < M)
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
        const int f = 4 * o + kg, tn = f / TM, tm = f % TM;
        if (f >= F) continue;
        const int m = m_wave + tm * 16 + lr;
        if constexpr (RMS) {
            float q = ssq[0];
#pragma unroll
            for (int t = 1; t < TM; ++t) q = tm == t ? ssq[t] : q;
            mine[o] *= 1.0f / __builtin_sqrtf(q / (float)K + a.eps);
        }
        uint16_t* const orow = a.out + (size_t)(m < M ? m : 0) * a.ldo;
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
                rope_pair(a.rope, a.rope.pos[m], n, y[0], y[1]);
                rope_pair(a.rope, a.rope.pos[m], n + 2, y[2], y[3]);
            } else if (has_rope(EPI)) {
                rope_pair_table(a.rope, m, n, y[0], y[1]);
                rope_pair_table(a.rope, m, n + 2, y[2], y[3]);
            }
            if (n + 3 < stop) {
                half4 hv;
                if (a.residual) {
                    const half4 rv = *reinterpret_cast<const half4_any*>(a.residual + (size_t)m * a.ldo + n);
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
                        if (a.residual) y[c] += half_bits_to_float(a.residual[(size_t)m * a.ldo + n + c]);
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
        hipLaunchKernelGGL(kern, dim3(p.tiles * p.S), dim3(MID_THREADS), lds, stream, a, p.tiles, p.S, ktiles, p.per, (int)p.rotate); \
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
    case 32: return launch_mid_cfg<32, BM, RMS>(a, epilogue, p, stream);
    case 48: return launch_mid_cfg<48, BM, RMS>(a, epilogue, p, stream);
    case 64: return launch_mid_cfg<64, BM, RMS>(a, epilogue, p, stream);
    case 80: return launch_mid_cfg<80, BM, RMS>(a, epilogue, p, stream);
    case 96: if constexpr (BM <= 96) return launch_mid_cfg<96, BM, RMS>(a, epilogue, p, stream); else break;
    case 112: if constexpr (BM <= 96) return launch_mid_cfg<112, BM, RMS>(a, epilogue, p, stream); else break;
    case 128: if constexpr (BM <= 32) return launch_mid_cfg<128, BM, RMS>(a, epilogue, p, stream); else break;
    case 144: if constexpr (BM <= 64) return launch_mid_cfg<144, BM, RMS>(a, epilogue, p, stream); else break;
    case 176: if constexpr (BM <= 32) return launch_mid_cfg<176, BM, RMS>(a, epilogue, p, stream); else break;
    default: break;
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_mid(const GemmArgs& a, int epilogue, const MidPlan& p, hipStream_t stream)
{
    if (a.M <= MID_DECODE_M) return a.gamma ? launch_mid_bm<32, true>(a, epilogue, p, stream) : launch_mid_bm<32, false>(a, epilogue, p, stream);
    if (a.gamma) return hipErrorInvalidValue;                // RMSNorm runs as a pass of its own in front
    if (a.M <= 64) return launch_mid_bm<64, false>(a, epilogue, p, stream);
    if (a.M <= 96) return launch_mid_bm<96, false>(a, epilogue, p, stream);
    if (a.M <= 128) return launch_mid_bm<128, false>(a, epilogue, p, stream);
    return hipErrorInvalidValue;
}

}  // namespace thi
