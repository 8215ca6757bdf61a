// Decode attention on gfx950: one new token per request against that request's own key/value cache
// (Eq. 6, softmax(Q K^T / sqrt(d)) V per head; Sec. III-D.1: attention runs per request because every
// request has its own cache).  HBM-bound: K and V are read once.
//
// What is kept from the paper's MT Attention (Sec. III-C.2): Q and O stay on chip for the whole pass
// (registers here) while K and V are streamed by; the scores and weights of a block never leave the
// chip (stages 1-3 run back to back on a block of positions, with a running maximum and sum so that
// one pass suffices).  What is not: its row-block/outer-product tiling for scratchpads.
//
// Layout: q[B,Hq,D], k/v[B,Hkv,S_max,D] (one head's positions contiguous), out[B,Hq,D], all fp16;
// seq_lens[B] int32 on the device.  Query head h reads cache head h / (Hq/Hkv).
//
// Work split: a workgroup (4 waves) takes one chunk of positions of one (request, cache head) -- chunk_size -- and up
// to GT query heads of that cache head's group.  16 (D = 128) or 8 (D = 64) lanes cover one row with
// 16-byte loads, so a wave instruction reads 4 or 8 consecutive positions = 1 KiB of contiguous memory;
// U such loads of K and of V are in flight per wave, one iteration ahead of the arithmetic.  A lane
// forms its 8-element share of q.k with packed fp16 dot products accumulated in fp32, the shares meet
// by lane shuffles, the weights stay fp32, and V is accumulated in fp32.  Row groups, waves and chunks
// each keep their own (maximum, sum, output) triple; triples are merged in a fixed order (row groups
// by shuffle, waves through LDS, chunks by a second small kernel), so results are reproducible.
#include "thi_internal.h"

#include <mutex>
#include <type_traits>

namespace thi {

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int AT_THREADS = 256;
constexpr int AT_WAVES = 4;

template <int GT> struct Unroll { static constexpr int U = (GT >= 4) ? 2 : 4; };

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Positions per chunk of a request with L live ones: all of them where requests are not cut (a.nsplit == 1) and up to
// a.whole, else 1/nsplit of them in whole multiples of 64, at least AT_MIN_CHUNK.  It is a function of the request's own
// length and of how many workgroups the call has (B, heads), so that a request's chunk borders, and with them the bits of its
// result, do not depend on its neighbours' lengths or on the size of the cache.  It also keeps the head of a workgroup short, one length and one
// division: a chunk size common to the batch, searched for on the device so that all chunks just fit the compute
// units, took ~1 us of scans in front of the first load (8 heads of 64, 2 requests of 468 positions 7.5 us, now 6.2; 5 requests of
// 332 with 40 heads of 128 14.1, now 11) and won only where one request is much longer than all others (7 requests x 8 cache heads, one
// of 14908 positions and the rest of 745: 24 us, now 45).
__device__ __forceinline__ int chunk_size(const AttnArgs& a, int L)
{
    if (a.nsplit == 1) return L;
    if (L <= a.whole) return a.whole;
    const int size = (int)(((unsigned)(L + a.nsplit - 1) / (unsigned)a.nsplit + 63u) & ~63u);
    return size > AT_MIN_CHUNK ? size : AT_MIN_CHUNK;
}

// What a workgroup works on: positions [c0, c1) of request b, its chunk number s (whole: its only one).
struct Item {
    int b, c0, c1, s;
    bool whole;
};

// false: nothing (the request has fewer chunks).  An empty request is one empty chunk, for its zeros.
__device__ __forceinline__ bool find_item(const AttnArgs& a, Item& it)
{
    const int b = blockIdx.y, s = blockIdx.z, L = a.seq_lens[b], size = chunk_size(a, L);
    const int c0 = s * size, c1 = c0 + size < L ? c0 + size : L;
    it = Item{b, c0, c1, s, L <= size};
    return s == 0 || c0 < L;
}

// Maximum over the wave's 64 lanes, by data-parallel primitives (a lane permutation through LDS costs some hundred cycles a step).
__device__ __forceinline__ float wave_max(float x)
{
    auto step = [&](auto ctrl, auto rows) {
        const int v = __builtin_bit_cast(int, x);
        x = __builtin_fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, decltype(ctrl)::value, decltype(rows)::value, 0xf, false)));
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});      // row_shr:1, 2, 4, 8
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});      // row_bcast:15 into rows 1 and 3
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});      // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// A workgroup's result for one query head (threads of a head together hold its D sums): the output itself if the
// request is one chunk, else the chunk's (sum, maximum, weight) triple.
template <int D>
__device__ __forceinline__ void put_result(const AttnArgs& a, const Item& it, int h, int d, float of, float lf, float mn)
{
    const size_t bh = (size_t)it.b * a.Hq + h;
    if (it.whole) {
        a.out[bh * D + d] = to_half_bits(of / lf);       // lf > 0: the chunk holds at least one live position
    } else {
        float* po = a.part + (bh * AT_MAX_SPLIT + it.s) * (D + 2);
        po[d] = of;
        if (d == 0) { po[D] = mn; po[D + 1] = lf; }
    }
}
// an empty request: its output is zero, and there is nothing to merge
template <int D>
__device__ __forceinline__ void put_empty(const AttnArgs& a, const Item& it, int h0, int heads)
{
    for (int idx = threadIdx.x; idx < heads * D; idx += AT_THREADS)
        a.out[((size_t)it.b * a.Hq + h0 + idx / D) * D + idx % D] = 0;
}

template <int D, int GT>
__global__ __launch_bounds__(AT_THREADS) void attn_decode(AttnArgs a)
{
    constexpr int LPR = D / 8;                 // lanes per row
    constexpr int RG = 64 / LPR;               // rows (positions) per wave instruction
    constexpr int U = Unroll<GT>::U;           // wave instructions of K (and of V) per iteration
    constexpr int WPOS = RG * U;               // positions per wave and iteration
    constexpr int GPOS = AT_WAVES * WPOS;      // positions per workgroup and iteration
    __shared__ float s_o[AT_WAVES][GT][D];
    __shared__ float s_m[AT_WAVES][GT], s_l[AT_WAVES][GT];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int passes = (a.group + GT - 1) / GT;
    const int g = blockIdx.x / passes, pass = blockIdx.x % passes;
    const int h0 = g * a.group + pass * GT;    // first query head of this workgroup
    const int heads = (a.group - pass * GT < GT) ? a.group - pass * GT : GT;
    Item item;
    if (!find_item(a, item)) return;
    const int b = item.b, c0 = item.c0, c1 = item.c1;
    if (c0 >= c1) {                            // an empty request (uniform: no barrier yet)
        put_empty<D>(a, item, h0, heads);
        return;
    }
    const int r = lane / LPR, piece = lane % LPR;

    // the query heads' 8-element shares, as fp16 pairs (zero for the heads past the group's end)
    half2_t qv[GT][4];
#pragma unroll
    for (int j = 0; j < GT; ++j) {
        uintx4 raw = {0u, 0u, 0u, 0u};
        if (j < heads) raw = *reinterpret_cast<const uintx4*>(a.q + ((size_t)(b * a.Hq + h0 + j)) * D + piece * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned w = raw[e];
            qv[j][e] = __builtin_bit_cast(half2_t, w);
        }
    }
    const uint16_t* kbase = a.k + ((size_t)(b * a.Hkv + g) * a.S_max) * D + piece * 8;
    const uint16_t* vbase = a.v + ((size_t)(b * a.Hkv + g) * a.S_max) * D + piece * 8;

    float m[GT], l[GT], o[GT][8];
#pragma unroll
    for (int j = 0; j < GT; ++j) {
        m[j] = -__builtin_inff();
        l[j] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[j][e] = 0.f;
    }

    // Loads are unconditional: a position past the chunk's end is redirected to the chunk's last row
    // (valid, cached) and its weight is forced to zero.
    auto issue = [&](int it, uintx4 (&kr)[U], uintx4 (&vr)[U]) {
        const int base = c0 + (it * AT_WAVES + wv) * WPOS;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int pos = base + u * RG + r;
            pos = pos < c1 ? pos : c1 - 1;
            kr[u] = ld_stream(kbase + (size_t)pos * D);
            vr[u] = ld_stream(vbase + (size_t)pos * D);
        }
    };

    const int n_it = (c1 - c0 + GPOS - 1) / GPOS;
    uintx4 kn[U], vn[U];
    issue(0, kn, vn);
    for (int it = 0; it < n_it; ++it) {
        uintx4 kc[U], vc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { kc[u] = kn[u]; vc[u] = vn[u]; }
        issue(it + 1, kn, vn);        // past the last iteration every lane is redirected to one cached row
        const int base = c0 + (it * AT_WAVES + wv) * WPOS;

        // stage 1: scores t[j][u] = scale2 * q_j . k_pos  (scale2 = scale * log2 e: weights via exp2)
        float t[GT][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            half2_t kp[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned w = kc[u][e];
                kp[e] = __builtin_bit_cast(half2_t, w);
            }
            const bool live = base + u * RG + r < c1;
#pragma unroll
            for (int j = 0; j < GT; ++j) {
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_fdot2(kp[e], qv[j][e], acc, false);
#pragma unroll
                for (int sh = 1; sh < LPR; sh <<= 1) acc += __shfl_xor(acc, sh);
                t[j][u] = live ? acc * a.scale2 : -__builtin_inff();
            }
        }
        // stage 2: running maximum and sum, weights of this block
        float p[GT][U], corr[GT];
#pragma unroll
        for (int j = 0; j < GT; ++j) {
            float mb = t[j][0];
#pragma unroll
            for (int u = 1; u < U; ++u) mb = __builtin_fmaxf(mb, t[j][u]);
            const float mn = __builtin_fmaxf(m[j], mb);
            const float ms = (mn == -__builtin_inff()) ? 0.f : mn;     // nothing live yet: keep everything at zero
            corr[j] = exp2_fast(m[j] - ms);
            float sum = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) { p[j][u] = exp2_fast(t[j][u] - ms); sum += p[j][u]; }
            l[j] = l[j] * corr[j] + sum;
            m[j] = mn;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[j][e] *= corr[j];
        }
        // stage 3: weights times V (a dead position's V is zeroed so that 0 * garbage cannot leak)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool live = base + u * RG + r < c1;
            float vf[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned w = live ? vc[u][e] : 0u;
                const half2_t hv = __builtin_bit_cast(half2_t, w);
                vf[2 * e] = (float)hv[0];
                vf[2 * e + 1] = (float)hv[1];
            }
#pragma unroll
            for (int j = 0; j < GT; ++j)
#pragma unroll
                for (int e = 0; e < 8; ++e) o[j][e] = __builtin_fmaf(p[j][u], vf[e], o[j][e]);
        }
    }

    // merge the row groups of the wave (fixed order: butterfly over the lane index)
#pragma unroll
    for (int sh = LPR; sh < 64; sh <<= 1) {
#pragma unroll
        for (int j = 0; j < GT; ++j) {
            const float m2 = __shfl_xor(m[j], sh), l2 = __shfl_xor(l[j], sh);
            const float mn = __builtin_fmaxf(m[j], m2);
            const float ms = (mn == -__builtin_inff()) ? 0.f : mn;
            const float ca = exp2_fast(m[j] - ms), cb = exp2_fast(m2 - ms);
            l[j] = l[j] * ca + l2 * cb;
            m[j] = mn;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float o2 = __shfl_xor(o[j][e], sh);
                o[j][e] = o[j][e] * ca + o2 * cb;
            }
        }
    }
    // the waves meet in LDS
    if (r == 0) {
#pragma unroll
        for (int j = 0; j < GT; ++j) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s_o[wv][j][piece * 8 + e] = o[j][e];
            if (piece == 0) { s_m[wv][j] = m[j]; s_l[wv][j] = l[j]; }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < heads * D; idx += AT_THREADS) {
        const int j = idx / D, d = idx % D;
        float mn = s_m[0][j];
#pragma unroll
        for (int w = 1; w < AT_WAVES; ++w) mn = __builtin_fmaxf(mn, s_m[w][j]);
        const float ms = (mn == -__builtin_inff()) ? 0.f : mn;
        float lf = 0.f, of = 0.f;
#pragma unroll
        for (int w = 0; w < AT_WAVES; ++w) {        // fixed order: waves 0..3
            const float cw = exp2_fast(s_m[w][j] - ms);
            lf += s_l[w][j] * cw;
            of += s_o[w][j][d] * cw;
        }
        put_result<D>(a, item, h0 + j, d, of, lf, mn);
    }
}

// Grouped-query variant (D = 128, four or more query heads per cache head; up to 16 per pass): both products on the
// matrix cores, all of K and V through wave-private LDS stages brought straight from memory.
//
// A wave takes 16 positions at a time.  Scores: K rows as the A operand (position lane % 16, 8-element k group
// lane / 16), the queries of up to 16 heads resident as the B operand: four v_mfma_f32_16x16x32_f16.  A lane then holds
// four consecutive positions of one head, which is exactly the B operand (k = position) of v_mfma_f32_16x16x16_f16 for
// O^T = V^T P^T; V^T comes as the A operand from LDS by ds_read_b64_tr_b16 (a 16-lane group reads four rows x 16
// columns, lane j of it receives column j of the four rows).  So neither product needs a lane permutation, a lane's
// accumulators belong to one head, and rescaling them is a plain multiply (done only when some head's maximum moved).
// The weights enter the matrix core as the sum of two fp16 values (split_weights): one alone is off by
// 2^-12 of a weight, which the result shows where values cancel.  The second product costs 1-2 %
// (6 requests of 2048..8029 positions, 8 x 8 heads, 28.3 -> 28.9 us); one MFMA with k = 32 over both summands and the values twice 28.9 too.
// The first version kept V on the vector ALU (one lane permutation and eight packed dot products per head and pair of
// positions): ~2 us of ALU work per 64 positions of a workgroup.  8 cache heads x 8 query heads: 6 requests of
// 2048..8029 positions 51.2 -> 28.9 us (chunks by each request's length included), 32 of 512..2007 (not cut) 37.8 -> 32.7.
//
// Stages: 16 rows x 256 bytes of K, then of V, AT_NS per wave; a row's 16-byte piece p lies at piece p ^ (row % 16), which
// spreads the K operand reads and the transposing V reads over the banks.  The loads are written in assembly
// and counted by hand (s_waitcnt vmcnt); nothing else in the loop touches vector memory.  Two stages and 80 KiB, so that
// two workgroups fit a CU: four stages and one workgroup were 4 % slower on long chunks and 20 % on many short requests.
constexpr int AT_NS = 2, AT_POS = 16, AT_GQA_HEADS = 16;
constexpr int AT_STAGE = 2 * AT_POS * 16;                   // 16-byte units: K rows, V rows
constexpr int AT_Q_UNITS = AT_GQA_HEADS * 16;
constexpr int AT_WAVE_UNITS = AT_Q_UNITS + AT_NS * AT_STAGE;
constexpr int AT_GQA_LDS = AT_WAVES * AT_WAVE_UNITS * 16;

typedef short short4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void at_dma(const void* base_uniform, unsigned lane_byte_offset, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 : : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr) : "memory");
}

// Weights p in [0, 1] as two fp16 summands of AT_WEIGHT_SCALE * p (a power of two: exact), for the matrix core.  A weight is
// then off by 2^-22 of itself at most down to weights of 2^-17, and by 2^-40 of the largest weight below that.  The large summand
// is truncated, so that the small one is never negative, and the small one of a weight that is not zero is at least fp16's
// smallest value: an infinite value then adds up to the infinity it stands for, and not to inf - inf or 0 * inf.
constexpr float AT_WEIGHT_SCALE = 32768.0f;

__device__ __forceinline__ void split_weights(const float (&p)[4], half4& large, half4& small)
{
    typedef unsigned short ushort4_t __attribute__((ext_vector_type(4)));
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = p[i] * AT_WEIGHT_SCALE;
    const half2_t h0 = __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(w[0], w[1]));
    const half2_t h1 = __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(w[2], w[3]));
    large = half4{h0[0], h0[1], h1[0], h1[1]};
#pragma unroll
    for (int i = 0; i < 4; ++i) small[i] = (_Float16)(w[i] - (float)large[i]);
    const ushort4_t one = {1, 1, 1, 1}, l = __builtin_bit_cast(ushort4_t, large), s = __builtin_bit_cast(ushort4_t, small);
    small = __builtin_bit_cast(half4, __builtin_elementwise_max(s, __builtin_elementwise_min(l, one)));
}

__global__ __launch_bounds__(AT_THREADS) void attn_decode_gqa(AttnArgs a)
{
    constexpr int D = 128, GT = AT_GQA_HEADS, DT = D / 16;
    extern __shared__ uintx4 at_smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int passes = (a.group + GT - 1) / GT;
    const int g = blockIdx.x / passes, pass = blockIdx.x % passes;
    const int h0 = g * a.group + pass * GT;
    const int heads = (a.group - pass * GT < GT) ? a.group - pass * GT : GT;
    Item item;
    if (!find_item(a, item)) return;
    const int b = item.b, c0 = item.c0, c1 = item.c1;
    if (c0 >= c1) {
        put_empty<D>(a, item, h0, heads);
        return;
    }
    const int lo = lane & 15, hi = lane >> 4;

    const uint16_t* const kbase = a.k + ((size_t)(b * a.Hkv + g) * a.S_max) * D;
    const uint16_t* const vbase = a.v + ((size_t)(b * a.Hkv + g) * a.S_max) * D;
    uintx4* const my = at_smem + wv * AT_WAVE_UNITS;       // the queries (16 rows like K's), then the stages
    const unsigned my_addr = (unsigned)(size_t)(__attribute__((address_space(3))) void*)my;
    const int blocks = (c1 - c0 + AT_POS - 1) / AT_POS;
    const int nb = (blocks - wv + AT_WAVES - 1) / AT_WAVES;   // this wave's blocks: wv, wv + 4, ...

    // load i of a block: rows 4 i + hi, physical piece lo; rows past the chunk's end come from its last row
    auto issue = [&](int blk, int st) __attribute__((always_inline)) {
        const int base = c0 + (blk * AT_WAVES + wv) * AT_POS;
        const int limit = c1 - 1 - base;
        const uint16_t* const kb = kbase + (size_t)base * D;
        const uint16_t* const vb = vbase + (size_t)base * D;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + hi, from = row < limit ? row : limit;
            const unsigned off = (unsigned)(from * (D * 2) + ((lo ^ row) << 4));
            at_dma(kb, off, my_addr + (unsigned)(AT_Q_UNITS + st * AT_STAGE + i * 64) * 16u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + hi, from = row < limit ? row : limit;
            const unsigned off = (unsigned)(from * (D * 2) + ((lo ^ row) << 4));
            at_dma(vb, off, my_addr + (unsigned)(AT_Q_UNITS + st * AT_STAGE + AT_POS * 16 + i * 64) * 16u);
        }
    };

    float m = -__builtin_inff(), l = 0.f;           // of head lo (l: this lane's positions only)
    floatx4 o[DT];                                  // O^T: rows d = 16 t + 4 hi + i of head lo
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = floatx4{0.f, 0.f, 0.f, 0.f};

    // the queries, once per wave: a row per head (columns past the group's end repeat its last head and are not used)
    if (nb > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + hi, from = row < heads ? row : heads - 1;
            at_dma(a.q + ((size_t)b * a.Hq + h0) * D, (unsigned)(from * (D * 2) + ((lo ^ row) << 4)), my_addr + (unsigned)(i * 64) * 16u);
        }
    }
#pragma unroll
    for (int st = 0; st < AT_NS; ++st)
        if (st < nb) issue(st, st);
    half8 qf[4];                                    // B operand of the scores: head lo, k group hi, per 32-wide k step
    for (int it = 0; it < nb; ++it) {
        const int st = it % AT_NS;
        // the block behind this one may still be in flight (AT_NS = 2: eight loads)
        if (it + 1 < nb) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (it == 0) {
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) qf[s4] = __builtin_bit_cast(half8, my[lo * 16 + ((4 * s4 + hi) ^ lo)]);
        }
        const uintx4* const ks = my + AT_Q_UNITS + st * AT_STAGE;
        uintx4* const vs = my + AT_Q_UNITS + st * AT_STAGE + AT_POS * 16;
        const int base = c0 + (it * AT_WAVES + wv) * AT_POS;
        const bool tail = base + AT_POS > c1;
        if (tail) {                                 // dead rows of V are zeroed: 0 * whatever stands there must stay 0
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (base + 4 * i + hi >= c1) vs[i * 64 + lane] = uintx4{0u, 0u, 0u, 0u};
            __builtin_amdgcn_wave_barrier();
        }
        half8 kf[4];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) kf[s4] = __builtin_bit_cast(half8, ks[lo * 16 + ((4 * s4 + hi) ^ lo)]);
        half4 vf[DT];
        {
            const int row = 4 * hi + (lo >> 2);
            const char* const vrow = reinterpret_cast<const char*>(vs + row * 16) + (lo & 1) * 8;
#pragma unroll
            for (int t = 0; t < DT; ++t)
                vf[t] = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) short4_t*)(vrow + (((2 * t + ((lo >> 1) & 1)) ^ row) << 4))));
        }
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s4], qf[s4], acc, 0, 0, 0);
        float t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = (base + 4 * hi + i < c1) ? acc[i] * a.scale2 : -__builtin_inff();
        float mb = __builtin_fmaxf(__builtin_fmaxf(t[0], t[1]), __builtin_fmaxf(t[2], t[3]));
        mb = __builtin_fmaxf(mb, __shfl_xor(mb, 16));
        mb = __builtin_fmaxf(mb, __shfl_xor(mb, 32));
        const float mn = __builtin_fmaxf(m, mb);
        const float ms = (mn == -__builtin_inff()) ? 0.f : mn;
        const float corr = exp2_fast(m - ms);
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = exp2_fast(t[i] - ms);
        l = l * corr + ((p[0] + p[1]) + (p[2] + p[3]));
        m = mn;
        if (__builtin_amdgcn_ballot_w64(corr != 1.0f) != 0ull) {
#pragma unroll
            for (int q = 0; q < DT; ++q) o[q] *= corr;
        }
        half4 hi4, lo4;
        split_weights(p, hi4, lo4);
#pragma unroll
        for (int q = 0; q < DT; ++q) o[q] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf[q], hi4, o[q], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < DT; ++q) o[q] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf[q], lo4, o[q], 0, 0, 0);
        // every read of this stage has returned before it is filled again
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (it + AT_NS < nb) issue(it + AT_NS, st);
    }

    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    // the waves meet in LDS: [wave][head][d], then [wave][head] maximum and weight
    float* const s_o = reinterpret_cast<float*>(at_smem);
    float* const s_m = s_o + AT_WAVES * GT * D;
    float* const s_l = s_m + AT_WAVES * GT;
    __syncthreads();                                // every wave has read its last stage
#pragma unroll
    for (int t = 0; t < DT; ++t) *reinterpret_cast<floatx4*>(s_o + (wv * GT + lo) * D + 16 * t + 4 * hi) = o[t] * (1.0f / AT_WEIGHT_SCALE);
    if (hi == 0) { s_m[wv * GT + lo] = m; s_l[wv * GT + lo] = l; }
    __syncthreads();
    for (int idx = tid; idx < heads * D; idx += AT_THREADS) {
        const int j = idx / D, d = idx % D;
        float mn = s_m[j];
#pragma unroll
        for (int w = 1; w < AT_WAVES; ++w) mn = __builtin_fmaxf(mn, s_m[w * GT + j]);
        const float ms = (mn == -__builtin_inff()) ? 0.f : mn;
        float lf = 0.f, of = 0.f;
#pragma unroll
        for (int w = 0; w < AT_WAVES; ++w) {        // fixed order: waves 0..3
            const float cw = exp2_fast(s_m[w * GT + j] - ms);
            lf += s_l[w * GT + j] * cw;
            of += s_o[(w * GT + j) * D + d] * cw;
        }
        put_result<D>(a, item, h0 + j, d, of, lf, mn);
    }
}

// Second pass when requests may have been cut into chunks: one workgroup per (request, query head) merges the
// chunks' triples in chunk order and normalises.  One memory round trip for up to eight chunks: the length that says how
// many there are, the maxima and weights (one chunk per lane) and the first eight sums are requested together, what
// lies behind the last chunk is not used; weights go from lane to lane by scalar reads, not through LDS.
template <int D>
__global__ __launch_bounds__(D) void attn_combine(AttnArgs a)
{
    const int bh = blockIdx.x, d = threadIdx.x, lane = threadIdx.x & 63;
    const float* const first = a.part + (size_t)bh * AT_MAX_SPLIT * (D + 2);
    const float mine = first[(size_t)(lane % AT_MAX_SPLIT) * (D + 2) + D];
    const float mine_l = first[(size_t)(lane % AT_MAX_SPLIT) * (D + 2) + D + 1];
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = first[(size_t)i * (D + 2) + d];
    const int L = a.seq_lens[bh / a.Hq], size = chunk_size(a, L);
    if (L <= size) return;                              // one chunk: the first pass has written this output
    const int live = (int)((unsigned)(L + size - 1) / (unsigned)size);
    float m = lane < live ? mine : -__builtin_inff();
    m = wave_max(m);
    const float w = lane < live ? exp2_fast(mine - m) : 0.f;
    auto of_lane = [](float x, int i) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), i)); };
    float l = 0.f, o = 0.f;
    for (int s0 = 0;;) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (s0 + i < live) {
                const float c = of_lane(w, s0 + i);
                l += of_lane(mine_l, s0 + i) * c;
                o += v[i] * c;
            }
        s0 += 8;
        if (s0 >= live) break;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = first[(size_t)(s0 + i < live ? s0 + i : live - 1) * (D + 2) + d];
    }
    a.out[(size_t)bh * D + d] = to_half_bits(o / l);
}

template <int D, int GT>
void launch_decode(const AttnArgs& a, dim3 grid, hipStream_t stream)
{
    hipLaunchKernelGGL((attn_decode<D, GT>), grid, dim3(AT_THREADS), 0, stream, a);
}

template <int D>
hipError_t launch_d(const AttnArgs& a, int gt, hipStream_t stream)
{
    const int passes = (a.group + gt - 1) / gt;
    // The chunk number varies slowest: workgroups are dealt to the eight XCDs in the order of their numbers, and requests shorter than
    // others have work in their first chunks only.  Varying fastest, with four chunks, it left all of that to two XCDs (17 requests of
    // 66 positions, 4 cache heads of 64: 9.7 us, with three or five chunks 7.9).
    const dim3 grid((unsigned)(a.Hkv * passes), (unsigned)a.B, (unsigned)a.nsplit);
    switch (gt) {
    case 1: launch_decode<D, 1>(a, grid, stream); break;
    case 2: launch_decode<D, 2>(a, grid, stream); break;
    case 4: if constexpr (D == 64) launch_decode<D, 4>(a, grid, stream); break;
    case 8: if constexpr (D == 64) launch_decode<D, 8>(a, grid, stream); break;
    default: {                  // D = 128 only
        static std::once_flag attr_once;
        std::call_once(attr_once, [] {
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(attn_decode_gqa), hipFuncAttributeMaxDynamicSharedMemorySize, AT_GQA_LDS);
        });
        hipLaunchKernelGGL(attn_decode_gqa, grid, dim3(AT_THREADS), AT_GQA_LDS, stream, a);
        break;
    }
    }
    if (a.nsplit > 1)
        hipLaunchKernelGGL((attn_combine<D>), dim3((unsigned)(a.B * a.Hq)), dim3(D), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attention(const AttnArgs& a, hipStream_t stream)
{
    const int gt = attention_heads_per_workgroup(a.D, a.group);
    if (a.D == 128) return launch_d<128>(a, gt, stream);
    if (a.D == 64) return launch_d<64>(a, gt, stream);
    return hipErrorInvalidValue;
}

}  // namespace thi
