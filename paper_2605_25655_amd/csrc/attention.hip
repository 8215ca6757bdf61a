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
// Work split: a workgroup (4 waves) takes one chunk of positions of one (request, cache head) -- find_item -- and up
// to GT query heads of that cache head's group.  16 (D = 128) or 8 (D = 64) lanes cover one row with
// 16-byte loads, so a wave instruction reads 4 or 8 consecutive positions = 1 KiB of contiguous memory;
// U such loads of K and of V are in flight per wave, one iteration ahead of the arithmetic.  A lane
// forms its 8-element share of q.k with packed fp16 dot products accumulated in fp32, the shares meet
// by lane shuffles, the weights stay fp32, and V is accumulated in fp32.  Row groups, waves and chunks
// each keep their own (maximum, sum, output) triple; triples are merged in a fixed order (row groups
// by shuffle, waves through LDS, chunks by a second small kernel), so results are reproducible.
#include "thi_internal.h"

#include <mutex>

namespace thi {

namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int AT_THREADS = 256;
constexpr int AT_WAVES = 4;

template <int GT> struct Unroll { static constexpr int U = (GT >= 4) ? 2 : 4; };

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// The number of live chunks of a (request, query head) is left behind its last partial result, as this word in the
// place of the next chunk's maximum (a NaN that no conversion from fp16 can produce).
constexpr int AT_END_MARK = 0x7fc0dead;

// What a workgroup works on: positions [c0, c1) of request b, chunk s of n (n = 0: nothing).
//
// With at least a workgroup per compute unit from the (request, cache head) pairs alone (a.nsplit == 1) a request is
// never cut.  Otherwise the requests are cut into chunks of one common size C, the smallest with which all chunks of a
// cache head fit a.workgroups -- chosen here, from the lengths themselves, because the host does not know
// them: cutting S_max instead leaves every request that is shorter than its cache with fewer workgroups and the
// longest one deciding (24 requests of 750..2940 positions in a cache of 3000, 8 cache heads: 55.9 us, with chunks of
// the live lengths 37.9).  C depends on the lengths as a set only, so a request's result does not
// depend on its place in the batch.  A request's chunks are then made equal.  Every wave computes this by
// itself (lengths one per lane); at most AT_MAX_SPLIT chunks per request, of at least a.chunk positions (a multiple of 64).
struct Item {
    int b, c0, c1, s, n;
};

// Inclusive scan over the wave's 64 lanes (lanes shifted in from outside a row count as 0) by data-parallel
// primitives: a few cycles a step where a lane permutation through LDS takes some hundred.
template <typename Op>
__device__ __forceinline__ int wave_scan(int v, Op op)
{
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));      // row_shr:1
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));      // row_shr:2
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));      // row_shr:4
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));      // row_shr:8
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));      // row_bcast:15 into rows 1 and 3
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));      // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ Item find_item(const AttnArgs& a)
{
    if (a.nsplit == 1) {
        const int b = blockIdx.z, L = a.seq_lens[b];
        return Item{b, 0, L, 0, 1};
    }
    auto round64 = [](int v) { return (v + 63) & ~63; };
    if (a.B == 1) {                                      // one request: nothing to add up
        const int L = a.seq_lens[0];
        int size = round64((int)((unsigned)(L + a.workgroups - 1) / (unsigned)a.workgroups));
        size = size > a.chunk ? size : a.chunk;
        const int n = L <= size ? 1 : (int)((unsigned)(L + size - 1) / (unsigned)size), s = blockIdx.x;
        if (s >= n) return Item{0, 0, 0, 0, 0};
        return Item{0, s * size, (s + 1) * size < L ? (s + 1) * size : L, s, n};
    }
    const int lane = threadIdx.x & 63, want = a.workgroups;
    auto add = [](int p, int q) { return p + q; };
    auto max2 = [](int p, int q) { return p > q ? p : q; };
    auto length = [&](int b) { return b < a.B ? a.seq_lens[b] : 0; };
    const int L0 = length(lane);                         // (one group of 64 requests is the rule: no second load for it)
    int total = 0, longest = 0;
    for (int b0 = 0; b0 < a.B; b0 += 64) {
        const int L = b0 == 0 ? L0 : length(b0 + lane);
        total += __builtin_amdgcn_readlane(wave_scan(L, add), 63);
        longest = max2(longest, __builtin_amdgcn_readlane(wave_scan(L, max2), 63));
    }
    int C = round64((int)((unsigned)(total + want - 1) / (unsigned)want));
    C = max2(C, round64((longest + AT_MAX_SPLIT - 1) / AT_MAX_SPLIT));
    C = max2(C, a.chunk);
    // chunks of request b (an empty one has a chunk too, to write its zeros)
    auto chunks = [&](int b, int L) { return b >= a.B ? 0 : L <= C ? 1 : (int)((unsigned)(L + C - 1) / (unsigned)C); };
    while (C < longest) {
        int n = 0;
        for (int b0 = 0; b0 < a.B; b0 += 64)
            n += __builtin_amdgcn_readlane(wave_scan(chunks(b0 + lane, b0 == 0 ? L0 : length(b0 + lane)), add), 63);
        if (n <= want) break;
        C += round64(C / 16);
    }
    int before = 0;
    const int x = blockIdx.x;
    for (int b0 = 0; b0 < a.B; b0 += 64) {
        const int L = b0 == 0 ? L0 : length(b0 + lane);
        const int n = chunks(b0 + lane, L), upto = before + wave_scan(n, add);
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(x >= upto - n && x < upto);
        if (hit != 0ull) {
            const int who = __builtin_ctzll(hit);
            const int Lb = __builtin_amdgcn_readlane(L, who), nb = __builtin_amdgcn_readlane(n, who);
            const int s = x - (__builtin_amdgcn_readlane(upto, who) - nb);
            const int size = round64((int)((unsigned)(Lb + nb - 1) / (unsigned)nb));      // <= C: the chunks of a request are equal
            const int c0 = s * size < Lb ? s * size : Lb;
            return Item{b0 + who, c0, c0 + size < Lb ? c0 + size : Lb, s, nb};
        }
        before = __builtin_amdgcn_readlane(upto, 63);
    }
    return Item{0, 0, 0, 0, 0};
}

// A workgroup's result for one query head (threads of a head together hold its D sums): the output itself if the
// request is one chunk, else the chunk's (sum, maximum, weight) triple; behind the last one the end mark.
// CUT = false: the caller knows that no request is cut.
template <int D, bool CUT>
__device__ __forceinline__ void put_result(const AttnArgs& a, const Item& it, int h, int d, float of, float lf, float mn)
{
    const size_t bh = (size_t)it.b * a.Hq + h;
    if (!CUT || it.n == 1) {
        a.out[bh * D + d] = to_half_bits(of / lf);       // lf > 0: the chunk holds at least one live position
    } else {
        float* po = a.part + (bh * AT_MAX_SPLIT + it.s) * (D + 2);
        po[d] = of;
        if (d == 0) { po[D] = mn; po[D + 1] = lf; }
    }
    if (CUT && a.nsplit > 1 && it.s == it.n - 1 && it.n < AT_MAX_SPLIT && d == 0)
        a.part[(bh * AT_MAX_SPLIT + it.n) * (D + 2) + D] = __builtin_bit_cast(float, AT_END_MARK);
}
// an empty request: its output is zero, and there is nothing to merge
template <int D, bool CUT>
__device__ __forceinline__ void put_empty(const AttnArgs& a, const Item& it, int h0, int heads)
{
    for (int idx = threadIdx.x; idx < heads * D; idx += AT_THREADS) {
        const size_t bh = (size_t)it.b * a.Hq + h0 + idx / D;
        a.out[bh * D + idx % D] = 0;
        if (CUT && a.nsplit > 1 && idx % D == 0)
            a.part[(bh * AT_MAX_SPLIT + 1) * (D + 2) + D] = __builtin_bit_cast(float, AT_END_MARK);
    }
}

// CUT = false where requests are not cut: such calls have hundreds of short workgroups, and the search for a chunk in front
// of each, though skipped, cost 0.1-0.2 us a call (32 requests of 512 positions, 32 heads: 28.6 us with it, 28.4 without).
template <int D, int GT, bool CUT>
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
    const int g = blockIdx.y / passes, pass = blockIdx.y % passes;
    const int h0 = g * a.group + pass * GT;    // first query head of this workgroup
    const int heads = (a.group - pass * GT < GT) ? a.group - pass * GT : GT;
    const Item item = CUT ? find_item(a) : Item{(int)blockIdx.z, 0, a.seq_lens[blockIdx.z], 0, 1};
    const int b = item.b, c0 = item.c0, c1 = item.c1;
    if (CUT && item.n == 0) return;
    if (c0 >= c1) {                            // an empty request (uniform: no barrier yet)
        put_empty<D, CUT>(a, item, h0, heads);
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
        put_result<D, CUT>(a, item, h0 + j, d, of, lf, mn);
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
// The weights enter the matrix core as fp16 (in [0,1]: 2^-11 relative rounding), sums and their weights are fp32.
// The first version kept V on the vector ALU (one lane permutation and eight packed dot products per head and pair of
// positions): ~2 us of ALU work per 64 positions of a workgroup.  8 cache heads x 8 query heads: 6 requests of
// 2048..8029 positions 50.8 -> 27.2 us (with the chunks of the live lengths), 32 of 512..2007 (not cut) 37.3 -> 31.6,
// 64 of 75..294 15.5 -> 12.0.
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

__global__ __launch_bounds__(AT_THREADS) void attn_decode_gqa(AttnArgs a)
{
    constexpr int D = 128, GT = AT_GQA_HEADS, DT = D / 16;
    extern __shared__ uintx4 at_smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int passes = (a.group + GT - 1) / GT;
    const int g = blockIdx.y / passes, pass = blockIdx.y % passes;
    const int h0 = g * a.group + pass * GT;
    const int heads = (a.group - pass * GT < GT) ? a.group - pass * GT : GT;
    const Item item = find_item(a);
    const int b = item.b, c0 = item.c0, c1 = item.c1;
    if (item.n == 0) return;
    if (c0 >= c1) {
        put_empty<D, true>(a, item, h0, heads);
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
        const half4 pf = {(_Float16)p[0], (_Float16)p[1], (_Float16)p[2], (_Float16)p[3]};
#pragma unroll
        for (int q = 0; q < DT; ++q) o[q] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf[q], pf, o[q], 0, 0, 0);
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
    for (int t = 0; t < DT; ++t) *reinterpret_cast<floatx4*>(s_o + (wv * GT + lo) * D + 16 * t + 4 * hi) = o[t];
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
        put_result<D, true>(a, item, h0 + j, d, of, lf, mn);
    }
}

// Second pass when requests may have been cut into chunks: one workgroup per (request, query head) merges the
// chunks' triples in chunk order and normalises.  How many there are the end mark says; maxima and weights are
// fetched one chunk per lane, the sums eight chunks at a time, so that the memory round trips overlap.
template <int D>
__global__ __launch_bounds__(D) void attn_combine(AttnArgs a)
{
    const int bh = blockIdx.x, d = threadIdx.x, lane = threadIdx.x & 63;
    const float* const first = a.part + (size_t)bh * AT_MAX_SPLIT * (D + 2);
    const float mine = first[(size_t)(lane < AT_MAX_SPLIT ? lane : 0) * (D + 2) + D];
    const float mine_l = first[(size_t)(lane < AT_MAX_SPLIT ? lane : 0) * (D + 2) + D + 1];
    const unsigned long long mark = __builtin_amdgcn_ballot_w64(lane < AT_MAX_SPLIT && lane > 0 && __builtin_bit_cast(int, mine) == AT_END_MARK);
    const int live = mark != 0ull ? __builtin_ctzll(mark) : AT_MAX_SPLIT;
    if (live == 1) return;                              // the first pass has written this output
    float m = lane < live ? mine : -__builtin_inff();
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) m = __builtin_fmaxf(m, __shfl_xor(m, sh));
    const float w = lane < live ? exp2_fast(mine - m) : 0.f;
    float l = 0.f, o = 0.f;
    for (int s0 = 0; s0 < live; s0 += 8) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = first[(size_t)(s0 + i < live ? s0 + i : live - 1) * (D + 2) + d];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (s0 + i < live) {
                const float c = __shfl(w, s0 + i);
                l += __shfl(mine_l, s0 + i) * c;
                o += v[i] * c;
            }
    }
    a.out[(size_t)bh * D + d] = to_half_bits(o / l);
}

template <int D, int GT>
void launch_decode(const AttnArgs& a, dim3 grid, hipStream_t stream)
{
    if (a.nsplit == 1) hipLaunchKernelGGL((attn_decode<D, GT, false>), grid, dim3(AT_THREADS), 0, stream, a);
    else hipLaunchKernelGGL((attn_decode<D, GT, true>), grid, dim3(AT_THREADS), 0, stream, a);
}

template <int D>
hipError_t launch_d(const AttnArgs& a, int gt, hipStream_t stream)
{
    const int passes = (a.group + gt - 1) / gt;
    // uncut: one workgroup per request, cache head and pass; else a.workgroups for the chunks of a cache head
    dim3 grid((unsigned)(a.nsplit == 1 ? 1 : a.workgroups), (unsigned)(a.Hkv * passes), (unsigned)(a.nsplit == 1 ? a.B : 1));
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
