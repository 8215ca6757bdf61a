// LDS-tiled fp16 MFMA GEMM for prefill (large M) on gfx950.
//
// Function: the paper's large-M linear operator (Sec. III-B.2) -- out = x W^T
// with fp16 operands and fp32 accumulation (Sec. III-B.4) -- plus the fused
// low-density operators behind it (Sec. III-C.1): SiLU(gate)*up, the rotary
// embedding, the residual.  RMSNorm in front runs as a small pass of its own
// (rmsnorm_rows below) so that both operand tiles can go from memory straight
// into LDS; fused into the staging of the activation tile it cost 25 % and
// three times the HBM reads.
// The paper's DDR->GSM->AM dataflow is specific to its scratchpad machine; here
// a workgroup owns a BN x BM output tile (up to 256 x 256), stages BN x 64 and
// BM x 64 operand tiles in LDS (two to four stages, XOR-swizzled 16-byte pieces so
// that both the staging writes and the MFMA operand reads are bank-conflict
// free) and runs v_mfma_f32_16x16x32_f16 on wave tiles of up to 64 x 128.
//
// Why 16x16x32 and not 32x32x16 (the same flops per cycle, the same operand bytes from LDS for a wave tile):
// the chip runs these kernels at its power limit, and the 32x32 form moves four times the accumulator bytes
// per instruction for twice the flops.  A loop of nothing but MFMAs on random operands sustains 1893 TFLOP/s
// with 16x16x32 against 1643 with 32x32x16.
//
// Operand roles: the weight tile is the MFMA "A" operand (rows = output
// features n), the activation tile the "B" operand (columns = tokens m), so a
// lane ends up with 4 consecutive n of one token per fragment -- an 8-byte
// store -- and, for SwiGLU, with g and u of the same (token, j) in registers of
// the same lane (a tile interleaves 16 gate rows with the 16 matching up rows).
//
// Scheduling: a fixed number of workgroups (one or two per CU).  Tiles that fill whole rounds of the
// grid are computed and finished in one piece; the ragged remainder (everything, when there are fewer
// tiles than workgroups) may be cut along K so that no CU idles -- into equal k ranges per tile, the
// same for every tile, when there are several token tiles (workgroups on neighbouring tiles then walk
// the same k range together and keep sharing operand panels through the L2), into equal contiguous
// stream-K shares when there is one token tile (every weight panel is read once anyway).  Tiles that
// were cut leave fp32 partial tiles in the workspace; a second, chip-wide kernel adds them in workgroup
// order (bitwise reproducible) and applies the epilogue.
//
// Workgroups are numbered so that the eight XCDs (one L2 each; hardware deals
// consecutive workgroup ids round-robin to them) each walk a contiguous range
// of tiles, token-tile fastest, so the weight panel an XCD streams is shared by
// the workgroups running on it at that moment.
#include "thi_internal.h"

#include <mutex>
#include <type_traits>

namespace thi {

namespace {

// A staged tile row holds GK halfs = GK/8 16-byte pieces.  Piece p of tile row `row` lives at 16-byte
// unit row*P + (p ^ f(row)), with f chosen so that 16 consecutive rows reading the same logical piece
// (an MFMA operand read) and the linear staging writes both spread over all LDS banks:
//   P = 16 (256-byte rows): 16 consecutive rows, 16 different pieces;
//   P = 8  (128-byte rows): f is a bijection on every aligned group of 8 rows and on the even and the odd
//                           rows of every aligned group of 16.
template <int P>
__device__ __forceinline__ int swz_f(int row)
{
    static_assert(P == 8 || P == 16, "staged rows of 64 or 128 k");
    if (P == 16) return row & 15;
    return ((row >> 1) & 7) ^ ((row & 1) << 2);
}
template <int P>
__device__ __forceinline__ int swz(int row, int piece) { return row * P + (piece ^ swz_f<P>(row)); }

__device__ __forceinline__ uint16_t to_half_bits(float v)
{
    _Float16 h = (_Float16)v;
    return __builtin_bit_cast(uint16_t, h);
}

// One 16-byte piece per lane straight from global memory into LDS (no VGPR staging): lane L of the
// wave lands at lds_base + 16*L (wave-uniform).  The address is split into a wave-uniform base (scalar
// registers) and a 32-bit per-lane byte offset: no vector ALU work per load.  Written in assembly because
// the builtin always takes 64-bit per-lane addresses.  The kernels that use it use M0 for nothing else and
// wait for these loads explicitly (s_waitcnt vmcnt) before the barrier that publishes the stage.
__device__ __forceinline__ void dma16_sbase(const void* base_uniform, unsigned lane_byte_offset, uintx4* lds_base)
{
    const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds_base;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_byte_offset), "s"(base_uniform), "s"(lds_addr)
                 : "memory");
}

// The k-steps of the shared tiles (tile t = units [t * ktiles, (t + 1) * ktiles)) dealt to G workers.
//   parts == 0: contiguous equal shares whatever the tile boundaries (the first `rem` workers take q + 1
//               units, the others q); a share may span the end of one tile and the start of the next.
//   parts >= 1: every shared tile is cut into `parts` equal k ranges, worker w takes range w % parts of
//               tile w / parts (workers past sk_tiles * parts take none).  Workers on neighbouring tiles
//               then walk the same k range at the same time, so the operand panels they have in common
//               are still fetched once per L2 instead of once per workgroup.
struct Deal {
    int q, rem, parts, ktiles, shared;
    __device__ __forceinline__ Deal(int sk_tiles, int ktiles_, int G, int parts_)
        : q(sk_tiles * ktiles_ / G), rem(sk_tiles * ktiles_ % G), parts(parts_), ktiles(ktiles_), shared(sk_tiles) {}
    __device__ __forceinline__ int begin(int w) const {
        if (parts == 0) return w * q + (w < rem ? w : rem);
        if (w >= shared * parts) return shared * ktiles;
        return (w / parts) * ktiles + (w % parts) * ktiles / parts;
    }
    __device__ __forceinline__ int end(int w) const {
        if (parts == 0) return begin(w + 1);
        if (w >= shared * parts) return shared * ktiles;
        return (w / parts) * ktiles + (w % parts + 1) * ktiles / parts;
    }
    // first and last worker with a share of tile t
    __device__ __forceinline__ int first(int t) const { return parts == 0 ? owner(t * ktiles) : t * parts; }
    __device__ __forceinline__ int last(int t) const { return parts == 0 ? owner(t * ktiles + ktiles - 1) : t * parts + parts - 1; }
    __device__ __forceinline__ int owner(int u) const {
        const int edge = rem * (q + 1);
        return u < edge ? u / (q + 1) : rem + (u - edge) / q;
    }
};

// Four consecutive outputs n .. n + 3 of token m (below M): rotation, residual, one rounding, store.
template <int EPI>
__device__ __forceinline__ void store_quad(const GemmArgs& a, int m, int n, const floatx4& f)
{
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = f[c];
    if (has_rope(EPI)) {                         // two complete pairs of one token; cos / sin from the table the RMSNorm pass left
        rope_pair_table(a.rope, m, n, v[0], v[1]);
        rope_pair_table(a.rope, m, n + 2, v[2], v[3]);
    }
    if (n + 3 < a.N) {
        half4 hv;
        if (a.residual) {
            const half4 rv = *reinterpret_cast<const half4_any*>(a.residual + (size_t)m * a.ldo + n);
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] += (float)rv[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) hv[c] = (_Float16)v[c];
        *reinterpret_cast<half4_any*>(a.out + (size_t)m * a.ldo + n) = hv;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (n + c < a.N) {
                if (a.residual) v[c] += half_bits_to_float(a.residual[(size_t)m * a.ldo + n + c]);
                a.out[(size_t)m * a.ldo + n + c] = to_half_bits(v[c]);
            }
    }
}

// Four consecutive h = silu(g) * u of token m (below M).
__device__ __forceinline__ void store_quad_swiglu(const GemmArgs& a, int m, int j, const floatx4& g, const floatx4& u)
{
    half4 hv;
#pragma unroll
    for (int c = 0; c < 4; ++c) hv[c] = (_Float16)(g[c] / (1.0f + __expf(-g[c])) * u[c]);
    if (j + 3 < a.N) {
        *reinterpret_cast<half4_any*>(a.out + (size_t)m * a.ldo + j) = hv;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (j + c < a.N) a.out[(size_t)m * a.ldo + j + c] = __builtin_bit_cast(uint16_t, hv[c]);
    }
}

// Epilogue for the two 16x16 accumulator fragments (2 tp, tm) and (2 tp + 1, tm) of a wave: a lane holds four
// consecutive n of one token of each.  For SwiGLU the first holds gate rows and the second the matching up rows.
template <int BN, int BM, int WN, int WM, int EPI>
__device__ __forceinline__ void store_pair(const GemmArgs& a, int tile_n, int tile_m, int wn, int wm, int tp,
                                           int tm, int lr, int hi, const floatx4& f0, const floatx4& f1)
{
    const int m = tile_m * BM + wm * (BM / WM) + tm * 16 + lr;
    if (m >= a.M) return;
    const int row = wn * (BN / WN) + tp * 32;            // first tile row of the pair
    if (is_swiglu(EPI)) {
        store_quad_swiglu(a, m, tile_n * (BN / 2) + (row >> 1) + 4 * hi, f0, f1);
        return;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) store_quad<EPI>(a, m, tile_n * BN + row + 16 * q + 4 * hi, q ? f1 : f0);
}

// The same for one fragment (waves with an odd number of them): for SwiGLU its first eight rows are gate rows and the
// others the matching up rows, exchanged between the wave's halves.
template <int BN, int BM, int WN, int WM, int EPI>
__device__ __forceinline__ void store_one(const GemmArgs& a, int tile_n, int tile_m, int wn, int wm, int tn,
                                          int tm, int lr, int hi, const floatx4& f)
{
    const int m = tile_m * BM + wm * (BM / WM) + tm * 16 + lr;
    const int row = wn * (BN / WN) + tn * 16;
    if (is_swiglu(EPI)) {
        floatx4 u;
#pragma unroll
        for (int c = 0; c < 4; ++c) u[c] = __shfl_xor(f[c], 32);
        if (hi < 2 && m < a.M) store_quad_swiglu(a, m, tile_n * (BN / 2) + (row >> 1) + 4 * hi, f, u);
    } else if (m < a.M) {
        store_quad<EPI>(a, m, tile_n * BN + row + 4 * hi, f);
    }
}

// Second pass for tiles that were cut along K: one workgroup per (shared tile, pair of accumulator fragments, FIXUP_WAVES of
// the main kernel's waves) adds the partial fragments of the tile's contributors in workgroup order and applies the epilogue.
// The thread <-> element mapping is the main kernel's, so the partials are read back as they were written.
// Two waves: a product of few tiles in many parts has all its partial tiles read by few compute units, and with the eight
// waves of the main kernel to a workgroup by a quarter of those (one tile in 26 parts, 447 x 120 x 1664: 18.3 us with eight waves, 15.6
// with two; 329 x 113 x 3584 30.8 -> 23.5; 4 waves the same, 1 wave 25.2).
constexpr int FIXUP_WAVES = 2;

template <int BN, int BM, int WN, int WM, int EPI>
__global__ __launch_bounds__(64 * FIXUP_WAVES) void gemm_fixup(GemmArgs a, int tiles_m, int ktiles, int sk_tiles, int G, int parts)
{
    constexpr int THREADS = 64 * WN * WM, GROUPS = WN * WM / FIXUP_WAVES;
    constexpr int TP = BN / WN / 32, TM = BM / WM / 16;
    static_assert(WN * WM % FIXUP_WAVES == 0, "whole workgroups");
    const int tid = (blockIdx.x % GROUPS) * 64 * FIXUP_WAVES + threadIdx.x;      // the main kernel's thread
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid / 64);
    const int wn = wv % WN, wm = wv / WN, lr = lane & 15, hi = lane >> 4;
    const int tf = blockIdx.x / GROUPS, t = tf / (TP * TM), frag = tf % (TP * TM);
    const int tp = frag / TM, tm = frag % TM;
    const Deal deal(sk_tiles, ktiles, G, parts);
    const int w_first = deal.first(t), w_last = deal.last(t);
    floatx4 g0 = {0.f, 0.f, 0.f, 0.f}, g1 = {0.f, 0.f, 0.f, 0.f};      // the pair's two fragments
    // a contributor's partial of this tile: slot 0 if the tile is the first of its share, else slot 1
    auto part = [&](int wc) -> const floatx4* {
        const int cslot = (deal.begin(wc) / ktiles == t) ? 0 : 1;
        return reinterpret_cast<const floatx4*>(a.partials + ((size_t)wc * 2 + cslot) * (BN * BM)) +
               (size_t)(2 * tp * TM + tm) * THREADS + tid;
    };
    constexpr int NEXT = TM * THREADS;          // from fragment (2 tp, tm) to (2 tp + 1, tm)
    auto add = [&](const floatx4& v0, const floatx4& v1) { g0 += v0; g1 += v1; };
    int wc = w_first;
    for (; wc + 3 <= w_last; wc += 4) {      // four contributors' loads in flight, added in order
        const floatx4 *p0 = part(wc), *p1 = part(wc + 1), *p2 = part(wc + 2), *p3 = part(wc + 3);
        const floatx4 a0 = p0[0], a1 = p0[NEXT], b0 = p1[0], b1 = p1[NEXT];
        const floatx4 c0 = p2[0], c1 = p2[NEXT], d0 = p3[0], d1 = p3[NEXT];
        add(a0, a1); add(b0, b1); add(c0, c1); add(d0, d1);
    }
    for (; wc <= w_last; ++wc) {
        const floatx4* p = part(wc);
        const floatx4 v0 = p[0], v1 = p[NEXT];
        add(v0, v1);
    }
    store_pair<BN, BM, WN, WM, EPI>(a, t / tiles_m, t % tiles_m, wn, wm, tp, tm, lr, hi, g0, g1);
}

// Workers are numbered so that consecutive ones (neighbouring tiles) share an XCD: hardware deals workgroup ids round-robin to the eight.
struct XcdShare {
    int first, count;        // the workers of an XCD
    __device__ __forceinline__ XcdShare(int G, int xcd) : first(xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8)), count(G / 8 + (xcd < G % 8)) {}
};

// What a compute unit without a tile does: it touches the weights of the tiles on its XCD, one dword of every 128 bytes, k-tile by k-tile for all
// rows, so that the workgroups multiplying them find them in the L2.  They have 64 KiB of loads in flight each, in order, and wait
// for memory; a touch brings a line for a dword of that, 75-110 GB/s a CU.  Nothing depends on it: no value is used, and it ends
// with its lines wherever the others are.  512 x 5120 x 5120 (160 tiles) 45.6 -> 38.5 us, 333 x 5001 x 1384 (120) 19.0 -> 16.1,
// 200 x 9000 x 2008 24.6 -> 20.8, 587 x 4984 x 3352 (195) 37.0 -> 32.0.  Touching the activations too gains nothing (39.1, 15.5, 20.7); touched by
// the workgroups that multiply, the lines are waited for in order: 43.9 instead of 38.5, with two token tiles no gain.
template <int BN>
__device__ __forceinline__ void touch_weights(const GemmArgs& a, int tiles_m, int G)
{
    const XcdShare on(G, blockIdx.x % 8);
    const int r0 = on.first / tiles_m * BN, past = ((on.first + on.count - 1) / tiles_m + 1) * BN;
    const int rows = (past < a.N ? past : a.N) - r0, lines = (a.K + 63) / 64;
    if (rows <= 0) return;
    const int each = (gridDim.x - G) / 8 * blockDim.x;         // threads on this XCD that touch
    const int dk = each / rows, dr = each % rows;
    int i = (blockIdx.x - G) / 8 * blockDim.x + threadIdx.x;
    int k = i / rows, r = i % rows;
    const long total = (long)rows * lines;
    constexpr int U = 8;
    for (long i0 = i - (long)(threadIdx.x % 64); i0 < total; i0 += (long)U * each) {       // (uniform in a wave)
        unsigned v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = *reinterpret_cast<const unsigned*>(a.w0 + (size_t)(r0 + r) * a.K + (k < lines ? k : lines - 1) * 64);
            k += dk;
            r += dr;
            if (r >= rows) { r -= rows; ++k; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) asm volatile("" ::"v"(v[u]));        // (loaded, not used)
    }
}

// BN x BM output tile, WN x WM waves; wave tile (BN/WN) x (BM/WM) built from 16x16 MFMA tiles.
// KTAIL: K is not a multiple of GK.  The last k-tile's pieces past K are loaded from the k-tile's first piece (valid
// memory) and overwritten with zeros once they have landed; K is a multiple of 8, so a 16-byte piece is entirely inside
// or outside.  (Until the direct loads took the ragged K as well it went through VGPRs in the two-per-CU 128x128
// configuration alone: 333 x 5001 x 1384 27.5 us, now 23.6.)
// Operand fragments are read from LDS one k-step of 32 ahead of their MFMAs (two fragment buffers).  The k-tile's
// one barrier sits in front of its last k-step: every read of the stage has been issued by then, the next
// k-tile must have landed, and its first fragments are read behind the barrier while the last k-step is multiplied.
// Against 32x32x16 MFMAs with the same tiles (one box, alternating): gate/up 2048 x 57344 x 8192 1553 -> 1482 us,
// 2048 x 8192 x 8192 244 -> 214, 2048 x 8192 x 28672 802 -> 721, 512 x 27648 x 5120 146 -> 138, same bits.
// What bounds it: with all direct loads of a k-tile right behind the barrier, the two waves of every SIMD queued for the load
// path at the same time and the matrix cores stood still: 2780 cycles a k-tile of 256x256x64 at 1.81 GHz, of which 2048 are
// MFMAs and 50 a wait for the loads.  So the loads go out one by one between the MFMAs of the whole k-tile, in a fixed order
// (`step`), and since a stage is free only behind the barrier, one operand has a stage more (NSW weight and NSX activation stages:
// 3 + 2 of 32 KiB are all of the LDS) and its loads go out half a k-tile later than the other's.  2340 cycles at 1.59 GHz: the power limit is
// what is left.  gate/up 2048 x 57344 x 8192 1471 -> 1381 us, 2048 x 8192 x 28672 732 -> 687, 512 x 5120 x 13824 88 -> 84 (256x256);
// gate/up 512 x 27648 x 5120 139.5 -> 125.8 (224 rows), 165 -> 150 (128 x 256), 203 x 12288 x 4096 (128x128, four
// stages) 42.5 -> 41.0.  The deeper operand alone, without the order, gains nothing with 256 rows and 4-8 % with 192.
// The 256x256 tile takes all 256 VGPRs and spills up to four (23 with a ragged K; gate/up none, 15 ragged) around a tile's
// prologue and epilogue; the k loop reloads nothing.
// The 128x128 tiles wait for memory: a CU has 64 KiB of loads in flight, in order, whatever the stages hold, so its rate is that over the
// latency (203 x 12288 x 4096: 39.5 us, with the loads alone 38.5, with the arithmetic alone 22.7, with weights from the L2 31).  Stages of
// 128 k ask for whole pairs of lines of a row: 512 x 5120 x 5120 51.4 -> 45.6 us, 900 x 9000 x 8008 197 -> 174 (a ragged row
// piece of 128 bytes lies on two lines, of 256 bytes on three); which K take them is plan_gemm's.
// Eight waves everywhere but in the 64-token configuration: with four (one per SIMD) nothing covers a wave's wait for
// its fragments, and the 256x128 and 128x128 tiles lost 8-10 %.
template <int BN, int BM, int WN, int WM, int GK, int NSW, int NSX, int EPI, bool KTAIL>
__global__ __launch_bounds__(64 * WN * WM) void gemm_streamk(GemmArgs a, int tiles_m, int ktiles, int sk_tiles, int parts, int workers)
{
    constexpr int NWAVES = WN * WM;
    constexpr int THREADS = 64 * NWAVES;
    constexpr int GPIECES = GK / 8;             // 16-byte pieces per tile row
    constexpr int KSTEPS = GK / 32;             // MFMA k-steps per staged tile (even)
    constexpr int ROWS_PER_DMA = 64 / GPIECES;  // tile rows covered by one wave-wide direct load
    constexpr int WBLKS = BN * GPIECES / 64;        // direct loads of the weight tile per k-tile,
    constexpr int WPASS = (WBLKS + NWAVES - 1) / NWAVES;    // ... per wave (at most),
    constexpr bool EVEN = WBLKS % NWAVES == 0;              // ... and whether every wave has as many
    constexpr int XPASS = BM * GPIECES / THREADS;
    constexpr int TN = BN / WN / 16;            // MFMA tiles per wave along n
    constexpr int TM = BM / WM / 16;
    constexpr bool SPREAD_K = BN == 128 && BM == 128 && NSW == 4 && !KTAIL;       // (a ragged last k-tile stays the last)
    constexpr bool TOUCH = BN == 128 && BM == 128 && (GK == 128 || NSW == 4) && !is_swiglu(EPI);
    constexpr bool PAIRS = TN % 2 == 0;          // gate and up rows alternate by fragments of 16 rows, else by 8 rows
    constexpr int JPT = is_swiglu(EPI) ? BN / 2 : BN;   // physical weight rows per tile
    constexpr int WSTAGE = BN * GPIECES, XSTAGE = BM * GPIECES;     // 16-byte units per stage; the weight stages come first
    constexpr int DEEP = NSW > NSX ? NSW : NSX, FLAT = NSW > NSX ? NSX : NSW;
    static_assert(FLAT >= 2 && DEEP <= 4 && (KSTEPS % 2) == 0 && (PAIRS || ROWS_PER_DMA <= 8), "pipeline shape");
    static_assert(WBLKS >= NWAVES && XPASS >= 1 && BM * GPIECES % THREADS == 0, "tile too small for the thread count");
    static_assert(EVEN || (NSW == 2 && !KTAIL), "waves with unequal numbers of weight loads: none of them may be left open by a wait");

    extern __shared__ uintx4 smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid / 64);     // wave index, known uniform to the compiler
    const int wn = wv % WN, wm = wv / WN;
    const int lr = lane & 15, hi = lane >> 4;       // operand row (column) and 8-element k group; token and quad of rows
    const int K = a.K;

    // Workgroups past the workers have no tile: they run ahead through the weights (plan_gemm says where)
    const int G = TOUCH ? workers : (int)gridDim.x;
    if constexpr (TOUCH) {
        if ((int)blockIdx.x >= G) {
            touch_weights<BN>(a, tiles_m, G);
            return;
        }
    }
    const int worker = XcdShare(G, blockIdx.x % 8).first + blockIdx.x / 8;
    // The first sk_tiles tiles are cut along K and dealt as `Deal` says; the others are taken whole,
    // round-robin.  The shared tiles come first: their partial tiles are long written when the kernel ends.
    const Deal deal(sk_tiles, ktiles, G, parts);
    const int u_begin = deal.begin(worker), u_end = deal.end(worker);
    const int first_tile = u_begin / ktiles;
    int t_whole = sk_tiles + worker;

    // A wave-wide load covers ROWS_PER_DMA tile rows = 64 consecutive LDS units; lane L owns unit L of it:
    // row (ROWS_PER_DMA*block + L/P), physical slot L%P, logical piece slot ^ f(row).
    const int slot = lane % GPIECES;

    for (int u = u_begin;;) {
        int t, kb, ke;
        if (u < u_end) {
            t = u / ktiles;
            kb = u - t * ktiles;
            ke = (ktiles - kb < u_end - u) ? ktiles : kb + (u_end - u);
            u += ke - kb;
        } else if (t_whole < a.tiles) {
            t = t_whole;
            kb = 0;
            ke = ktiles;
            t_whole += G;
        } else {
            break;
        }
        const int tile_m = t % tiles_m, tile_n = t / tiles_m;

        // Operand sources: a wave-uniform base pointer per wave instruction (scalar registers, advanced by
        // scalar adds) plus a 32-bit per-lane byte offset that never changes, so that issuing a k-tile's
        // loads costs no vector ALU work.
        const uint16_t* wsrc[WPASS];
        const uint16_t* xsrc[XPASS];
        unsigned woff[WPASS], xoff[XPASS];
#pragma unroll
        for (int i = 0; i < WPASS; ++i) {
            const int blk = EVEN ? wv * WPASS + i : wv + NWAVES * i; // (uniform) block of ROWS_PER_DMA rows
            const int v = blk * ROWS_PER_DMA + lane / GPIECES;
            const int piece = slot ^ swz_f<GPIECES>(v);
            if (is_swiglu(EPI)) {                                    // a wave instruction covers gate rows or up rows only
                const int j0 = tile_n * JPT;                         // first row of the tile: always valid
                int j = j0 + (PAIRS ? (v >> 5) * 16 + (v & 15) : (v >> 4) * 8 + (v & 7));
                j = j < a.N ? j : a.N - 1;
                wsrc[i] = (((blk * ROWS_PER_DMA) >> (PAIRS ? 4 : 3)) & 1 ? a.w1 : a.w0) + (size_t)j0 * K;
                woff[i] = (unsigned)((j - j0) * K + piece * 8) * 2u;
            } else {
                const int n0 = tile_n * BN;
                int n = n0 + v;
                n = n < a.N ? n : a.N - 1;
                wsrc[i] = a.w0 + (size_t)n0 * K;
                woff[i] = (unsigned)((n - n0) * K + piece * 8) * 2u;
            }
        }
#pragma unroll
        for (int i = 0; i < XPASS; ++i) {
            const int v = (wv * XPASS + i) * ROWS_PER_DMA + lane / GPIECES;
            const int piece = slot ^ swz_f<GPIECES>(v);
            const int m0 = tile_m * BM;
            int m = m0 + v;
            m = m < a.M ? m : a.M - 1;       // rows past M are loaded from a valid row and never stored
            xsrc[i] = a.x + (size_t)m0 * K;
            xoff[i] = (unsigned)((m - m0) * K + piece * 8) * 2u;
        }

        // KTAIL: the logical piece (of this lane's unit of load `blk`) if it lies past K in k-tile kt, else 0
        auto past_k = [&](int blk, int kt) {
            const int piece = slot ^ swz_f<GPIECES>(blk * ROWS_PER_DMA + lane / GPIECES);
            return kt * GK + piece * 8 >= K ? piece : 0;
        };
        auto dma_w = [&](int kt, int buf, int i) {
            const bool tail = KTAIL && kt == ktiles - 1;
            const int blk = EVEN ? wv * WPASS + i : wv + NWAVES * i;
            if (EVEN || blk < WBLKS)
                dma16_sbase(wsrc[i] + kt * GK, tail ? woff[i] - 16u * past_k(blk, kt) : woff[i], smem + buf * WSTAGE + blk * 64);
        };
        auto dma_x = [&](int kt, int buf, int i) {
            const bool tail = KTAIL && kt == ktiles - 1;
            dma16_sbase(xsrc[i] + kt * GK, tail ? xoff[i] - 16u * past_k(wv * XPASS + i, kt) : xoff[i],
                        smem + NSW * WSTAGE + buf * XSTAGE + (wv * XPASS + i) * 64);
        };
        // zeros where this wave's loads of k-tile kt (landed, in stages wbuf and xbuf) lay past K
        auto zero_tail = [&](int kt, int wbuf, int xbuf) {
            if (!KTAIL || kt != ktiles - 1) return;
#pragma unroll
            for (int i = 0; i < WPASS; ++i)
                if (past_k(wv * WPASS + i, kt)) smem[wbuf * WSTAGE + (wv * WPASS + i) * 64 + lane] = uintx4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < XPASS; ++i)
                if (past_k(wv * XPASS + i, kt)) smem[NSW * WSTAGE + xbuf * XSTAGE + (wv * XPASS + i) * 64 + lane] = uintx4{0u, 0u, 0u, 0u};
        };

        floatx4 acc[TN][TM];
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

        half8 wa[2][TN], xb[2][TM];
        // The r-th operand fragment of a k-step, weights first: where a lane reads is its place in the k-step's first fragment
        // of the stage (a wave's fragments are 16 rows apart, and the swizzle repeats after 16 rows) and a constant.
        auto read_frag = [&](int r, const uintx4* wl, const uintx4* xl, int fs) {
            if (r < TN) wa[fs][r] = __builtin_bit_cast(half8, wl[r * 16 * GPIECES]);
            else xb[fs][r - TN] = __builtin_bit_cast(half8, xl[(r - TN) * 16 * GPIECES]);
        };
        auto w_lane = [&](int buf, int kk) { return smem + buf * WSTAGE + swz<GPIECES>(wn * (BN / WN) + lr, 4 * kk + hi); };
        auto x_lane = [&](int buf, int kk) { return smem + NSW * WSTAGE + buf * XSTAGE + swz<GPIECES>(wm * (BM / WM) + lr, 4 * kk + hi); };
        // The MFMAs of one k-step in a fixed order: a read of the next k-step's fragments in front of every GAP-th while there are
        // any, the direct loads at equal distances.
        constexpr int NMF = TN * TM, NRD = TN + TM;
        auto step = [&](int fs, auto gap, auto read, auto nloads, auto load) {
            constexpr int GAP = decltype(gap)::value, NL = decltype(nloads)::value;
#pragma unroll
            for (int i = 0; i < NMF; ++i) {
                if (i % GAP == 0 && i / GAP < NRD) read(i / GAP);
#pragma unroll
                for (int d = 0; d < NL; ++d)
                    if (d * NMF / (NL ? NL : 1) == i) load(d);
                const int tn = i / TM, tm = i % TM;
                acc[tn][tm] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wa[fs][tn], xb[fs][tm], acc[tn][tm], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        // ---- prologue: the first k-tiles into the stages, oldest first
        constexpr int LPT = WPASS + XPASS;           // direct loads per k-tile per wave
        constexpr bool W_LATE = NSW >= NSX && NSW >= 3, X_LATE = NSX > NSW;
        const int nk = ke - kb;
        // Two token tiles of the 128x128 kernel with 64-k stages (129..256 tokens): the tile rows start spread over the range and wrap round, so
        // that the workgroups do not all ask for one k of rows that lie a multiple of some KiB apart, that is for few of the memory's channels
        // (203 tokens: 4096 x 4096 23.9 -> 21.4 us, 12288 x 4096 40.7 -> 39.3, 4096 x 11008 37.4 -> 36.3).  With more token tiles
        // (333 x 12288 x 4096 55.5, 55.4; 1024 x 4096 x 4096 39.6, 40.0) and larger ones sharing the activations counts as much.
        int rot = 0;
        if constexpr (SPREAD_K) rot = tiles_m == 2 ? (int)((long)tile_n * nk / (a.tiles / tiles_m)) : 0;
        auto k_of = [&](int i) {
            if constexpr (!SPREAD_K) return kb + i;
            const int k = i + rot;
            return kb + (k < nk ? k : k - nk);
        };
#pragma unroll
        for (int st = 0; st < DEEP; ++st) {
            if (st < NSX - X_LATE && st < nk)
#pragma unroll
                for (int i = 0; i < XPASS; ++i) dma_x(k_of(st), st, i);
            if (st < NSW - W_LATE && st < nk)
#pragma unroll
                for (int i = 0; i < WPASS; ++i) dma_w(k_of(st), st, i);
        }
        // Only the first k-tile has to have landed (all of them where that is not a fixed number of loads: ranges shorter
        // than the stages, waves with unequal numbers of loads); the loop waits for the others one by one.  Waiting for all
        // stages cost most where a range is a few k-tiles long, the more the more stages there are (128x128 tiles, four stages:
        // 108 x 451 x 624 11.1 -> 10.6 us; 345 calls of 129..2048 tokens 1.2 % on average).
        constexpr int FIRST = (NSX - 1 - X_LATE) * XPASS + (NSW - 1 - W_LATE) * WPASS;
        static_assert(FIRST < 64, "wait count out of range");
        if (EVEN && nk >= DEEP) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FIRST) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (KTAIL && nk == 1) zero_tail(kb, 0, 0);
        __syncthreads();

        // Direct loads complete in order.  In front of k-tile it+1 the newest loads that must have landed are those of its operand
        // with the fewer stages; behind them, in flight, are the deeper operand's of the same turn and the later turns' of both.
        constexpr int STEADY = (FLAT - 2) * LPT + (NSW > NSX ? WPASS : NSX > NSW ? XPASS : 0);
        static_assert(STEADY < 64, "wait count out of range");
#pragma unroll
        for (int r = 0; r < NRD; ++r) read_frag(r, w_lane(0, 0), x_lane(0, 0), 0);
        int ws = 0, xs = 0, wprev = NSW - 1, xprev = NSX - 1;     // stages of k-tile it and of the one in front
        // One k-tile.  The loads of the operand with fewer stages go out behind the barrier, into the stage that was read last; those of
        // the deeper one in the next k-tile's first k-step (its last stage is therefore still empty when the loop starts).  LAST: the
        // k-tiles whose successors in the same stages may lie past the range.
        constexpr int EARLY = (W_LATE ? 0 : WPASS) + (X_LATE ? 0 : XPASS), LATE = LPT - EARLY;
        constexpr int SPREAD = NMF / NRD;
        auto ktile = [&](int it, auto last) {
            constexpr bool LAST = decltype(last)::value;
            const int wnext = ws + 1 == NSW ? 0 : ws + 1, xnext = xs + 1 == NSX ? 0 : xs + 1;
            auto late = [&](int d) {
                if (W_LATE && (!LAST || it - 1 + NSW < nk)) dma_w(k_of(it - 1 + NSW), wprev, d);
                if (X_LATE && (!LAST || it - 1 + NSX < nk)) dma_x(k_of(it - 1 + NSX), xprev, d);
            };
            auto none = [](int) {};
            using std::integral_constant;
#pragma unroll
            for (int kk = 0; kk < KSTEPS - 1; ++kk) {
                const uintx4 *wl = w_lane(ws, kk + 1), *xl = x_lane(xs, kk + 1);
                auto read = [&](int r) { read_frag(r, wl, xl, (kk + 1) & 1); };
                if (kk == 0 && KSTEPS == 2) step(0, integral_constant<int, 1>{}, read, integral_constant<int, LATE>{}, late);
                else if (kk == 0) step(0, integral_constant<int, SPREAD>{}, read, integral_constant<int, LATE>{}, late);
                else if (kk < KSTEPS - 2) step(kk & 1, integral_constant<int, SPREAD>{}, read, integral_constant<int, 0>{}, none);
                else step(kk & 1, integral_constant<int, 1>{}, read, integral_constant<int, 0>{}, none);
            }
            // Every read of this k-tile's stages has been issued.  The compiler does not carry these
            // loads across the loop edge, hence the explicit wait.
            if (STEADY > 0 && (!LAST || it + DEEP <= nk)) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STEADY) : "memory");
            else if (DEEP == 4 && FLAT >= 3 && it + 3 <= nk) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPT) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (KTAIL && LAST && it + 1 < nk) zero_tail(kb + it + 1, wnext, xnext);
            __syncthreads();
            auto early = [&](int d) {
                if (!X_LATE && d < XPASS) { if (!LAST || it + NSX < nk) dma_x(k_of(it + NSX), xs, d); }
                else if (!LAST || it + NSW < nk) dma_w(k_of(it + NSW), ws, X_LATE ? d : d - XPASS);
            };
            const bool more = !LAST || it + 1 < nk;              // (behind the last k-tile: read and never used)
            const uintx4 *wl = w_lane(more ? wnext : ws, 0), *xl = x_lane(more ? xnext : xs, 0);
            auto read = [&](int r) { read_frag(r, wl, xl, 0); };
            step((KSTEPS - 1) & 1, integral_constant<int, SPREAD>{}, read, integral_constant<int, EARLY>{}, early);
            wprev = ws;
            xprev = xs;
            ws = wnext;
            xs = xnext;
        };
        int it = 0;
        for (; it + DEEP < nk; ++it) ktile(it, std::false_type{});
        for (; it < nk; ++it) ktile(it, std::true_type{});

        // ---- whole tile: finished below; shared tile: leave the fp32 partial for the fix-up kernel ---
        const bool whole = (kb == 0 && ke == ktiles);
        if (PAIRS && !whole) {                       // (an odd number of fragments: never cut)
            const int pslot = (t == first_tile) ? 0 : 1;
            floatx4* ps = reinterpret_cast<floatx4*>(a.partials + ((size_t)worker * 2 + pslot) * (BN * BM));
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) ps[(tn * TM + tm) * THREADS + tid] = acc[tn][tm];
        }

        // ---- epilogue ------------------------------------------------------------------------
        if (whole) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                if constexpr (PAIRS) {
#pragma unroll
                    for (int tp = 0; tp < TN / 2; ++tp)
                        store_pair<BN, BM, WN, WM, EPI>(a, tile_n, tile_m, wn, wm, tp, tm, lr, hi, acc[2 * tp][tm], acc[2 * tp + 1][tm]);
                } else {
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
                        store_one<BN, BM, WN, WM, EPI>(a, tile_n, tile_m, wn, wm, tn, tm, lr, hi, acc[tn][tm]);
                }
            }
        }
        // the next run rewrites the LDS stages only after this barrier
        __syncthreads();
    }
}

// ALL = also build the variant for a ragged K (KTAIL), with RAGGED_NSW weight stages.
template <int BN, int BM, int WN, int WM, int GK, int NSW, int NSX, bool ALL, int RAGGED_NSW = NSW>
hipError_t launch_cfg(GemmArgs a, int epilogue, const GemmPlan& p, hipStream_t stream)
{
    constexpr bool CUT = BN / WN / 16 % 2 == 0;
    const GemmTile tile = gemm_tile(p.config);
    if (tile.BN != BN || tile.BM != BM || tile.GK != GK || tile.cut != CUT || tile.ragged != ALL) return hipErrorInvalidValue;
    a.tiles = p.tiles;
    const int tiles_m = p.tiles_m, ktiles = p.ktiles, grid = p.grid, sk_tiles = p.sk_tiles, parts = p.parts;
    dim3 g((unsigned)(grid + p.helpers)), b(64 * WN * WM);
#define THI_LAUNCH_K(E, KT)                                                                                  \
    do {                                                                                                     \
        constexpr int W_STAGES = KT ? RAGGED_NSW : NSW;                                                      \
        constexpr size_t lds = ((size_t)W_STAGES * BN + (size_t)NSX * BM) * (GK / 8) * sizeof(uintx4);       \
        auto kern = gemm_streamk<BN, BM, WN, WM, GK, W_STAGES, NSX, E, KT>;                                  \
        static std::once_flag attr_once;      /* one opt-in per kernel variant, safe from several threads */  \
        std::call_once(attr_once, [&] {                                                                      \
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                                   \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                 \
        });                                                                                                  \
        hipLaunchKernelGGL(kern, g, b, lds, stream, a, tiles_m, ktiles, sk_tiles, parts, grid);              \
        if constexpr (CUT) {                                                                                 \
            if (sk_tiles > 0)                                                                                \
                hipLaunchKernelGGL((gemm_fixup<BN, BM, WN, WM, E>),                                                   \
                                   dim3(sk_tiles * (BN / WN / 32) * (BM / WM / 16) * (WN * WM / FIXUP_WAVES)),        \
                                   dim3(64 * FIXUP_WAVES), 0, stream, a, tiles_m, ktiles, sk_tiles, grid, parts);            \
        }                                                                                                    \
    } while (0)
#define THI_LAUNCH(E)                                                                                        \
    do {                                                                                                     \
        if constexpr (ALL) {                                                                                 \
            if (a.K % GK) THI_LAUNCH_K(E, true);                                                             \
            else THI_LAUNCH_K(E, false);                                                                     \
        } else {                                                                                             \
            THI_LAUNCH_K(E, false);                                                                          \
        }                                                                                                    \
    } while (0)
    switch (epilogue) {
    case EPI_PLAIN: THI_LAUNCH(EPI_PLAIN); break;
    case EPI_ROPE: THI_LAUNCH(EPI_ROPE); break;
    case EPI_RMSNORM:            // RMSNorm runs as a pass of its own in front of the GEMM: the dispatcher
    case EPI_RMSNORM_ROPE:       // calls this with the plain / rotary / SwiGLU kinds only
    case EPI_RMSNORM_SWIGLU:
        return hipErrorInvalidValue;
    default: THI_LAUNCH(EPI_SWIGLU); break;
    }
#undef THI_LAUNCH
#undef THI_LAUNCH_K
    return hipGetLastError();
}

}  // namespace

namespace {

// One workgroup per token row: sum of squares in fp32, then the normalised row in fp16 (one rounding of
// x * r * gamma).  Memory-bound over M*K elements; with few rows it is one chain of latencies, so the row and
// gamma are requested together up front and the row stays in registers (NP 16-byte pieces a thread; NP = 0: any K, the
// row is read twice). (M x K = 2048 x 8192
// with the QKV GEMM behind it 310 -> 306 us, 72 x 4096 37.9 -> 36.9.)
template <int NP>
__global__ __launch_bounds__(256) void rmsnorm_rows(const uint16_t* x, const uint16_t* gamma, float eps, uint16_t* xn, int K,
                                                    RopeArgs rope)
{
    __shared__ float s_part[4];
    const uint16_t* row = x + (size_t)blockIdx.x * K;
    uint16_t* dst = xn + (size_t)blockIdx.x * K;
    half8 v[NP ? NP : 1], g[NP ? NP : 1];
    float ss = 0.f;
    if constexpr (NP > 0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int k = (i * 256 + (int)threadIdx.x) * 8, kc = k < K ? k : 0;
            v[i] = __builtin_bit_cast(half8, *reinterpret_cast<const uintx4*>(row + kc));
            g[i] = __builtin_bit_cast(half8, *reinterpret_cast<const uintx4*>(gamma + kc));
        }
    }
    // the rotary epilogue's table for this token: fp32 angle, full-range sincosf (positions reach
    // thousands of radians); done here so that the GEMM's epilogue needs neither
    if (rope.cs && (int)threadIdx.x < (rope.head_dim >> 1)) {
        float sn, cs;
        sincosf((float)rope.pos[blockIdx.x] * rope.theta[threadIdx.x], &sn, &cs);
        float* e = const_cast<float*>(rope.cs) + ((size_t)blockIdx.x * (rope.head_dim >> 1) + threadIdx.x) * 2;
        e[0] = cs;
        e[1] = sn;
    }
    if constexpr (NP > 0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if ((i * 256 + (int)threadIdx.x) * 8 < K) {
#pragma unroll
                for (int e = 0; e < 8; ++e) { const float f = (float)v[i][e]; ss = __builtin_fmaf(f, f, ss); }
            }
        }
    } else {
        for (int k = threadIdx.x * 8; k < K; k += 256 * 8) {
            const half8 xv = __builtin_bit_cast(half8, *reinterpret_cast<const uintx4*>(row + k));
#pragma unroll
            for (int e = 0; e < 8; ++e) { const float f = (float)xv[e]; ss = __builtin_fmaf(f, f, ss); }
        }
    }
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) ss += __shfl_xor(ss, sh);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float r = 1.0f / __builtin_sqrtf(((s_part[0] + s_part[1]) + (s_part[2] + s_part[3])) / (float)K + eps);
    auto put = [&](int k, const half8& xv, const half8& gv) {
        half8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (_Float16)((float)xv[e] * r * (float)gv[e]);
        *reinterpret_cast<uintx4*>(dst + k) = __builtin_bit_cast(uintx4, o);
    };
    if constexpr (NP > 0) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int k = (i * 256 + (int)threadIdx.x) * 8;
            if (k < K) put(k, v[i], g[i]);
        }
    } else {
        for (int k = threadIdx.x * 8; k < K; k += 256 * 8)
            put(k, __builtin_bit_cast(half8, *reinterpret_cast<const uintx4*>(row + k)),
                __builtin_bit_cast(half8, *reinterpret_cast<const uintx4*>(gamma + k)));
    }
}

}  // namespace

hipError_t launch_rmsnorm_rows(const uint16_t* x, const uint16_t* gamma, float eps, uint16_t* xn, int M, int K,
                               const RopeArgs& rope, hipStream_t stream)
{
    if (rope.cs && rope.head_dim > 2 * 256) return hipErrorInvalidValue;     // one thread per pair of the head
    const int np = (K + 2047) / 2048;
    const dim3 g((unsigned)M), b(256);
    if (np <= 1) hipLaunchKernelGGL((rmsnorm_rows<1>), g, b, 0, stream, x, gamma, eps, xn, K, rope);
    else if (np <= 2) hipLaunchKernelGGL((rmsnorm_rows<2>), g, b, 0, stream, x, gamma, eps, xn, K, rope);
    else if (np <= 4) hipLaunchKernelGGL((rmsnorm_rows<4>), g, b, 0, stream, x, gamma, eps, xn, K, rope);
    else if (np <= 8) hipLaunchKernelGGL((rmsnorm_rows<8>), g, b, 0, stream, x, gamma, eps, xn, K, rope);
    else hipLaunchKernelGGL((rmsnorm_rows<0>), g, b, 0, stream, x, gamma, eps, xn, K, rope);
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs& a, int epilogue, int num_cus, hipStream_t stream)
{
    if (is_rms(epilogue)) return hipErrorInvalidValue;
    const GemmPlan p = plan_product(a.M, a.N, a.K, epilogue, num_cus, a.token_tiles);
    switch (p.config) {
    case GEMM_MID: return launch_mid(a, epilogue, p.mid, stream);
    case GEMM_FEW64: return launch_cfg<128, 64, 4, 1, 128, 3, 3, false>(a, epilogue, p, stream);
    case GEMM_FEW256: return launch_cfg<256, 128, 4, 2, 64, 3, 3, false>(a, epilogue, p, stream);
    case GEMM_BIG: return launch_cfg<256, 256, 4, 2, 64, 3, 2, true>(a, epilogue, p, stream);
    case GEMM_R224: return launch_cfg<224, 256, 2, 4, 64, 2, 3, false>(a, epilogue, p, stream);
    case GEMM_R192: return launch_cfg<192, 256, 2, 4, 64, 3, 2, false>(a, epilogue, p, stream);
    case GEMM_R160: return launch_cfg<160, 256, 2, 4, 64, 2, 3, false>(a, epilogue, p, stream);
    case GEMM_ONE: case GEMM_TALL: return launch_cfg<128, 256, 2, 4, 64, 3, 3, false>(a, epilogue, p, stream);
    case GEMM_FEW128: return launch_cfg<128, 128, 2, 4, 64, 4, 4, true>(a, epilogue, p, stream);
    case GEMM_DEEP: return launch_cfg<128, 128, 2, 4, 128, 3, 2, true>(a, epilogue, p, stream);
    // (a ragged K with two weight stages: a third lost 5 % on average over 26 products of 448 <= K <= 11000 -- 1198 x 7769 x 6104 169 -> 187 us,
    // gate/up 1206 x 4024 x 10928 280 -> 312, 772 x 6280 x 4024 75 -> 83, 500 x 14464 x 3680 the other way 84.6 -> 79.6; an even K is the same with both)
    case GEMM_SMALL: return launch_cfg<128, 128, 2, 4, 64, 3, 2, true, 2>(a, epilogue, p, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace thi
