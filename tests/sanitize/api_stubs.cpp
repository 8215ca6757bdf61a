// Host-only stand-ins for the kernel launchers of libthi (test infrastructure): they launch nothing,
// check the few preconditions the real launchers check, and report success -- so that csrc/api.hip's
// validation, workspace carving and dispatch arithmetic (with the library's own csrc/plan.hip) can run
// under AddressSanitizer / UndefinedBehaviorSanitizer on a machine without a GPU.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

namespace thi {

static int g_launches = 0;
int stub_launch_count() { return g_launches; }

hipError_t launch_skinny(const SkinnyArgs& a, int, int, hipStream_t)
{
    ++g_launches;
    return (a.M >= 1 && a.M <= 16 * SK_MAX_MT && a.handover && a.counters) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_rowslab(const SkinnyArgs& a, int epilogue, int num_cus, hipStream_t)
{
    ++g_launches;
    return ((a.K >= 1024 || rowslab_small_ok(a.N, a.K, epilogue, num_cus)) && a.K <= ROWSLAB_MAX_K && a.tiles >= 1 && a.M <= 32) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_rowblock(const SkinnyArgs& a, int epilogue, int num_cus, hipStream_t, int ksplit)
{
    ++g_launches;
    if (a.K < 1024 || a.K > ROWSLAB_MAX_K || a.N < 1 || a.M > 32) return hipErrorInvalidValue;
    if (ksplit > 1 && !rowblock_split_ok(a.N, a.K, epilogue, num_cus, ksplit)) return hipErrorInvalidValue;
    const RowBlockPlan p = plan_rowblock(a.N, epilogue, num_cus, ksplit);
    return (p.T >= 2 && p.T <= 6 && p.grid >= 1) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_mlp_fused(const SkinnyArgs& up, const SkinnyArgs& down, int epilogue_up, int num_cus, hipStream_t, int ksplit_down)
{
    ++g_launches;
    return (mlp_fused_ok(up.M, up.K, up.N, epilogue_up, num_cus, ksplit_down) && down.x == up.out) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_gemm(const GemmArgs& a, int epilogue, int num_cus, hipStream_t)
{
    ++g_launches;
    if (is_rms(epilogue) || !a.partials || !a.counters) return hipErrorInvalidValue;
    const GemmPlan p = plan_gemm(a.M, a.N, a.K, epilogue, num_cus);
    const size_t region = gemm_partial_bytes();
    if (p.grid < 1 || p.tiles < 1) return hipErrorInvalidValue;
    const bool decode = a.M <= MID_DECODE_M;
    if (a.gamma && (!decode || p.config != GEMM_MID)) return hipErrorInvalidValue;
    if (p.config == GEMM_MID) {      // partial tiles: at decode sizes `partials` may be no more than the hand-over slots
        const int BM = decode ? 32 : a.M <= 64 ? 64 : a.M <= 96 ? 96 : 128;
        const bool fits = p.mid.S == 1 || (size_t)p.grid * mid_slot_floats(p.mid.BN, BM, decode) * sizeof(float) <= (decode ? skinny_handover_bytes() : region);
        const bool built = epilogue != EPI_ROPE || a.gamma || !decode;
        return a.M <= 128 && p.grid == p.mid.tiles * p.mid.S && p.grid <= num_cus && p.mid.tiles <= 1024 && fits && built ? hipSuccess : hipErrorInvalidValue;
    }
    const GemmTile t = gemm_tile(p.config);
    const bool covers = (long)p.tiles_m * t.BM >= a.M && (long)p.tiles / p.tiles_m * t.BN >= (is_swiglu(epilogue) ? 2L : 1L) * a.N && p.ktiles * (long)t.GK >= a.K;
    const bool cut = p.sk_tiles == 0 || (t.cut && (size_t)p.grid * 2 * t.BN * t.BM * 4 <= region &&
                                         (p.parts == 0 || ((long)p.sk_tiles * p.parts <= p.grid && p.parts <= p.ktiles)));
    // workgroups that touch the weights ahead: as many for each XCD, one per compute unit with the others, and only in the kernels that tell them apart
    const bool helped = p.helpers == 0 || (p.helpers > 0 && p.helpers % 8 == 0 && p.grid + p.helpers <= num_cus && p.sk_tiles == 0 && p.grid == p.tiles &&
                                           !is_swiglu(epilogue) && (p.config == GEMM_DEEP || p.config == GEMM_FEW128));
    return covers && cut && helped && (t.ragged || a.K % t.GK == 0) && p.sk_tiles <= p.tiles ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_rmsnorm_rows(const uint16_t*, const uint16_t*, float, uint16_t* xn, int, int, const RopeArgs&, hipStream_t)
{
    ++g_launches;
    return xn ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_attention(const AttnArgs& a, hipStream_t)
{
    ++g_launches;
    return (a.nsplit >= 1 && a.nsplit <= AT_MAX_SPLIT && a.whole >= AT_MIN_CHUNK && a.part) ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_fill_words(void*, size_t, uint32_t, hipStream_t)
{
    ++g_launches;
    return hipSuccess;
}

}  // namespace thi
