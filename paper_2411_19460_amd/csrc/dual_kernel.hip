// Launchers of the dual-form passes (see dual_body.h) as kernels of their own.
#include "dual_body.h"

namespace ssdk {
namespace {

using namespace dualk;

template <int Q, int EPI>
__global__ __launch_bounds__(DualCfg<Q>::NTHR) void mk_dual(SegParams sp) {
    __shared__ __attribute__((aligned(16))) DualLds<Q> L;
    dual_body<Q, EPI>(sp, L, blockIdx.x, gridDim.x);
}

template <int Q, int EPI>
hipError_t launch_dual_q(const SegParams& sp0, int kid, hipStream_t st) {
    SegParams sp = sp0;
    // with other launches in flight: as few head slices as still give every compute unit a workgroup, the persistent
    // operands are then shared by as many heads as possible.  Alone: the fewest rounds over the machine (10007 tokens of 80
    // heads, eight slices in two rounds -> five in one: 96.6 -> 76.3 us; chunks of 64, see pick_rounds)
    const int64_t base = (int64_t)sp.Bt * sp.nc * sp.G;
    sp.dual_split = sp.wg_target < 256 ? pick_split(sp.hpg, base, sp.wg_target) : pick_rounds(sp.hpg, base, Q == 256 ? 1 : 2, 70);
    SSDK_LAUNCH(kid, st, (mk_dual<Q, EPI>), dim3(sp.Bt * sp.nc * sp.G * sp.dual_split), dim3(DualCfg<Q>::NTHR), sp);
    return hipSuccess;
}

}  // namespace

hipError_t mfma_launch_dual(const SegParams& sp, int epi, hipStream_t st) {
    if (epi == 0) switch (sp.Q) {
        case 64: return launch_dual_q<64, 0>(sp, K_MFMA_CHUNK_OUT, st);
        case 128: return launch_dual_q<128, 0>(sp, K_MFMA_CHUNK_OUT, st);
        case 256: return launch_dual_q<256, 0>(sp, K_MFMA_CHUNK_OUT, st);
    }
    // longer chunks: part of a launch with the other passes over the heads (mk_bwd_trio)
    if (epi == 2 && sp.Q == 64) return launch_dual_q<64, 2>(sp, K_MFMA_BWD_MAIN, st);
    return hipErrorInvalidValue;
}

}  // namespace ssdk
