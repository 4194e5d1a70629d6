// fb_split.hip -- Hermite steps of one bucket with two or four lanes a
// body (fb_split.h).
#include "fb_split.h"

namespace fb {
namespace {

template <int N, int G, bool ADV>
__global__ __launch_bounds__(64) void k_bpl_split(Bucket B, StepParams P)
{
    extern __shared__ char fb_dyn_lds[];
    constexpr int S = split_systems(N, G);
    const int first = blockIdx.x * S;
    int slot;
    split_run<N, G, ADV>(*reinterpret_cast<BplLds *>(fb_dyn_lds), B, first, min(S, B.count - first),
                    nullptr, P, slot);
}

template <int N, int G>
__global__ __launch_bounds__(64) void k_solo_split(SoloIO io, StepParams P)
{
    extern __shared__ char fb_dyn_lds[];
    constexpr int S = split_systems(N, G);
    const int first = blockIdx.x * S;
    int slot;
    split_run<N, G, false, true>(*reinterpret_cast<BplLds *>(fb_dyn_lds), Bucket(), first,
                                 min(S, io.n_sys - first), nullptr, P, slot, io);
}

}  // namespace

hipError_t launch_solo_split(const SoloIO &io, int n, int G, const StepParams &P, hipStream_t s)
{
    if (io.n_sys <= 0)
        return hipSuccess;
    if (P.adaptive || P.stop_rules || (G != 2 && G != 4) || n < kMinSplit)
        return hipErrorInvalidValue;
    const int S = split_systems(n, G);
    const dim3 grid((unsigned)((io.n_sys + S - 1) / S));
#define FB_L(NN)                                                                                       \
    case NN:                                                                                           \
        if (G == 4) hipLaunchKernelGGL((k_solo_split<NN, 4>), grid, dim3(64), sizeof(BplLds), s, io, P); \
        else hipLaunchKernelGGL((k_solo_split<NN, 2>), grid, dim3(64), sizeof(BplLds), s, io, P);      \
        break
    switch (n) {
        FB_L(5); FB_L(6); FB_L(7); FB_L(8); FB_L(9); FB_L(10);
        FB_L(11); FB_L(12); FB_L(13); FB_L(14); FB_L(15); FB_L(16);
    default: return hipErrorInvalidValue;
    }
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_split(const Bucket &B, int G, const StepParams &P, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if ((G != 2 && G != 4) || B.n < kMinSplit)
        return hipErrorInvalidValue;
    const int S = split_systems(B.n, G);
    const dim3 grid((unsigned)((B.count + S - 1) / S));
    const bool adv = P.adaptive || P.stop_rules;
#define FB_K(NN, GG, A) hipLaunchKernelGGL((k_bpl_split<NN, GG, A>), grid, dim3(64), sizeof(BplLds), s, B, P)
#define FB_L(NN)                                                         \
    case NN:                                                             \
        if (G == 4) { if (adv) FB_K(NN, 4, true); else FB_K(NN, 4, false); } \
        else { if (adv) FB_K(NN, 2, true); else FB_K(NN, 2, false); }    \
        break
    switch (B.n) {
        FB_L(5); FB_L(6); FB_L(7); FB_L(8); FB_L(9); FB_L(10);
        FB_L(11); FB_L(12); FB_L(13); FB_L(14); FB_L(15); FB_L(16);
    default: return hipErrorInvalidValue;
    }
#undef FB_L
#undef FB_K
    return hipGetLastError();
}

}  // namespace fb
