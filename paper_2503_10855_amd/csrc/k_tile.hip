// k_tile.hip -- per-image kernels of the short sweep (tile_impl.h): the
// STORE pass 1 and the stage hook of images too small to fill the chip with
// long tiles, and the blur of the sizes the long sweep does not take.
#include "tile_impl.h"

namespace hx {
namespace {

// One wave per tile; the waves of a workgroup fold their maxima in LDS, so
// one atomic per workgroup reaches the image's slot.
template <int KS, int C, int MODE>
__global__ __launch_bounds__(256) void k_tile(ImgArgs a, Taps tp, int ty, int nstrips,
                                              int ntiles, StageOut so) {
    using S = TileShape<KS, C, MODE>;
    extern __shared__ __align__(16) float smem[];
    const int nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = xcd_remap(blockIdx.x, gridDim.x) * nw + wave;
    float gmax = 0.0f;
    if (t < ntiles) {
        const int by = t / nstrips, bx = t - by * nstrips;
        lds_float* lds = (lds_float*)smem + wave * S::lds_floats(ty);
        const int x0 = bx * S::OW, y0 = by * ty;
        tile_load<C>(a, x0 - S::HL, y0 - S::HY, min(ty, a.H - y0) + 2 * S::HY, lds);
        tile_loads_done();
        tile_sweep<KS, C, MODE>(a, tp, x0, y0, ty, 0.0f, gmax, lds, nullptr, &so);
    }
    if constexpr (S::DO_MAX) {
        gmax = wave_max(gmax);
        __syncthreads();   // every wave is done with its rows
        if (lane_id() == 0) smem[wave] = gmax;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < nw; ++w) gmax = __builtin_fmaxf(gmax, smem[w]);
            atomic_max_g2(slot_word(a, blockIdx.x), gmax);
        }
    }
}

template <int KS, int C, int MODE>
hipError_t launch_t(int ty, const ImgArgs& a, const Taps& t, const StageOut& so, hipStream_t s) {
    using S = TileShape<KS, C, MODE>;
    const int nstrips = (a.W + S::OW - 1) / S::OW;
    const int ntiles = nstrips * ((a.H + ty - 1) / ty);
    const int bytes = S::lds_floats(ty) * (int)sizeof(float);
    int nw = 4;
    while (nw > 1 && nw * bytes > 65536) nw /= 2;
    hipLaunchKernelGGL((k_tile<KS, C, MODE>), dim3((ntiles + nw - 1) / nw), dim3(64 * nw),
                       nw * bytes, s, a, t, ty, nstrips, ntiles, so);
    return hipGetLastError();
}

template <int KS, int MODE>
hipError_t launch_c(int c, int ty, const ImgArgs& a, const Taps& t, const StageOut& so,
                    hipStream_t s) {
    if (c == 1) return launch_t<KS, 1, MODE>(ty, a, t, so, s);
    if (c == 2) return launch_t<KS, 2, MODE>(ty, a, t, so, s);
    if (c == 4) return launch_t<KS, 4, MODE>(ty, a, t, so, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_tile(int mode, int ks, int c, int ty, const ImgArgs& a, const Taps& t,
                       const StageOut& so, hipStream_t s) {
    if (ty < kTurn || ty % kTurn != 0 || ty > 32) return hipErrorInvalidValue;
#define HX_T(K)                                                              \
    if (ks == K) {                                                           \
        if (mode == SM_STORE) return launch_c<K, SM_STORE>(c, ty, a, t, so, s); \
        if (mode == TM_STAGES) return launch_c<K, TM_STAGES>(c, ty, a, t, so, s); \
    }
#define HX_B(K) \
    if (ks == K && mode == TM_BLUR) return launch_c<K, TM_BLUR>(c, ty, a, t, so, s);
    HX_T(1) HX_T(3) HX_T(5) HX_T(7)
    HX_B(9) HX_B(11) HX_B(13) HX_B(15)
#undef HX_T
#undef HX_B
    return hipErrorInvalidValue;
}

}  // namespace hx
