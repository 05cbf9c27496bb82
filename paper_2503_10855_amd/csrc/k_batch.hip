// k_batch.hip -- host side of the batched launch: geometry and launchers
// (the kernels: batch_impl.h, instantiated by batch_inst.hip).
#include <hip/hip_ext.h>

#include "batch_impl.h"

namespace hx {

int batch_sweep_c() { return kBC; }
int batch_sweep_ty() { return kBTY; }
int batch_p2_rows(int64_t W) { return p2_rows(W); }

size_t batch_table_bytes(int n, int64_t n1, int64_t n2, int64_t n0) {
    return sizeof(BatchHeader) + (size_t)n * sizeof(ImgArgs) +
           (size_t)(n1 + n2 + n0) * sizeof(BatchItem);
}

int64_t batch_sample_items(int ks, int64_t H, int64_t W) {
    const SweepGeom g{ks, kBC, kSampleRows};
    const int st = sample_stride(H);
    return g.strips(W) * ((H + st - 1) / st);
}

static __global__ void k_batch_reset(const uint8_t* __restrict__ table) {
    const BatchHeader& h = *reinterpret_cast<const BatchHeader*>(table);
    const ImgArgs* imgs = reinterpret_cast<const ImgArgs*>(table + sizeof(BatchHeader));
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < h.n_images;
         i += gridDim.x * blockDim.x)
        for (int w = 0; w < imgs[i].ways; ++w) imgs[i].slot[(int64_t)w * h.slot_step] = 0;
}

hipError_t launch_batch_reset(const void* d_table, int max_images, hipStream_t s) {
    int grid = (max_images + 255) / 256;
    if (grid > 1024) grid = 1024;
    hipLaunchKernelGGL(k_batch_reset, dim3(grid), dim3(256), 0, s, (const uint8_t*)d_table);
    return hipGetLastError();
}

#define HX_DECL(K, P) const void* batch_kernel_k##K##_p##P(int pass, int phase, bool alt);
#define HX_DECL_K(K) HX_DECL(K, 0) HX_DECL(K, 1) HX_DECL(K, 2) HX_DECL(K, 3)
HX_DECL_K(3)
HX_DECL_K(5)
HX_DECL_K(7)
#undef HX_DECL_K
#undef HX_DECL

static const void* batch_kernel_ptr(int ks, int pass, int phase, bool alt) {
    const void* k = nullptr;
#define HX_P(K, P) \
    if (ks == K && !k) k = batch_kernel_k##K##_p##P(pass, phase, alt);
#define HX_PK(K) HX_P(K, 0) HX_P(K, 1) HX_P(K, 2) HX_P(K, 3)
    HX_PK(3) HX_PK(5) HX_PK(7)
#undef HX_PK
#undef HX_P
    return k;
}

static hipError_t launch(const void* k, int64_t grid, void** args, int lds, hipStream_t s,
                         hipEvent_t done) {
    if (!done) return hipLaunchKernel(k, dim3((unsigned)grid), dim3(64), args, lds, s);
    return hipExtLaunchKernel(k, dim3((unsigned)grid), dim3(64), args, lds, s, nullptr, done,
                              0);
}

hipError_t launch_batch_short(int ks, int c, int phase, const ShortArgs& s, const Taps& t,
                              hipStream_t stream, hipEvent_t done) {
    const void* k = batch_kernel_ptr(ks, kPassShort, phase, c == 1);
    if (!k || s.n < 1 || (c != 1 && c != 2) || phase < 1 || phase > 2)
        return hipErrorInvalidValue;
    ShortArgs sc = s;
    Taps tc = t;
    void* args[] = {(void*)&sc, (void*)&tc};
    return launch(k, s.n, args, 0, stream, done);
}

hipError_t launch_batch_phase(int ks, int pass_mode, int phase, int ty, int64_t items,
                              const void* d_table, const Taps& t, hipStream_t s,
                              hipEvent_t done, bool claim) {
    const bool spec = pass_mode == HX_PASS_SPECULATE;
    const bool short_tile = spec && phase == 1 && ty <= kShortTile;
    const void* k = batch_kernel_ptr(ks, pass_mode, phase, short_tile || (spec && phase == 2 && claim));
    if (!k || items < 0) return hipErrorInvalidValue;
    const int64_t grid = items < 1 ? 1 : items;
    int lds = 0;
    if (short_tile) lds = (ty + 2 * (ks / 2 + 2)) * 64 * kBC * (int)sizeof(float);
    const uint8_t* tab = (const uint8_t*)d_table;
    Taps tc = t;
    void* args[] = {(void*)&tab, (void*)&tc};
    return launch(k, grid, args, lds, s, done);
}

}  // namespace hx
