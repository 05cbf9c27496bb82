// batch_inst.hip -- instantiates the batched launch's kernels for one blur
// size HX_KS and one part (the build compiles this file once per pair, in
// parallel): 0 the short sweeps and the thresholds, 1 SPECULATE's pass 1,
// 2 STORE's pass 1, 3 RECOMPUTE.
#include "batch_impl.h"

#if !defined(HX_KS) || !defined(HX_PART)
#error "HX_KS and HX_PART must be defined"
#endif

#define HX_CAT2(a, b, c, d) a##b##c##d
#define HX_CAT(a, b, c, d) HX_CAT2(a, b, c, d)

namespace hx {

// The kernel of (pass structure, phase); alt: SPECULATE's pass 1 on tiles of
// up to kShortTile rows and its pass 2 that claims registers, kPassShort's
// one-column tiles.  nullptr: not in this part.
const void* HX_CAT(batch_kernel_k, HX_KS, _p, HX_PART)(int pass, int phase, bool alt) {
    (void)pass, (void)phase, (void)alt;
#if HX_PART == 0
    if (pass == kPassShort)
        return phase == 1 ? (alt ? (const void*)k_batch_short_max<HX_KS, 1>
                                 : (const void*)k_batch_short_max<HX_KS, 2>)
                          : (alt ? (const void*)k_batch_short_mask<HX_KS, 1>
                                 : (const void*)k_batch_short_mask<HX_KS, 2>);
    if (pass == HX_PASS_SPECULATE) {
        if (phase == 0) return (const void*)k_batch_p0<HX_KS>;
        if (phase == 1 && alt) return (const void*)k_batch_p1t<HX_KS>;
        if (phase == 2)
            return alt ? (const void*)k_batch_p2s<HX_KS, true>
                       : (const void*)k_batch_p2s<HX_KS, false>;
    }
    if (pass == HX_PASS_STORE && phase == 2) return (const void*)k_batch_p2<HX_KS, HX_PASS_STORE>;
#elif HX_PART == 1
    if (pass == HX_PASS_SPECULATE && phase == 1 && !alt)
        return (const void*)k_batch_p1s<HX_KS>;
#elif HX_PART == 2
    if (pass == HX_PASS_STORE && phase == 1)
        return (const void*)k_batch_p1<HX_KS, HX_PASS_STORE>;
#else
    if (pass == HX_PASS_RECOMPUTE)
        return phase == 1   ? (const void*)k_batch_p1<HX_KS, HX_PASS_RECOMPUTE>
               : phase == 2 ? (const void*)k_batch_p2<HX_KS, HX_PASS_RECOMPUTE>
                            : nullptr;
#endif
    return nullptr;
}

}  // namespace hx
