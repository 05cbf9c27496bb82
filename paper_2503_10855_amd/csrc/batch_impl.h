// batch_impl.h -- kernels of the batched launch: a whole batch of images of
// any sizes as an outer fork over images whose inner fork factors differ per
// image, flattened into lists of work items.
//
//   reset   zeroes each image's max slot;
//   pass 1  one item = one sweep tile (one wave) of one image: STORE writes
//           the pass-1 code of its pixels, RECOMPUTE computes blur + Sobel
//           only; both fold the tile's G^2 maximum into the image's slot;
//   pass 2  one item = a run of rows (STORE: code -> mask) or one sweep tile
//           (RECOMPUTE: every stage -> mask) of one image.
// SPECULATE adds pass 0 (one item = one 8-row sampled band tile: blur +
// Sobel -> a lower bound of the max), runs every stage in pass 1 (mask
// against the bound's threshold, plus the list of pixels it set), and
// re-decides only the listed pixels in pass 2 (one wave per pass-1 tile).
// A tile whose list did not hold its pixels is queued by pass 1 and redone
// by pass 2 in 8-row pieces.
// Pass 2 starts after pass 1 has finished (a kernel boundary), so every max
// is final when it is read; no workgroup ever waits for another one.  Each
// wave takes the item of its index (the host sizes each grid to its pass's
// item count).  The item lists live in the descriptor table, from which the
// kernels read every size; a repeated batch reuses it.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/hx.h"
#include "sweep_impl.h"
#include "thresh_impl.h"
#include "tile_impl.h"

namespace hx {

#ifndef HX_BATCH_C
#define HX_BATCH_C 4
#endif
#ifndef HX_BATCH_TY
#define HX_BATCH_TY 64
#endif
#ifndef HX_SWEEP_WAVES
#define HX_SWEEP_WAVES 3
#endif
#ifndef HX_SWEEP_WAVES_SMALL_K
#define HX_SWEEP_WAVES_SMALL_K HX_SWEEP_WAVES
#endif
#ifndef HX_BATCH_WG_WAVES
#define HX_BATCH_WG_WAVES 1
#endif
constexpr int kBC = HX_BATCH_C;    // columns per lane of the batch sweep
constexpr int kBTY = HX_BATCH_TY;  // default rows per sweep tile
// Waves per workgroup of the pass kernels.  One: a wave slot freed by a
// finished tile takes the next item at once, where a 4-wave workgroup
// waits for room for all four; with calls in flight on several streams
// that lets one call's last partial round of tiles overlap the next call.
constexpr int kWG = HX_BATCH_WG_WAVES;
// Waves per SIMD the sweep kernels are compiled for (their register cap):
// the 7-tap blur's longer row ring needs more registers than k <= 5.
constexpr int sweep_waves(int ks) { return ks <= 5 ? HX_SWEEP_WAVES_SMALL_K : HX_SWEEP_WAVES; }


__host__ __device__ inline int p2_rows(int64_t W) {
    const int64_t r = 4096 / (W > 0 ? W : 1);
    return r < 1 ? 1 : (r > (1 << 20) ? (1 << 20) : (int)r);
}

// The bound's threshold is scaled down by this factor so that it stays at
// or below the true max's threshold even if the square root were not
// monotone to the last ulp; it only lists a few more pixels.
constexpr float kSpecSafety = 0.99999f;

struct TableView {
    BatchHeader hdr;
    const ImgArgs* imgs;
    const BatchItem* items1;
    const BatchItem* items2;
    const BatchItem* items0;
    // Item k of a list; a batch of one image has no lists.
    __device__ __forceinline__ BatchItem item(const BatchItem* items, int64_t k) const {
        if (hdr.n_images == 1) return BatchItem{0, (int32_t)k};
        return items[k];
    }
};

__device__ __forceinline__ TableView view(const uint8_t* __restrict__ table) {
    TableView v;
    v.hdr = *reinterpret_cast<const BatchHeader*>(table);
    v.imgs = reinterpret_cast<const ImgArgs*>(table + sizeof(BatchHeader));
    v.items1 = reinterpret_cast<const BatchItem*>(v.imgs + v.hdr.n_images);
    v.items2 = v.items1 + v.hdr.n_items1;
    v.items0 = v.items2 + v.hdr.n_items2;
    return v;
}

// Index of this wave among all waves of the grid (XCD-contiguous).
__device__ __forceinline__ int global_wave() {
    return __builtin_amdgcn_readfirstlane(xcd_remap(blockIdx.x, gridDim.x) * kWG +
                                          (int)(threadIdx.x >> 6));
}

// Word w of the bounds of image a.
__device__ __forceinline__ unsigned long long* bound_word(const BatchHeader& h, const ImgArgs& a,
                                                          int w) {
    return h.bound + ((int64_t)a.way0 + w) * h.slot_step;
}

// SPECULATE pass 0: G^2 on the sampled bands, folded into the images'
// bounds under the current epoch.  Any pixel's G^2 is at most the image's
// max, so each then holds a lower bound of it.  The first item of each
// image also clears the image's max slot (pass 1 folds into it after this
// kernel), so SPECULATE needs no reset kernel; the first item of all
// empties pass 1's queue.  The long sweep's form (64 x 1080p 15.3 us): the
// short sweep takes as long alone (16), and with its LDS does not fit beside
// another call's pass 1.
template <int KS>
__global__ __launch_bounds__(64 * kWG) __attribute__((amdgpu_waves_per_eu(sweep_waves(KS))))
void k_batch_p0(const uint8_t* __restrict__ table, Taps tp) {
    using S = SweepShape<KS, kBC, SM_MAXONLY>;
    const TableView tv = view(table);
    const int nw = gridDim.x * kWG;
    const uint64_t ep = (uint64_t)*as_global(tv.hdr.epoch) << 32;
    for (int k = global_wave(); k < tv.hdr.n_items0; k += nw) {
        const BatchItem it = tv.item(tv.items0, k);
        const ImgArgs a = tv.imgs[it.image];
        if (it.local == 0 && lane_id() < a.ways)
            as_global(a.slot)[(int64_t)lane_id() * a.slot_step] = 0u;
        if (k == 0 && lane_id() == 0) *as_global(tv.hdr.redo_n) = 0u;
        const int nstrips = (a.W + S::OW - 1) / S::OW;
        float gmax = 0.0f;
        sweep_tile<KS, kBC, SM_MAXONLY>(a, tp, (it.local % nstrips) * S::OW,
                                         (it.local / nstrips) * sample_stride(a.H), kSampleRows,
                                         0.0f, gmax);
        gmax = wave_max(gmax);
        if (lane_id() == 0)
            atomicMax(bound_word(tv.hdr, a, k & (a.ways - 1)),
                      (unsigned long long)(ep | __float_as_uint(gmax)));
    }
}

// SPECULATE pass 1's threshold on G^2 of an image: pass 0 finished before
// this kernel began, and nothing writes the bounds meanwhile.  (Reading the
// image's slot, which the other tiles keep raising, measured much slower:
// each read waits behind this wave's own atomic on the same address.)
__device__ __forceinline__ float bound_thr2(const BatchHeader& h, const ImgArgs& a) {
    uint32_t lb2 = 0u;
    if (lane_id() < a.ways) {
        const uint64_t bv = *as_global(bound_word(h, a, lane_id()));
        if ((uint32_t)(bv >> 32) == *as_global(h.epoch)) lb2 = (uint32_t)bv;
    }
    uint32_t top = __builtin_amdgcn_readfirstlane(lb2);
    for (int w = 1; w < a.ways; ++w)
        top = max(top, (uint32_t)__builtin_amdgcn_readlane((int)lb2, w));
    return thr2_from(top, h.theta) * kSpecSafety;
}
__device__ __forceinline__ SpecTile list_of(const BatchHeader& h, const ImgArgs& a, int local) {
    const int64_t base = (int64_t)a.list_base + (int64_t)local * a.list_cap;
    return SpecTile{h.cand_code + base * kBC, h.cand_row + base, 0u, a.list_cap};
}
// Count item k's entries; a list that did not hold them queues the tile.
__device__ __forceinline__ void finish_list(const BatchHeader& h, const ImgArgs& a, int k,
                                            uint32_t n) {
    if (lane_id() == 0) {
        as_global(h.cand_n)[k] = n;
        if (n > a.list_cap) h.redo[atomicAdd(h.redo_n, 1u)] = k;
    }
}

template <int KS, int PASS>
__device__ __forceinline__ void batch_p1_body(const uint8_t* __restrict__ table,
                                              const Taps& tp) {
    constexpr int M1 = PASS == HX_PASS_STORE       ? SM_STORE
                       : PASS == HX_PASS_SPECULATE ? SM_SPEC
                                                   : SM_MAXONLY;
    using S = SweepShape<KS, kBC, M1>;
    const TableView tv = view(table);
    const int nw = gridDim.x * kWG;
    for (int k = global_wave(); k < tv.hdr.n_items1; k += nw) {
        const BatchItem it = tv.item(tv.items1, k);
        const ImgArgs a = tv.imgs[it.image];
        const int nstrips = (a.W + S::OW - 1) / S::OW;
        float gmax = 0.0f;
        float thr2 = 0.0f;
        SpecTile sp{nullptr, nullptr, 0u, 0u};
        if constexpr (PASS == HX_PASS_SPECULATE) {
            thr2 = bound_thr2(tv.hdr, a);
            sp = list_of(tv.hdr, a, it.local);
        }
        // Odd bands sweep upwards (their halo rows are then read while the
        // neighbouring bands read them too).
        const int band = it.local / nstrips;
        sweep_tile<KS, kBC, M1>(a, tp, (it.local % nstrips) * S::OW, band * a.ty, a.ty, thr2,
                                gmax, &sp, (band & 1) != 0);
        if constexpr (PASS == HX_PASS_SPECULATE) finish_list(tv.hdr, a, k, sp.n);
        gmax = wave_max(gmax);
        if (lane_id() == 0) atomic_max_g2(slot_word(a, k), gmax);
    }
}

// The sweep kernels are capped at three waves per SIMD (at most 168
// registers): left alone, the scheduler keeps more rows in flight and
// the kernels fall to two waves per SIMD, which measured slower.
template <int KS, int PASS>
__global__ __launch_bounds__(64 * kWG) __attribute__((amdgpu_waves_per_eu(sweep_waves(KS))))
void k_batch_p1(const uint8_t* __restrict__ table, Taps tp) {
    batch_p1_body<KS, PASS>(table, tp);
}

template <int KS>
__global__ __launch_bounds__(64 * kWG) __attribute__((amdgpu_waves_per_eu(sweep_waves(KS))))
void k_batch_p1s(const uint8_t* __restrict__ table, Taps tp) {
    batch_p1_body<KS, HX_PASS_SPECULATE>(table, tp);
}

// SPECULATE pass 1 on tiles of up to kShortTile rows: the short sweep (the
// same tiles and list entries as the long one's), its rows in dynamic LDS.
template <int KS>
__global__ __launch_bounds__(64)
void k_batch_p1t(const uint8_t* __restrict__ table, Taps tp) {
    using S = TileShape<KS, kBC, SM_SPEC>;
    static_assert(S::OW == SweepShape<KS, kBC, SM_SPEC>::OW &&
                  S::HL == SweepShape<KS, kBC, SM_SPEC>::HL, "one tile geometry");
    extern __shared__ __align__(16) float rows[];
    const TableView tv = view(table);
    const int k = xcd_remap(blockIdx.x, gridDim.x);
    if (k >= tv.hdr.n_items1) return;
    const BatchItem it = tv.item(tv.items1, k);
    const ImgArgs a = tv.imgs[it.image];
    const int nstrips = (a.W + S::OW - 1) / S::OW;
    const int x0 = (it.local % nstrips) * S::OW, y0 = (it.local / nstrips) * a.ty;
    lds_float* lds = (lds_float*)rows;
    tile_load<kBC>(a, x0 - S::HL, y0 - S::HY, min(a.ty, a.H - y0) + 2 * S::HY, lds);
    const float thr2 = bound_thr2(tv.hdr, a);
    SpecTile sp = list_of(tv.hdr, a, it.local);
    tile_loads_done();
    float gmax = 0.0f;
    tile_sweep<KS, kBC, SM_SPEC>(a, tp, x0, y0, a.ty, thr2, gmax, lds, &sp);
    finish_list(tv.hdr, a, k, sp.n);
    gmax = wave_max(gmax);
    if (lane_id() == 0) atomic_max_g2(slot_word(a, k), gmax);
}

// Pass 2 of STORE and RECOMPUTE.  RECOMPUTE's mask-only sweep keeps the
// three-wave cap at every k: at four it spills.
template <int KS, int PASS>
__global__ __launch_bounds__(64 * kWG) __attribute__((amdgpu_waves_per_eu(HX_SWEEP_WAVES)))
void k_batch_p2(const uint8_t* __restrict__ table, Taps tp) {
    using S = SweepShape<KS, kBC, SM_MASK>;
    const TableView tv = view(table);
    const int nw = gridDim.x * kWG;
    const int lane = lane_id();
    for (int k = global_wave(); k < tv.hdr.n_items2; k += nw) {
        const BatchItem it = tv.item(tv.items2, k);
        const ImgArgs a = tv.imgs[it.image];
        const uint32_t m2 = slot_max(a);
        const float thr2 = thr2_from(m2, tv.hdr.theta);
        if (it.local == 0 && lane == 0 && a.dmax) *as_global(a.dmax) = max_from(m2);
        if constexpr (PASS == HX_PASS_STORE) {
            const int rb = p2_rows(a.W);
            const int r0 = it.local * rb;
            const int r1 = min(a.H, r0 + rb);
            const int wq = (a.W + 3) / 4;
            const bool mvec = ((reinterpret_cast<uintptr_t>(a.mask) % 4) == 0) &
                              ((a.mp % 4) == 0);
            for (int y = r0; y < r1; ++y)
                for (int q = lane; q < wq; q += 64) threshold4(a, y, q * 4, thr2, mvec);
        } else {
            const int nstrips = (a.W + S::OW - 1) / S::OW;
            float unused = 0.0f;
            const int band = it.local / nstrips;
            sweep_tile<KS, kBC, SM_MASK>(a, tp, (it.local % nstrips) * S::OW, band * a.ty, a.ty,
                                         thr2, unused, nullptr, (band & 1) != 0);
        }
    }
}

// The form of small batches (kPassShort): the maxima of all tiles, then the
// masks against them, in two launches of the short sweep on 8-row tiles.  A
// small batch is bound by its launches and by what one wave takes for its
// tile, so a third launch, and pass 1's wider tiles with their lists, cost
// more than the second blur.  Whole calls, us, this form and SPECULATE: 16
// images of 64..256 k3 10.9 and 22.6, 4 x 512x512 k5 15.9 and 22.7,
// 1080x1920 k5 17.3 and 23.2, 2 of them 22.2 and 25.7, 3 of them 27.8 and
// 31.0, 4 of them 52.5 and 33.1.  Each tile's arguments come from the launch
// where they can, which saves a chain of loads through the table's header.
template <int KS, int C>
__global__ __launch_bounds__(64) void k_batch_short_max(ShortArgs s, Taps tp) {
    using S = TileShape<KS, C, SM_MAXONLY>;
    constexpr int OW = TileShape<KS, C, SM_MASK>::OW;
    static_assert(S::OW >= OW, "the mask's tiles cover the image");
    __shared__ __align__(16) float rows[S::lds_floats(kShortBatchRows)];
    const int k = xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem it = s.items ? s.items[k] : BatchItem{0, k};
    const ImgArgs a = s.imgs[it.image];
    const int nstrips = (a.W + OW - 1) / OW;
    const int x0 = (it.local % nstrips) * OW, y0 = (it.local / nstrips) * kShortBatchRows;
    lds_float* lds = (lds_float*)rows;
    tile_load<C>(a, x0 - S::HL, y0 - S::HY, min(kShortBatchRows, a.H - y0) + 2 * S::HY, lds);
    tile_loads_done();
    float gmax = 0.0f;
    tile_sweep<KS, C, SM_MAXONLY>(a, tp, x0, y0, kShortBatchRows, 0.0f, gmax, lds);
    gmax = wave_max(gmax);
    if (lane_id() == 0) atomic_max_g2(slot_word(a, k) + s.set, gmax);
}

template <int KS, int C>
__global__ __launch_bounds__(64) void k_batch_short_mask(ShortArgs s, Taps tp) {
    using S = TileShape<KS, C, SM_MASK>;
    __shared__ __align__(16) float rows[S::lds_floats(kShortBatchRows)];
    const int k = xcd_remap(blockIdx.x, gridDim.x);
    const BatchItem it = s.items ? s.items[k] : BatchItem{0, k};
    ImgArgs a = s.imgs[it.image];
    const int nstrips = (a.W + S::OW - 1) / S::OW;
    const int x0 = (it.local % nstrips) * S::OW, y0 = (it.local / nstrips) * kShortBatchRows;
    lds_float* lds = (lds_float*)rows;
    tile_load<C>(a, x0 - S::HL, y0 - S::HY, min(kShortBatchRows, a.H - y0) + 2 * S::HY, lds);
    a.slot += s.set;
    const uint32_t m2 = slot_max(a);
    if (it.local == 0 && lane_id() == 0 && a.dmax) *as_global(a.dmax) = max_from(m2);
    // The next call's words.
    for (int w = blockIdx.x * 64 + lane_id(); w < s.nzero; w += gridDim.x * 64)
        as_global(s.other)[(int64_t)w * a.slot_step] = 0u;
    tile_loads_done();
    float unused = 0.0f;
    tile_sweep<KS, C, SM_MASK>(a, tp, x0, y0, kShortBatchRows, thr2_from(m2, s.theta), unused,
                               lds);
}

// Columns per lane and rows of the pieces SPECULATE's pass 2 redoes queued
// tiles in (8 KB of LDS per wave at k = 5).
constexpr int kRedoC = 2, kRedoRows = 8;

// SPECULATE pass 2: one wave per tile, as short as the loads it waits for
// allow (item and count, image, max and entries), so many waves are kept in
// flight: the redo of queued tiles is the short sweep's, which leaves the
// kernel 73 registers and 11 KB of code (the long sweep's mask-only form took
// 130 and 250 KB), so a wave of it fits beside three of another call's pass 1
// on each SIMD.  Queued tiles are redone by all waves of the grid, a piece of
// 8 rows at a time.  64 x 1080p 19 us, 256 uneven images 21.6; as workgroups
// of four waves with 32 KB that shared a run of lists 19 and 23.6, and four
// calls in flight took 0.157 ms each, not 0.150.
// CLAIM: the same with 128 registers claimed, so that its waves take places of
// another call's pass 1 (136 registers, three on a SIMD) instead of squeezing
// in beside it.  Which is faster with calls in flight depends on how their
// rounds of tiles fall together, so the batch tuner tries both.  us a call,
// beside / claimed: 64 x 1080p k5 on 3 and 4 streams 161 / 147 and 137..150 /
// 132, 2 streams 163 / 165, alone 183.4 / 184.7; 200 images of 64..2048 on 2
// and 4 streams 105 / 114 and 97 / 101; 256 x 512x512 on 2 streams 97 / 105.
template <int KS, bool CLAIM>
__global__ __launch_bounds__(64)
void k_batch_p2s(const uint8_t* __restrict__ table, Taps tp) {
    using S = SweepShape<KS, kBC, SM_SPEC>;
    using RS = TileShape<KS, kRedoC, SM_MASK>;
    __shared__ __align__(16) float rows[RS::lds_floats(kRedoRows)];
    if constexpr (CLAIM) asm volatile("" ::: "v127");
    const TableView tv = view(table);
    const int lane = lane_id();
    const int k = xcd_remap(blockIdx.x, gridDim.x);
    if (k < tv.hdr.n_items2) {
        const BatchItem it = tv.item(tv.items2, k);
        const int n_listed = (int)as_global(tv.hdr.cand_n)[k];
        const ImgArgs a = tv.imgs[it.image];
        const SpecTile sp = list_of(tv.hdr, a, it.local);
        const uint32_t m2 = a.ways > 1 ? slot_max(a) : *as_global(a.slot);
        const float thr2 = thr2_from(m2, tv.hdr.theta);
        if (it.local == 0 && lane == 0 && a.dmax) *as_global(a.dmax) = max_from(m2);
        // The last reader of this batch's bounds has finished: advance the
        // epoch for the next batch on this context.
        if (k == 0 && lane == 0) *as_global(tv.hdr.epoch) += 1u;
        const int nstrips = (a.W + S::OW - 1) / S::OW;
        const int left = (it.local % nstrips) * S::OW - S::HL;
        const int y0 = (it.local / nstrips) * a.ty;
        const int n = (uint32_t)n_listed > sp.cap ? 0 : n_listed;   // incomplete: queued
        const bool mvec = ((reinterpret_cast<uintptr_t>(a.mask) % 4) == 0) & ((a.mp % 4) == 0);
        for (int t = lane; t < n; t += 64) {
            const gptr<const VecF<kBC>> q = (gptr<const VecF<kBC>>)as_global(sp.code) + t;
            const uint32_t rw = (uint32_t)as_global(sp.row)[t];
            const int cbase = left + kBC * (int)((rw >> 4) & 63u);
            const gptr<uint8_t> rp =
                as_global(a.mask) + (int64_t)(y0 + (int)(rw >> 10)) * a.mp + cbase;
            // Pass 1 set every listed pixel to 1 and left the others of the
            // lane-row at 0.  Only a listed pixel at or below the true
            // threshold changes (to 0): the lane-row is rewritten, as one
            // aligned word when it lies inside the image, only if one did.
            // Those are few when the bound is close to the max, and
            // scattered partial writes are what this pass spends its time
            // on.  Both loads are unconditional, so they are in flight
            // together.
            float g2v[kBC];
#pragma unroll
            for (int e = 0; e < kBC; ++e) g2v[e] = q->v[e];
            uint32_t w = 0, was = 0;
#pragma unroll
            for (int e = 0; e < kBC; ++e) {
                const uint32_t listed = (rw >> e) & 1u;
                was |= listed << (8 * e);
                w |= (listed & (uint32_t)(g2v[e] > thr2)) << (8 * e);
            }
            if (w != was) {
                if (kBC == 4 && mvec && cbase + 4 <= a.W) {
                    *(gptr<uint32_t>)rp = w;
                } else {
#pragma unroll
                    for (int e = 0; e < kBC; ++e)
                        if (((was ^ w) >> (8 * e)) & 1u) rp[e] = 0;
                }
            }
        }
    }
    // Queued tiles, against the true threshold (every pixel's final value,
    // also where a piece's last strip reaches into the next tile).
    const uint32_t nq = *as_global(tv.hdr.redo_n);
    if (nq == 0) return;
    constexpr int kAcross = (S::OW + RS::OW - 1) / RS::OW;
    const int per = kAcross * ((tv.hdr.ty + kRedoRows - 1) / kRedoRows);
    lds_float* lds = (lds_float*)rows;
    for (int64_t c = blockIdx.x; c < (int64_t)nq * per; c += gridDim.x) {
        const int kq = __builtin_amdgcn_readfirstlane(as_global(tv.hdr.redo)[c / per]);
        const int r = (int)(c % per);
        const BatchItem it = tv.item(tv.items2, kq);
        const ImgArgs a = tv.imgs[it.image];
        const int nstrips = (a.W + S::OW - 1) / S::OW;
        const int x0 = (it.local % nstrips) * S::OW + (r % kAcross) * RS::OW;
        const int y0 = (it.local / nstrips) * a.ty + (r / kAcross) * kRedoRows;
        if (x0 >= a.W || y0 >= a.H) continue;
        tile_load<kRedoC>(a, x0 - RS::HL, y0 - RS::HY, min(kRedoRows, a.H - y0) + 2 * RS::HY,
                          lds);
        const float thr2 = thr2_from(slot_max(a), tv.hdr.theta);
        tile_loads_done();
        float unused = 0.0f;
        tile_sweep<KS, kRedoC, SM_MASK>(a, tp, x0, y0, kRedoRows, thr2, unused, lds);
    }
}

}  // namespace hx
