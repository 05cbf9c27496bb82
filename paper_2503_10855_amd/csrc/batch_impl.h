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
// re-decides only the listed pixels in pass 2 (the lists of up to
// kP2Tiles pass-1 tiles per workgroup).  A tile whose list did not hold its
// pixels is queued by pass 1 and redone by pass 2 in 8-row pieces.
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

// Columns per lane of pass 0's tiles.  They are 8 rows tall, so the short
// sweep runs them (see tile_impl.h).  On 64 x 1080p the pass reads 41 MB and
// is bound by that: 17.0 us by the long sweep, 15.8 by this one (17.0 with 4
// columns per lane); on 16 images of 64..256, 5.2 and 4.5 us.
constexpr int kP0C = 2;

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
// empties pass 1's queue.
template <int KS>
__global__ __launch_bounds__(64)
void k_batch_p0(const uint8_t* __restrict__ table, Taps tp) {
    using S = TileShape<KS, kP0C, SM_MAXONLY>;
    __shared__ __align__(16) float rows[S::lds_floats(kSampleRows)];
    const TableView tv = view(table);
    const uint64_t ep = (uint64_t)*as_global(tv.hdr.epoch) << 32;
    const int k = xcd_remap(blockIdx.x, gridDim.x);   // one item per workgroup
    if (k >= tv.hdr.n_items0) return;
    const BatchItem it = tv.item(tv.items0, k);
    const ImgArgs a = tv.imgs[it.image];
    const int nstrips = (a.W + S::OW - 1) / S::OW;
    const int x0 = (it.local % nstrips) * S::OW;
    const int y0 = (it.local / nstrips) * sample_stride(a.H);
    lds_float* lds = (lds_float*)rows;
    tile_load<kP0C>(a, x0 - S::HL, y0 - S::HY, min(kSampleRows, a.H - y0) + 2 * S::HY, lds);
    if (it.local == 0 && lane_id() < a.ways)
        as_global(a.slot)[(int64_t)lane_id() * a.slot_step] = 0u;
    if (k == 0 && lane_id() == 0) *as_global(tv.hdr.redo_n) = 0u;
    tile_loads_done();
    float gmax = 0.0f;
    tile_sweep<KS, kP0C, SM_MAXONLY>(a, tp, x0, y0, kSampleRows, 0.0f, gmax, lds);
    gmax = wave_max(gmax);
    if (lane_id() == 0)
        atomicMax(bound_word(tv.hdr, a, k & (a.ways - 1)),
                  (unsigned long long)(ep | __float_as_uint(gmax)));
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
// images of 64..256 k3 14.5 and 24.4, 4 x 512x512 k5 17.1 and 28.0,
// 1080x1920 k5 18.6 and 25.4, 2 of them 25.0 and 28.8, 3 of them 30.8 and
// 32.0, 4 of them 39.8 and 33.8.  Each tile's arguments come from the launch
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

// Tiles whose lists one workgroup of SPECULATE's pass 2 takes, at most, and
// the columns per lane of the pieces it redoes queued tiles in (8 rows
// each; four waves' rows are 32 KB of LDS at k = 5, five workgroups per CU).
constexpr int kP2Tiles = 16, kRedoC = 2, kRedoRows = 8;

// SPECULATE pass 2.  A tile's list is short (about 110 entries on average
// on 1080p frames), so the pass is bound by latency: one wave per tile had
// 8700 waves each wait for item, count and entries in turn (16 us, 38 us
// when one of them redid a whole 64-row tile).  Here each workgroup reads
// the state of up to kP2Tiles tiles with one lane each, and its 256 threads
// then walk the concatenated lists, several entries in flight per thread;
// tiles are dealt out one per workgroup in turn, as dense lists are
// neighbours.  Queued tiles are redone by all waves of the grid, a piece
// of 8 rows at a time.  64 x 1080p (51 queued tiles): 38.3 -> 17.7 us; 256
// images of 64..2048 (172 queued): 43.4 -> 22.8 us.
template <int KS>
__global__ __launch_bounds__(256)
void k_batch_p2s(const uint8_t* __restrict__ table, Taps tp) {
    using S = SweepShape<KS, kBC, SM_SPEC>;
    using RS = TileShape<KS, kRedoC, SM_MASK>;
    struct Tile {
        const float* code;
        const int32_t* row;
        uint8_t* mask;    // of column 0 of lane 0's first column, top row
        int64_t mp;
        float thr2;
        int left;         // columns from there to the image's right edge
        int words;        // mask rows are word aligned
    };
    __shared__ Tile st[kP2Tiles];
    __shared__ uint32_t first[kP2Tiles + 1];   // entries before tile j
    __shared__ __align__(16) float rows[4 * RS::lds_floats(kRedoRows)];
    const TableView tv = view(table);
    const int tid = threadIdx.x;
    const int n = tv.hdr.n_items2, G = gridDim.x;
    // 16 threads per tile read its state (and the words of its image's max).
    static_assert(kP2Tiles * 16 == 256, "16 threads per tile");
    {
        const int j = tid >> 4, l = tid & 15;
        const int64_t k = blockIdx.x + (int64_t)j * G;
        uint32_t cnt = 0;
        if (k < n) {
            const BatchItem it = tv.item(tv.items2, k);
            const ImgArgs& a = tv.imgs[it.image];
            cnt = as_global(tv.hdr.cand_n)[k];
            uint32_t m2 = 0;
            for (int w = l; w < a.ways; w += 16)
                m2 = max(m2, as_global(a.slot)[(int64_t)w * a.slot_step]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) m2 = max(m2, (uint32_t)__shfl_xor((int)m2, o, 16));
            const int nstrips = (a.W + S::OW - 1) / S::OW;
            const int x0 = (it.local % nstrips) * S::OW, y0 = (it.local / nstrips) * a.ty;
            const SpecTile sp = list_of(tv.hdr, a, it.local);
            if (cnt > sp.cap) cnt = 0;   // incomplete: queued
            if (l == 0) {
                if (it.local == 0 && a.dmax) *as_global(a.dmax) = max_from(m2);
                st[j] = Tile{sp.code, sp.row, a.mask + (int64_t)y0 * a.mp + (x0 - S::HL), a.mp,
                             thr2_from(m2, tv.hdr.theta), a.W - (x0 - S::HL),
                             ((reinterpret_cast<uintptr_t>(a.mask) | (uint64_t)a.mp) & 3u) == 0};
            }
        }
        if (l == 0) first[j + 1] = cnt;
    }
    __syncthreads();
    if (tid < kP2Tiles) {
        uint32_t sum = first[tid + 1];
#pragma unroll
        for (int o = 1; o < kP2Tiles; o <<= 1) {
            const uint32_t up = __shfl_up(sum, o, kP2Tiles);
            if (tid >= o) sum += up;
        }
        first[tid + 1] = sum;
        if (tid == 0) {
            first[0] = 0;
            // The last reader of this batch's bounds has finished: advance
            // the epoch for the next batch on this context.
            if (blockIdx.x == 0) *as_global(tv.hdr.epoch) += 1u;
        }
    }
    __syncthreads();
    const uint32_t total = first[kP2Tiles];
    constexpr int U = 4;   // entries in flight per thread
    for (uint32_t t0 = tid; t0 < total; t0 += 256 * U) {
        VecF<kBC> g2[U];
        uint32_t rw[U];
        int tj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t t = min(t0 + 256u * u, total - 1);
            int j = 0;
#pragma unroll
            for (int b = kP2Tiles / 2; b > 0; b >>= 1)
                if (first[j + b] <= t) j += b;
            const uint32_t i = t - first[j];
            const gptr<const VecF<kBC>> q = (gptr<const VecF<kBC>>)as_global(st[j].code) + i;
#pragma unroll
            for (int e = 0; e < kBC; ++e) g2[u].v[e] = q->v[e];
            rw[u] = (uint32_t)as_global(st[j].row)[i];
            tj[u] = j;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t0 + 256u * u >= total) break;
            // Pass 1 set every listed pixel to 1 and left the others of the
            // lane-row at 0.  Only a listed pixel at or below the true
            // threshold changes (to 0): the lane-row is rewritten, as one
            // aligned word when it lies inside the image, only if one did.
            const Tile& T = st[tj[u]];
            uint32_t w = 0, was = 0;
#pragma unroll
            for (int e = 0; e < kBC; ++e) {
                const uint32_t listed = (rw[u] >> e) & 1u;
                was |= listed << (8 * e);
                w |= (listed & (uint32_t)(g2[u].v[e] > T.thr2)) << (8 * e);
            }
            if (w != was) {
                const int col = kBC * (int)((rw[u] >> 4) & 63u);
                const gptr<uint8_t> rp =
                    as_global(T.mask) + (int64_t)(rw[u] >> 10) * T.mp + col;
                if (kBC == 4 && T.words && col + 4 <= T.left) {
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
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = kAcross * ((tv.hdr.ty + kRedoRows - 1) / kRedoRows);
    lds_float* lds = (lds_float*)rows + wave * RS::lds_floats(kRedoRows);
    for (int64_t c = (int64_t)blockIdx.x * 4 + wave; c < (int64_t)nq * per; c += 4 * (int64_t)G) {
        const int k = __builtin_amdgcn_readfirstlane(as_global(tv.hdr.redo)[c / per]);
        const int r = (int)(c % per);
        const BatchItem it = tv.item(tv.items2, k);
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
