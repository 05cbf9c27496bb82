// tile_impl.h -- the short fused sweep: the stages of sweep_impl.h over a
// short tile (8 to 16 rows), in a loop of one row per turn.
//
// What bounds a short tile is neither memory nor arithmetic but
// instruction fetch: the long sweep unrolls its pipeline fill and eight
// rows of its steady state (about 22 KB per border variant, 130-300 KB per
// kernel), every launch starts with a cold instruction cache, and a tile of
// 8 or 16 rows runs each of those instructions once or twice.  This sweep
// keeps the row loop small (the turns of one stage set share one body,
// unrolled by kTurn so that row rings rotate without moves) and has one
// variant for every border and alignment, chosen by uniform branches, so a
// whole kernel is a few KB and each instruction is fetched once per wave
// group.
//
// Input: all rows of the tile go to LDS at once, by direct buffer-to-LDS
// loads with clamped rows and columns (one memory latency per tile instead
// of one per prefetch distance); each wave reads only what it loaded, so
// no barrier is needed.  Arithmetic and its order are hx_device.h's, as in
// every other schedule: the same bits.
#pragma once

#include "sweep_impl.h"

namespace hx {

template <int KS, int C, int MODE>
struct TileShape {
    static constexpr int R = KS / 2;
    static constexpr int HY = MODE == TM_BLUR ? R : MODE == SM_MAXONLY ? R + 1 : R + 2;
    static constexpr int HL = ((HY + C - 1) / C) * C;      // left halo (whole lanes)
    static constexpr int SW = 64 * C;
    static constexpr int OW = ((SW - HL - HY) / C) * C;
    static constexpr bool NEED_C = MODE != TM_BLUR;        // Sobel and the max
    static constexpr bool NEED_Z =
        MODE == SM_STORE || MODE == TM_STAGES || MODE == SM_MASK || MODE == SM_SPEC;
    static constexpr bool DO_MAX = NEED_C && MODE != SM_MASK;
    static constexpr bool CODE = MODE == SM_STORE || MODE == TM_STAGES;
    static constexpr bool TO_MASK = MODE == SM_MASK || MODE == SM_SPEC;
    // Floats of LDS one wave's tile of ty rows takes.
    __host__ __device__ static constexpr int lds_floats(int ty) { return (ty + 2 * HY) * SW; }
};

// Turns per loop body: the longest row ring's length for k = 5 (4-row
// bodies measured 0-4 % faster than 2-row ones, 1-row bodies 10 % slower).
constexpr int kTurn = 4;

typedef __attribute__((address_space(3))) float lds_float;

// Input rows y0 - HY .. y0 + ty + HY - 1 of columns xs .. xs + SW - 1,
// clamped into the image, to the wave's LDS rows.  Interior strips of
// C = 4 take one 16-byte load per lane and row; the others one 4-byte load
// per column group (lane l of group j holds column 64 j + l).
template <int C>
__device__ __forceinline__ void tile_load(const ImgArgs& a, int xs, int row0, int rows,
                                          lds_float* lds) {
    constexpr int SW = 64 * C;
    const int lane = lane_id();
    const int in0 = clampi(row0, 0, a.H - 1), in1 = clampi(row0 + rows - 1, 0, a.H - 1);
    const RowSpan src(a.src, in0, in1 - in0 + 1, a.sp, 4, a.W);
    if (C == 4 && xs >= 0 && xs + SW <= a.W) {
        const uint32_t off = (uint32_t)(xs + 4 * lane) * 4u;
        for (int t = 0; t < rows; ++t)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                src.r, (__attribute__((address_space(3))) void*)(lds + t * SW), 16, off,
                src.soff(clampi(row0 + t, 0, a.H - 1)), 0, 0);
    } else {
        uint32_t off[C];
#pragma unroll
        for (int j = 0; j < C; ++j)
            off[j] = (uint32_t)clampi(xs + 64 * j + lane, 0, a.W - 1) * 4u;
        for (int t = 0; t < rows; ++t) {
            const uint32_t so = src.soff(clampi(row0 + t, 0, a.H - 1));
#pragma unroll
            for (int j = 0; j < C; ++j)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    src.r, (__attribute__((address_space(3))) void*)(lds + t * SW + 64 * j), 4,
                    off[j], so, 0, 0);
        }
    }
}

// Every load of this wave into LDS has arrived.
__device__ __forceinline__ void tile_loads_done() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int C>
__device__ __forceinline__ void lds_row(const lds_float* lds, int t, float (&v)[C]) {
    const lds_float* p = lds + t * (64 * C) + C * lane_id();
    if constexpr (C == 1) {
        v[0] = *p;
    } else {
        typedef float vec __attribute__((ext_vector_type(C)));
        const vec r = *(const __attribute__((address_space(3))) vec*)p;
#pragma unroll
        for (int e = 0; e < C; ++e) v[e] = r[e];
    }
}

// A lane's C mask bytes (in w) at byte offset off of mask row `row`: whole
// words where the row is word aligned, else naturally aligned pieces (rem,
// the row's low address bits, is the same for every lane since a lane's
// first column is a multiple of 4); with fewer than C columns inside the
// image, single bytes.
template <int C>
__device__ __forceinline__ void store_mask(const RowSpan& msk, int row, uint32_t off, uint32_t w,
                                           uint32_t mlo, int ncol) {
    const uint32_t so = msk.soff(row);
    const uint32_t rem = (mlo + so) & 3u;
    if (C == 4 && ncol >= C) {
        if (rem == 0u) {
            __builtin_amdgcn_raw_buffer_store_b32(w, msk.r, off, so, 0);
        } else if (rem == 2u) {
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(w & 0xffffu), msk.r, off, so, 0);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(w >> 16), msk.r, off + 2u, so, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(w & 0xffu), msk.r, off, so, 0);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)((w >> 8) & 0xffffu), msk.r,
                                                  off + 1u, so, 0);
            __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(w >> 24), msk.r, off + 3u, so, 0);
        }
    } else {
#pragma unroll
        for (int e = 0; e < C; ++e)
            if (e < ncol)
                __builtin_amdgcn_raw_buffer_store_b8((unsigned char)((w >> (8 * e)) & 0xffu),
                                                     msk.r, off + e, so, 0);
    }
}

// A lane's C floats at column `col` of row `row` of a plane; ncol of them
// lie inside the plane's rows.
template <int C>
__device__ __forceinline__ void store_floats(const RowSpan& p, int row, int col,
                                             const float (&v)[C], int ncol) {
    if (ncol >= C) {
        span_store<C>(p, row, (uint32_t)col * 4u, v);
    } else {
#pragma unroll
        for (int e = 0; e < C; ++e)
            if (e < ncol)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[e]), p.r,
                                                      (uint32_t)(col + e) * 4u, p.soff(row), 0);
    }
}

// The values at columns -1 and W of a row whose columns lie outside the
// image there: column 0's and column W - 1's (no stage reaches further than
// one column past what it replaces).  left_fix: the lane that holds column
// -1 (in its last element); right_fix[e]: column W is this lane's element e.
template <int C>
__device__ __forceinline__ void edge_cols(float (&x)[C], bool left_fix,
                                          const bool (&right_fix)[C]) {
    const float from_r = lane_fetch<1>(x[0]);
    x[C - 1] = left_fix ? from_r : x[C - 1];
    const float from_l = lane_fetch<-1>(x[C - 1]);
#pragma unroll
    for (int e = C - 1; e > 0; --e) x[e] = right_fix[e] ? x[e - 1] : x[e];
    x[0] = right_fix[0] ? from_l : x[0];
}

// One tile: output columns [x0, x0 + OW) x rows [y0, y0 + ty) clipped to the
// image, which must hold (x0, y0); ty a multiple of kTurn.  BD: the tile's
// window crosses a border of the image.  lds: the wave's
// TileShape::lds_floats(ty) floats, filled by tile_load.  gmax, thr2, sp: as
// sweep_tile.
template <int KS, int C, int MODE, bool BD>
__device__ __forceinline__ void tile_body(const ImgArgs& a, const Taps& tp, int x0, int y0,
                                          int ty, float thr2, float& gmax, const lds_float* lds,
                                          SpecTile* sp, const StageOut* so) {
    using S = TileShape<KS, C, MODE>;
    constexpr int R = S::R, HY = S::HY, HL = S::HL;
    constexpr int NB = KS > 1 ? KS - 1 : 1;   // earlier Bh rows the vertical blur reads
    const int H = a.H, W = a.W, lane = lane_id();
    const int xs = x0 - HL, cbase = xs + C * lane;
    const int ylim = BD ? min(y0 + ty, H) : y0 + ty;
    const int NS = ylim - y0 + 2 * HY;
    const bool lane_out = (cbase >= x0) & (cbase < x0 + S::OW) & (!BD || cbase < W);
    const int ncol = lane_out ? (BD ? min(W - cbase, C) : C) : 0;  // output columns
    const bool left_fix = BD && cbase + C == 0;
    bool right_fix[C];
    uint32_t emw = 0;   // the lane's output columns, as 0xff bytes
#pragma unroll
    for (int e = 0; e < C; ++e) {
        right_fix[e] = BD && cbase + e == W;
        emw |= e < ncol ? (0xffu << (8 * e)) : 0u;
    }

    const RowSpan msk(S::TO_MASK ? (const void*)a.mask : (const void*)a.src, y0, ylim - y0,
                      S::TO_MASK ? a.mp : 0, 1, W);
    const uint32_t mlo =
        S::TO_MASK
            ? (uint32_t)(reinterpret_cast<uintptr_t>(a.mask) + (uint64_t)y0 * (uint64_t)a.mp) & 3u
            : 0u;
    constexpr bool TO_F = S::CODE || MODE == TM_BLUR;
    // Rows of fout hold a.op >= round_up(W, 4) floats, so a lane whose first
    // column is inside the image writes all its C.
    const RowSpan fo(TO_F ? (const void*)a.fout : (const void*)a.src, y0, ylim - y0,
                     TO_F ? a.op : 0, 4, TO_F ? (int)a.op : W);

    float bh[NB][C];             // bh[i]: horizontal blur, i + 1 rows ago
    float b1[C], b2[C];          // B one and two rows ago
    float ew1[C], sy1[C], sy2[C];
    uint32_t ho1 = 0, ho2 = 0, ha1 = 0, ha2 = 0, tbd = 0;
    float g2d[C];
    float gacc = 0.0f;
    float in[C];
    lds_row<C>(lds, 0, in);
#pragma unroll
    for (int e = 0; e < C; ++e) {
        b1[e] = b2[e] = ew1[e] = sy1[e] = sy2[e] = g2d[e] = 0.0f;
#pragma unroll
        for (int i = 0; i < NB; ++i) bh[i][e] = 0.0f;
    }

    // One turn: input row y0 - HY + t; ST: stages active (1: horizontal
    // blur, 2: and B, 3: and L, G^2, 4: and Z with the output).
    auto turn = [&](auto stt, int t) {
        constexpr int ST = decltype(stt)::value;
        const int v = y0 - HY + t;
        float nxt[C];
        lds_row<C>(lds, min(t + 1, NS - 1), nxt);

        // ---- A
        float h[C];
        {
            float ext[C + 2 * R];
            static_for([&](auto kt) {
                constexpr int kk = decltype(kt)::value - R;
                constexpr int q = kk >= 0 ? kk / C : -((-kk + C - 1) / C);
                ext[kk + R] = lane_fetch<q>(in[kk - q * C]);
            }, std::make_integer_sequence<int, C + 2 * R>{});
#pragma unroll
            for (int e = 0; e < C; ++e) h[e] = blur_chain<KS>(&ext[e], tp);
        }
#pragma unroll
        for (int e = 0; e < C; ++e) in[e] = nxt[e];

        // ---- B: row vb
        if constexpr (ST >= 2) {
            const int vb = v - R;
            float b[C];
#pragma unroll
            for (int e = 0; e < C; ++e) {
                float col[KS];
                col[KS - 1] = h[e];
#pragma unroll
                for (int i = 0; i < KS - 1; ++i) col[i] = bh[KS - 2 - i][e];
                b[e] = blur_chain<KS>(col, tp);
            }
            if constexpr (MODE == TM_BLUR) {
                if (ncol > 0) store_floats<C>(fo, vb, cbase, b, C);
            } else {
                if constexpr (BD) {
                    if (vb >= H) {
#pragma unroll
                        for (int e = 0; e < C; ++e) b[e] = b1[e];
                    }
                    edge_cols<C>(b, left_fix, right_fix);
                }
                const float bl0 = lane_fetch<-1>(b[C - 1]);
                const float br0 = lane_fetch<1>(b[0]);
                float ew[C], sy[C];
#pragma unroll
                for (int e = 0; e < C; ++e) {
                    const float l = e > 0 ? b[e - 1] : bl0;
                    const float r = e < C - 1 ? b[e + 1] : br0;
                    ew[e] = l + r;
                    sy[e] = sobel_sy(ew[e], b[e]);
                }
                if constexpr (BD) {
                    if (vb == 0) {   // the row above the image is row 0
#pragma unroll
                        for (int e = 0; e < C; ++e) {
                            b1[e] = b[e];
                            sy1[e] = sy[e];
                        }
                    }
                }
                // ---- C: row vl
                if constexpr (ST >= 3) {
                    const int vl = vb - 1;
                    const bool row_out = (vl >= y0) & (vl < ylim);
                    float ns[C], vs[C], g2[C];
#pragma unroll
                    for (int e = 0; e < C; ++e) {
                        ns[e] = b2[e] + b[e];
                        vs[e] = sobel_vs(ns[e], b1[e]);
                    }
                    const float vsl0 = lane_fetch<-1>(vs[C - 1]);
                    const float vsr0 = lane_fetch<1>(vs[0]);
#pragma unroll
                    for (int e = 0; e < C; ++e)
                        g2[e] = sobel_g2(e > 0 ? vs[e - 1] : vsl0, e < C - 1 ? vs[e + 1] : vsr0,
                                         sy2[e], sy[e]);
                    if constexpr (S::DO_MAX) {
                        if constexpr (BD) {
                            if (row_out) {
#pragma unroll
                                for (int e = 0; e < C; ++e)
                                    gacc = __builtin_fmaxf(gacc, e < ncol ? g2[e] : 0.0f);
                            }
                        } else {
                            // Every row here is a real pixel row, and the
                            // max is idempotent.
#pragma unroll
                            for (int e = 0; e < C; ++e) gacc = __builtin_fmaxf(gacc, g2[e]);
                        }
                    }
                    if constexpr (S::NEED_Z) {
                        float l[C];
#pragma unroll
                        for (int e = 0; e < C; ++e) l[e] = lap_from(ns[e], ew1[e], b1[e]);
                        if constexpr (MODE == TM_STAGES) {
                            if (row_out) {
                                if (so->B) {
                                    const RowSpan p(so->B, vl, 1, W, 4, W);
                                    store_floats<C>(p, vl, cbase, b1, ncol);
                                }
                                if (so->L) {
                                    const RowSpan p(so->L, vl, 1, W, 4, W);
                                    store_floats<C>(p, vl, cbase, l, ncol);
                                }
                                if (so->G) {
                                    const RowSpan p(so->G, vl, 1, W, 4, W);
                                    float g[C];
#pragma unroll
                                    for (int e = 0; e < C; ++e) g[e] = __builtin_sqrtf(g2[e]);
                                    store_floats<C>(p, vl, cbase, g, ncol);
                                }
                            }
                        }
                        if constexpr (BD) edge_cols<C>(l, left_fix, right_fix);
                        uint32_t sb[C];
#pragma unroll
                        for (int e = 0; e < C; ++e) sb[e] = pos_bit(l[e]);
                        const uint32_t sw = col_bytes<C>(sb);
                        const uint32_t sl = cols_from_left<C>(sw), sr = cols_from_right<C>(sw);
                        uint32_t ho = sw | sl | sr, ha = sw & sl & sr;
                        if constexpr (BD) {
                            if (vl >= H) {
                                ho = ho1;
                                ha = ha1;
                            }
                            if (vl == 0) {
                                ho1 = ho;
                                ha1 = ha;
                            }
                        }
                        // ---- D: row vz
                        if constexpr (ST >= 4) {
                            const int vz = vl - 1;
                            const uint32_t zw = (ho2 | ho1 | ho) & ~(ha2 & ha1 & ha);
                            const bool out = ncol > 0 && (!BD || vz < ylim);
                            if constexpr (S::CODE) {
                                float cd[C];
#pragma unroll
                                for (int e = 0; e < C; ++e)
                                    cd[e] = pass1_code((zw >> (8 * e)) & 1u, g2d[e]);
                                if (out) store_floats<C>(fo, vz, cbase, cd, C);
                            }
                            if constexpr (MODE == TM_STAGES) {
                                if (so->Z && out) {
                                    const RowSpan p(so->Z, vz, 1, W, 1, W);
                                    const uint32_t zlo =
                                        (uint32_t)(reinterpret_cast<uintptr_t>(so->Z) +
                                                   (uint64_t)vz * (uint64_t)W) & 3u;
                                    store_mask<C>(p, vz, (uint32_t)cbase, zw, zlo, ncol);
                                }
                            }
                            if constexpr (S::TO_MASK) {
                                const uint32_t mw = zw & tbd & emw;
                                if (out) store_mask<C>(msk, vz, (uint32_t)cbase, mw, mlo, ncol);
                                if constexpr (MODE == SM_SPEC) {
                                    const lmask bal = __ballot(out && mw != 0u);
                                    if (bal) {
                                        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                                            (uint32_t)(bal >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                                        const uint32_t idx = sp->n + below;
                                        if (out & (mw != 0u) & (idx < sp->cap)) {
                                            const gptr<VecF<C>> q = at_off<VecF<C>>(
                                                as_global(sp->code), idx * (uint32_t)(4 * C));
#pragma unroll
                                            for (int e = 0; e < C; ++e) q->v[e] = g2d[e];
                                            *at_off<int32_t>(as_global(sp->row), idx * 4u) =
                                                (int32_t)(((uint32_t)(vz - y0) << 10) |
                                                          ((uint32_t)lane << 4) |
                                                          col_nibble(mw));
                                        }
                                        sp->n += (uint32_t)__builtin_popcountll(bal);
                                    }
                                }
                            }
                        }
#pragma unroll
                        for (int e = 0; e < C; ++e) g2d[e] = g2[e];
                        if constexpr (S::TO_MASK) {
                            float d[C];
#pragma unroll
                            for (int e = 0; e < C; ++e) d[e] = thr2 - g2[e];
                            tbd = col_sign_bytes<C>(d);
                        }
                        ho2 = ho1;
                        ho1 = ho;
                        ha2 = ha1;
                        ha1 = ha;
                    }
                }
#pragma unroll
                for (int e = 0; e < C; ++e) {
                    b2[e] = b1[e];
                    b1[e] = b[e];
                    ew1[e] = ew[e];
                    sy2[e] = sy1[e];
                    sy1[e] = sy[e];
                }
            }
        }
        if constexpr (KS > 1) {
#pragma unroll
            for (int i = NB - 1; i > 0; --i)
#pragma unroll
                for (int e = 0; e < C; ++e) bh[i][e] = bh[i - 1][e];
#pragma unroll
            for (int e = 0; e < C; ++e) bh[0][e] = h[e];
        }
    };

    // The fill (each stage's first turns), then kTurn turns of the full
    // stage set per loop body: the row rings rotate by renaming.  At a
    // border the last body may run past the tile's rows: such turns re-read
    // its last row and write nothing.
    int t = 0;
#pragma unroll 1
    for (; t < 2 * R; ++t) turn(IC<1>{}, t);
    constexpr int FULL = MODE == TM_BLUR ? 2 : S::NEED_Z ? 4 : 3;
    if constexpr (FULL >= 3) {
#pragma unroll 1
        for (; t < 2 * R + 2; ++t) turn(IC<2>{}, t);
    }
    if constexpr (FULL >= 4) {
#pragma unroll 1
        for (; t < 2 * R + 4; ++t) turn(IC<3>{}, t);
    }
#pragma unroll 1
    for (; t < NS; t += kTurn)
        static_for([&](auto k) {
            if (MODE != TM_BLUR || !BD || t + (int)k < NS) turn(IC<FULL>{}, t + k);
        }, std::make_integer_sequence<int, kTurn>{});
    if constexpr (S::DO_MAX) gmax = __builtin_fmaxf(gmax, ncol > 0 ? gacc : 0.0f);
}

template <int KS, int C, int MODE>
__device__ __forceinline__ void tile_sweep(const ImgArgs& a, const Taps& tp, int x0, int y0,
                                           int ty, float thr2, float& gmax, const lds_float* lds,
                                           SpecTile* sp = nullptr,
                                           const StageOut* so = nullptr) {
    using S = TileShape<KS, C, MODE>;
    const int xs = x0 - S::HL;
    const bool bd = (xs < 0) | (xs + S::SW > a.W) | (y0 - S::HY < 0) | (y0 + ty + S::HY > a.H);
    if (bd)
        tile_body<KS, C, MODE, true>(a, tp, x0, y0, ty, thr2, gmax, lds, sp, so);
    else
        tile_body<KS, C, MODE, false>(a, tp, x0, y0, ty, thr2, gmax, lds, sp, so);
}

}  // namespace hx
