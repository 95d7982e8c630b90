// Epilogue of the tiled projection kernels.
#pragma once
#include <math.h>

#include "swift_device.h"
#include "swift_kernels.h"

namespace swift {

// Values in the grouped layout (kv_vt_index) are written two bytes at a time into 128-byte lines that the
// pass fills only partly, and such a store completes only once the rest of the line has been fetched.  The
// projection kernel therefore touches the lines its epilogue will write while the weights stream: this is where lane
// (block row r, half) of the calling wavefront reads one word, in the line that holds elements 8 g .. 8 g + 7 (+ d/2) of row r's
// slot, or nullptr: rg is no row group of the value part of the fused q|k|v matrix.  The word is never used.
__device__ inline const uint32_t *mv_value_line(const MvArgs &a, int rg, int lane) {
    const int d = a.head_dim, half = d >> 1, lg = __builtin_ctz(half >> 3);  // (16 .. 128: a power of two)
    const int hh = rg >> lg, head = hh - a.n_q_heads - a.n_kv_heads;
    const int r = lane >> 1;
    if (a.nb32 <= 0 || head < 0 || head >= a.n_kv_heads || r >= a.R) return nullptr;
    const int i = 8 * (rg - (hh << lg)) + (lane & 1) * half;
    return (const uint32_t *)((const uint16_t *)a.vcache + (kv_vt_index(head, a.nb32, d, a.pos0 + r, i) & ~(size_t)1));
}
// What follows the dot products of one 16-row group, run by one whole wavefront.
// Y(r, j): finished dot product of block row r and tile row j (before the norm scale).
// rot: optional LDS copy of the rotary rows (k_mv1), [R][d/2] cosines, then sines at mv1_rot_pitch; nullptr = read the tables.
// Several wavefronts may share a row group: wavefront it0 of it_step takes every it_step-th pass of 64 results.
// X: EPI_RESID's residual values, requested ahead of time (mv_residuals), or NoResiduals.
struct NoResiduals {
    static constexpr int N = 0;
};
template <int XN>
struct Residuals {
    static constexpr int N = XN;
    float x[XN], gain;
};
// The residual values that the first XN passes of a wavefront's share of a row group's epilogue add to, and the gain of the lane's row.
template <int XN>
__device__ inline Residuals<XN> mv_residuals(const MvArgs &a, int rg, int lane, int it0 = 0, int it_step = 1) {
    Residuals<XN> X;
    const int row = min(16 * rg + (lane & 15), a.O - 1);
    X.gain = a.gain_next[row];
#pragma unroll
    for (int k = 0; k < XN; ++k) X.x[k] = a.out_f32[(size_t)min(4 * (it0 + k * it_step) + (lane >> 4), a.R - 1) * a.ld_out + row];
    return X;
}
template <int EPI, typename YF, typename XT = NoResiduals>
__device__ inline void mv_epilogue(const MvArgs &a, int rg, int lane, const float *rs, const float *rot, YF Y, int it0 = 0,
                                   int it_step = 1, const XT &X = XT()) {
    const int R = a.R, NT = block_terms(a.RL), NC = NT * layout_rows(a.RL);  // NC: column pitch of the split outputs
    if (EPI == EPI_RESID || EPI == EPI_LOGITS) {
        const int iters = (16 * R + 63) >> 6;
        const int j = lane & 15, row = 16 * rg + j;
        auto pass = [&](int it, float x, float gain) {
            const int r = 4 * it + (lane >> 4);
            const bool ok = r < R && row < a.O;
            if (EPI == EPI_LOGITS) {
                if (ok) a.out_f32[(size_t)r * a.ld_out + row] = Y(r, j) * rs[r];
            } else {
                float xn = 0.f;
                if (ok) {
                    xn = x + Y(r, j);
                    a.out_f32[(size_t)r * a.ld_out + row] = xn;
                    uint16_t hi, mid, lo;
                    split3(xn, gain, hi, mid, lo);
                    uint16_t *p = a.out_s + ((size_t)(row >> 3) * NC + NT * r) * 8 + (row & 7);
                    p[0] = hi;
                    p[8] = mid;
                    if (NT == 3) p[16] = lo;
                }
                const float ss = row_sum_of_squares(xn);
                if (r < R && j == 0) a.pss_out[(size_t)rg * a.rp + r] = ss;
            }
        };
        if constexpr (EPI == EPI_RESID && XT::N > 0) {
#pragma unroll
            for (int k = 0; k < XT::N; ++k)
                if (it0 + k * it_step < iters) pass(it0 + k * it_step, X.x[k], X.gain);
        }
        for (int it = it0 + XT::N * it_step; it < iters; it += it_step) {
            float x = 0.f, gain = 0.f;
            if (EPI == EPI_RESID && row < a.O) {
                x = a.out_f32[(size_t)min(4 * it + (lane >> 4), R - 1) * a.ld_out + row];
                gain = a.gain_next[row];
            }
            pass(it, x, gain);
        }
    } else {
        const int iters = (8 * R + 63) >> 6;
        for (int it = it0; it < iters; it += it_step) {
            const int idx = it * 64 + lane;
            const int r = idx >> 3, j = idx & 7;
            if (r >= R) continue;
            const float sc = rs[r];
            const float ya = Y(r, j) * sc, yb = Y(r, j + 8) * sc;
            if (EPI == EPI_SWIGLU) {
                if (2 * (8 * rg + j) < a.O) {
                    uint16_t hi, mid, lo;
                    split3(ya / (1.0f + expf(-ya)), yb, hi, mid, lo);
                    uint16_t *p = a.out_s + ((size_t)rg * NC + NT * r) * 8 + j;
                    p[0] = hi;
                    p[8] = mid;
                    if (NT == 3) p[16] = lo;
                }
            } else {
                const int d = a.head_dim, half = d >> 1, lg = __builtin_ctz(half >> 3);
                const int hh = rg >> lg, i = 8 * (rg - (hh << lg)) + j;
                const int nq = a.n_q_heads, nkv = a.n_kv_heads, pos = a.pos0 + r, rpos = mv_rope_pos(a, r);
                if (hh < nq + nkv) {
                    const float c = rot ? rot[r * half + i] : a.cos_tab[(size_t)rpos * half + i];
                    const float s = rot ? rot[((R * half + 63) & ~63) + r * half + i] : a.sin_tab[(size_t)rpos * half + i];
                    const float qa = ya * c - yb * s, qb = yb * c + ya * s;
                    if (hh < nq) {
                        float *qp = a.out_f32 + (size_t)r * a.ld_out + hh * d + i;
                        qp[0] = qa;
                        qp[half] = qb;
                        if (a.q_s) {
                            uint16_t *qs = a.q_s + ((size_t)(r * nq + hh) * 2) * d + i;
                            const uint32_t ha = f32_to_bf16_rne_finite(qa), hb = f32_to_bf16_rne_finite(qb);
                            qs[0] = (uint16_t)ha;
                            qs[half] = (uint16_t)hb;
                            qs[d] = (uint16_t)f32_to_bf16_rne_finite(qa - __uint_as_float(ha << 16));
                            qs[d + half] = (uint16_t)f32_to_bf16_rne_finite(qb - __uint_as_float(hb << 16));
                        }
                    } else {
                        uint16_t *kc = (uint16_t *)a.kcache + ((size_t)(hh - nq) * a.max_seq + pos) * d + i;
                        kc[0] = f32_to_bf16_rne(qa);
                        kc[half] = f32_to_bf16_rne(qb);
                    }
                } else if (a.nb32 > 0) {  // values in groups of eight slots
                    uint16_t *vc = (uint16_t *)a.vcache + kv_vt_index(hh - nq - nkv, a.nb32, d, pos, i);
                    vc[0] = f32_to_bf16_rne(ya);
                    vc[half * 8] = f32_to_bf16_rne(yb);
                } else {
                    uint16_t *vc = (uint16_t *)a.vcache + ((size_t)(hh - nq - nkv) * a.max_seq + pos) * d + i;
                    vc[0] = f32_to_bf16_rne(ya);
                    vc[half] = f32_to_bf16_rne(yb);
                }
            }
        }
    }
}

}  // namespace swift
