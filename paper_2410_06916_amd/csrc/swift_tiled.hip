// gfx950 kernels of the bf16 path: tiled weights streamed once from HBM into MFMA, activations
// kept in fp32 precision as three bf16 terms (two in blocks of more than 16 rows).  k_mv1 handles blocks of 1-5 activation rows whose
// activation fits in LDS (draft pass, plain decoding, short verify blocks), k_mvR and k_mvN blocks of up to
// 32 and 64 rows (longer verify blocks, prefill, candidate evaluation).
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "swift_device.h"
#include "swift_kernels.h"
#include "swift_mv.h"

namespace swift {

// Events for the next projection launch (see set_launch_events in swift_kernels.h).
static thread_local hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;
void set_launch_events(hipEvent_t start, hipEvent_t stop) {
    g_ev_start = start;
    g_ev_stop = stop;
}
template <typename K, typename... Args>
static hipError_t launch_maybe_timed(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, Args... args) {
    if (g_ev_start) {
        hipEvent_t a = g_ev_start, b = g_ev_stop;
        g_ev_start = g_ev_stop = nullptr;
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, s, a, b, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// weight layout conversion
// ------------------------------------------------------------------------------------------
__global__ void k_tile_weights(TileArgs a) {
    // one thread per 16-byte chunk of the destination
    const int64_t n_chunks = (int64_t)a.n_rg * a.T * 64;
    const uint16_t *src = (const uint16_t *)a.src;
    u32x4 *dst = (u32x4 *)a.dst;
    const int d = a.head_dim, half = d >> 1, gph = half >> 3;  // row groups per head (TILE_PAIR)
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n_chunks;
         c += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(c & 63);
        const int64_t tile = c >> 6;
        const int t = (int)(tile % a.T);
        const int rg = (int)(tile / a.T);
        const int j = l & 15, k0 = 32 * t + 8 * (l >> 4);
        int row;
        if (a.mode == TILE_PLAIN) {
            row = 16 * rg + j;
        } else if (a.mode == TILE_PAIR) {
            const int head = rg / gph, g = rg - head * gph;
            row = head * d + 8 * g + (j & 7) + (j >= 8 ? half : 0);
        } else {
            if ((j >= 8) != (a.part == 1)) continue;  // the other half of the tile comes from the other tensor
            row = 8 * rg + (j & 7);
        }
        u32x4 v = {0u, 0u, 0u, 0u};
        if (row < a.src_rows) {
            if (k0 + 8 <= a.K) {
                v = *(const u32x4 *)(src + (size_t)row * a.K + k0);
            } else {
                uint16_t e[8];
                for (int i = 0; i < 8; ++i) e[i] = (k0 + i < a.K) ? src[(size_t)row * a.K + k0 + i] : (uint16_t)0;
                v.x = e[0] | ((uint32_t)e[1] << 16);
                v.y = e[2] | ((uint32_t)e[3] << 16);
                v.z = e[4] | ((uint32_t)e[5] << 16);
                v.w = e[6] | ((uint32_t)e[7] << 16);
            }
        }
        dst[c] = v;
    }
}

hipError_t launch_tile_weights(const TileArgs &a, hipStream_t s) {
    const int64_t n_chunks = (int64_t)a.n_rg * a.T * 64;
    if (n_chunks <= 0) return hipSuccess;
    int64_t grid = (n_chunks + 255) / 256;
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(k_tile_weights, dim3((unsigned)grid), dim3(256), 0, s, a);
    return hipGetLastError();
}


// ------------------------------------------------------------------------------------------
// embedding gather for R rows: fp32 residual, split of x * gain_next, partial sums of squares
// ------------------------------------------------------------------------------------------
// One thread per row and eight elements (16 bytes in, 32 + 16 per term out); the two threads of a 16-element group add its
// squares.  A prompt's macro block is one launch for every 512 rows, as many token ids as the launch arguments carry (512 rows
// of 4096: 9.9 us, against 33 as eight launches of 64 rows with a thread per element).
template <int N>
struct EmbedTokens {
    int32_t id[N];
};
template <int N>
__global__ __launch_bounds__(256) void k_embed_rows(EmbedRowsArgs a, EmbedTokens<N> tok) {
    const int NT = block_terms(a.RL), NC = NT * layout_rows(a.RL);
    const int cpr = ((a.H + 15) >> 4) * 2;  // 8-element chunks of a row (whole 16-element groups)
    const int total = a.R * cpr, idx = blockIdx.x * 256 + threadIdx.x;
    const int r = min(idx, total - 1) / cpr, c = min(idx, total - 1) - r * cpr;
    const int sub = r >> 6, rs = N > kMaxBlockRows ? r & 63 : r;  // sub-block, row of it
    const bool ok = idx < total && 8 * c < a.H;                   // (H is a multiple of 8)
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.f;
    if (ok) {
        const int id = a.feed ? min(max(a.feed[0], 0), a.V - 1) : tok.id[r];
        const u32x4 e = *(const u32x4 *)(a.E + (size_t)id * a.H + 8 * c);
        const f32x4 g0 = *(const f32x4 *)(a.gain_next + 8 * c), g1 = *(const f32x4 *)(a.gain_next + 8 * c + 4);
        float *x = a.x + sub * a.sub_x + (size_t)rs * a.H + 8 * c;
        u32x4 t[3];
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            v[i] = __uint_as_float(e[i >> 1] << 16);
            v[i + 1] = __uint_as_float(e[i >> 1] & 0xffff0000u);
            uint16_t h[2], m[2], l[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) split3(v[i + j] * (i < 4 ? g0[i + j & 3] : g1[i + j & 3]), h[j], m[j], l[j]);
            t[0][i >> 1] = pack2(h[0], h[1]);
            t[1][i >> 1] = pack2(m[0], m[1]);
            t[2][i >> 1] = pack2(l[0], l[1]);
        }
        *(f32x4 *)x = f32x4{v[0], v[1], v[2], v[3]};
        *(f32x4 *)(x + 4) = f32x4{v[4], v[5], v[6], v[7]};
        u32x4 *p = (u32x4 *)(a.xs + sub * a.sub_xs) + (size_t)c * NC + NT * rs;
        p[0] = t[0];
        p[1] = t[1];
        if (NT == 3) p[2] = t[2];
    }
    float q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = v[i] * v[i];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] += __shfl_xor(q[i], 1, 64);
    const float ss = ((q[0] + q[4]) + (q[2] + q[6])) + ((q[1] + q[5]) + (q[3] + q[7]));
    if (idx < total && (c & 1) == 0) a.pss[sub * a.sub_pss + (size_t)(c >> 1) * a.rp + rs] = ss;
}

template <int N>
static hipError_t launch_embed_rows_n(const EmbedRowsArgs &a, const int32_t *tokens, hipStream_t s) {
    EmbedTokens<N> tok;
    memcpy(tok.id, tokens, sizeof(int32_t) * a.R);
    const int grid = (a.R * ((a.H + 15) / 16 * 2) + 255) / 256;
    hipLaunchKernelGGL(k_embed_rows<N>, dim3(grid), dim3(256), 0, s, a, tok);
    return hipGetLastError();
}

hipError_t launch_embed_rows(const EmbedRowsArgs &a, const int32_t *tokens, hipStream_t s) {
    if (a.R < 1 || (a.H & 7) != 0 || (a.feed && a.R != 1)) return hipErrorInvalidValue;
    if (a.R <= kMaxBlockRows) return launch_embed_rows_n<kMaxBlockRows>(a, tokens, s);
    for (int r0 = 0; r0 < a.R; r0 += kEmbedRows) {
        EmbedRowsArgs b = a;
        const int sub = r0 / kMaxBlockRows;
        b.R = std::min(kEmbedRows, a.R - r0);
        b.x += sub * a.sub_x;
        b.xs += sub * a.sub_xs;
        b.pss += sub * a.sub_pss;
        const hipError_t e = launch_embed_rows_n<kEmbedRows>(b, tokens + r0, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------
// shared pieces of the projection kernels
// ------------------------------------------------------------------------------------------
// RMSNorm scale per block row from the producer's partial sums of squares [n_pss][16].  All 512
// threads load (thread = (partial p mod 32, row r)); mv_norm_load issues the first eight loads per
// thread (enough for 256 partials, hidden <= 4096) so that the caller can put them ahead of the
// weight loads; mv_norm_finish adds the rest, then 16 threads add the 32 per-lane sums in order:
// the summation order is fixed.  One barrier, before the final sums.  (Full barriers: LDS-only ones, which would leave the
// caller's first weight loads in flight, measured 0.3 us slower per launch.)
struct NormPart {
    float v[8];
};
__device__ inline NormPart mv_norm_load(const MvArgs &a) {
    NormPart np;
    const int tid = threadIdx.x, r = tid & 15, q = tid >> 4;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int p = q + 32 * u;
        np.v[u] = (a.pss && p < a.n_pss) ? a.pss[(size_t)p * a.rp + r] : 0.f;
    }
    return np;
}
template <bool LDS_ONLY = false>
__device__ inline void mv_norm_finish(const MvArgs &a, const NormPart &np, float *rs /* LDS [16] */,
                                      float *scratch /* LDS [512] */) {
    const int tid = threadIdx.x, r = tid & 15, q = tid >> 4;
    if (a.pss) {
        float ss = 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) ss += np.v[u];
        for (int p0 = 256; p0 < a.n_pss; p0 += 256) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int p = p0 + q + 32 * u;
                v[u] = p < a.n_pss ? a.pss[(size_t)p * a.rp + r] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) ss += v[u];
        }
        scratch[q * 16 + r] = ss;
    }
    if (LDS_ONLY)
        lds_barrier();
    else
        __syncthreads();
    if (tid < 16) {
        float ss = 0.f;
        if (a.pss)
            for (int q2 = 0; q2 < 32; ++q2) ss += scratch[q2 * 16 + tid];
        rs[tid] = a.pss ? 1.0f / sqrtf(ss / (float)a.norm_dim + a.eps) : 1.0f;
    }
    // (no barrier here: the scales are read by the epilogue only, and every caller has a barrier between
    // this point and its epilogue)
}

// The same for exact layouts of 17..32 rows (row pitch 64), in the summation order of mv_norm_load /
// mv_norm_finish -- a row's scale must not depend on the rows it shares a pass with: thread (row r, q) adds
// the partials q + 32 u and q + 16 + 32 u, u = 0, 1, .., as two sums; then 32 threads add the 32 sums in
// order.  In two parts: the loads of the first 256 partials (hidden <= 4096: all of them), and the rest with an
// LDS-only barrier.
struct NormPart32 {
    float v[2][8];
};
__device__ inline void mv_norm32_load(const MvArgs &a, int p0, NormPart32 &np) {
    const int tid = threadIdx.x, r = tid & 31, q0 = tid >> 5;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = p0 + q0 + 16 * half + 32 * u;
            np.v[half][u] = (a.pss && p < a.n_pss) ? a.pss[(size_t)p * a.rp + r] : 0.f;
        }
}
__device__ inline void mv_norm32_finish(const MvArgs &a, NormPart32 &np, float *rs /* LDS [32] */, float *scratch /* LDS [1024] */) {
    const int tid = threadIdx.x, r = tid & 31, q0 = tid >> 5;
    float ss[2] = {0.f, 0.f};
    for (int p0 = 0;;) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float t = 0.f;
            if (p0 == 0) {
#pragma unroll
                for (int u = 0; u < 8; ++u) t += np.v[half][u];
                ss[half] = t;
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) ss[half] += np.v[half][u];
            }
        }
        p0 += 256;
        if (p0 >= a.n_pss) break;
        mv_norm32_load(a, p0, np);
    }
    scratch[q0 * 32 + r] = ss[0];
    scratch[(q0 + 16) * 32 + r] = ss[1];
    lds_barrier();
    if (tid < 32) {
        float t = 0.f;
        for (int q2 = 0; q2 < 32; ++q2) t += scratch[q2 * 32 + tid];
        rs[tid] = a.pss ? 1.0f / sqrtf(t / (float)a.norm_dim + a.eps) : 1.0f;
    }
}

// The same for bulk layouts of 64 rows: thread = (partial p mod 8, row r), then 64 threads add the 8 per-thread sums in order.
struct NormPart64 {
    float v[32];
};
__device__ inline void mv_norm64_load(const MvArgs &a, int p0, NormPart64 &np) {
    const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
        const int p = p0 + q + 8 * u;
        np.v[u] = (a.pss && p < a.n_pss) ? a.pss[(size_t)p * a.rp + r] : 0.f;
    }
}
__device__ inline void mv_norm64_finish(const MvArgs &a, NormPart64 &np, float *rs /* LDS [64] */, float *scratch /* LDS [512] */) {
    const int tid = threadIdx.x, r = tid & 63, q = tid >> 6;
    float ss = 0.f;
    for (int p0 = 0;;) {
#pragma unroll
        for (int u = 0; u < 32; ++u) ss += np.v[u];
        p0 += 256;
        if (p0 >= a.n_pss) break;
        mv_norm64_load(a, p0, np);
    }
    scratch[q * 64 + r] = ss;
    lds_barrier();
    if (tid < 64) {
        float t = 0.f;
        for (int q2 = 0; q2 < 8; ++q2) t += scratch[q2 * 64 + tid];
        rs[tid] = a.pss ? 1.0f / sqrtf(t / (float)a.norm_dim + a.eps) : 1.0f;
    }
}

// Slices (of the 8 K slices of a row group) whose sums are added first, in slice order, before the
// group sums are added in group order: 8, 4, 2 or 1.  It is the number of slices one workgroup of
// the block kernel covers when that kernel splits K over workgroups to fill the chip, and it
// depends on the matrix (and the device) only, so that every kernel adds a row's slice sums in the
// same order whatever the number of rows in the pass.
static int mv_slice_group(const MvArgs &a, int n_cu) {
    const int n_rb = (a.n_rg + 7) / 8;
    int ksp = n_cu / n_rb;
    if (ksp < 1) ksp = 1;
    if (ksp > 8) ksp = 8;
    int p2 = 1;
    while (p2 * 2 <= ksp) p2 *= 2;
    ksp = p2;
    const int n_c = (a.T + 7) / 8;
    // (a workgroup's K range holds at least 8 tiles; the partial sums fit the scratch)
    while (ksp > 1 && (n_c * (8 / ksp) < 8 || (int64_t)ksp * a.n_rg > a.part_capacity)) ksp /= 2;
    return 8 / ksp;
}

// ------------------------------------------------------------------------------------------
// 1..5 activation rows: Y = W . X, MFMA, whole activation in LDS, K split over wavefronts
// ------------------------------------------------------------------------------------------
// The NC = 3R term columns of X (R <= 5, so NC <= 15) fit one MFMA column block; lanes of columns
// >= NC read a zero chunk.  A workgroup has 8 wavefronts; KS of them share one 16-row group of W,
// each taking a contiguous slice of its k-tiles, so a workgroup works on G = 8/KS row groups at a
// time and the slices (and the three terms) are added in LDS in a fixed order.  Every wavefront
// keeps a rolling window of NS (10..16) 1 KB tile loads in flight, walked in blocks of NS slots (the
// launcher picks the depth that cuts the slice with the fewest unused slots); the first window is
// issued before the activation is staged, and the window rolls on from one round into the next.
template <int EPI, int KS, int NS>
__global__ __launch_bounds__(512, 4) void k_mv1(MvArgs a) {  // 4 wavefronts per SIMD: <= 128 VGPRs, two workgroups per CU
    extern __shared__ __align__(16) unsigned char smem[];
    const int R = a.R, NC = 3 * R;
    // LDS: [16 B zeros][4T chunks x NC x 8 bf16][2 x 8 wavefronts x NC x 16 fp32][16 scales][512 scratch][R x d rotary]
    float *red = (float *)(smem + 16 + (size_t)a.T * 64 * NC);
    float *rs = red + 2 * 8 * 16 * NC;
    float *nscratch = rs + 16;
    float *rot = nscratch + 512;  // per block row: [d/2 cos | d/2 sin] at that row's position
    constexpr int G = 8 / KS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform from here on
    const int g = wave / KS, ks = wave - g * KS;
    const int T = a.T;
    const int n = (T + KS - 1) / KS;           // k-tiles per wavefront and row group
    const int t0 = min(ks * n, T - 1);
    const int nv = max(0, min(n, T - ks * n)); // ... of which exist
    const int nvm1 = max(nv - 1, 0);
    const u32x4 *Wt = (const u32x4 *)a.Wt;
    const int W = a.n_wg;
    if (EPI == EPI_QKV && (int)blockIdx.x >= W) {
        // Cache warm-up for the attention launch that follows: warm-up workgroup p reads the committed keys
        // and values of the kv heads congruent to p.  Workgroups go to the dies round-robin by index, and the
        // attention kernel's workgroup for head g has index g (+ a multiple of 8 per further row), so with
        // pf_first and the number of warm-up workgroups multiples of 8 the lines land in the L2
        // that kernel's loads will ask.  No result; no barrier.
        // (pf_wgs warm-up workgroups, a multiple of 8: workgroup p takes the heads congruent to p modulo pf_wgs)
        const int p = (int)blockIdx.x - a.pf_first;
        if (p < 0) return;
        const size_t head_units = (size_t)a.max_seq * a.head_dim / 8;  // 16-byte units of one head
        const int n_units = a.pf_rows * a.head_dim / 8;
        // (values in groups of eight slots: the groups that hold rows [0, pf_rows) are contiguous too)
        const size_t v_head_units = a.nb32 > 0 ? (size_t)a.nb32 * 32 * a.head_dim / 8 : head_units;
        const int v_units = a.nb32 > 0 ? (a.pf_rows + 31) / 32 * 32 * a.head_dim / 8 : n_units;
        u32x4 x = {0u, 0u, 0u, 0u};
        for (int gh = p; gh < a.pf_heads; gh += a.pf_wgs) {
            const u32x4 *kp = (const u32x4 *)a.kcache + (size_t)gh * head_units;
            const u32x4 *vp = (const u32x4 *)a.vcache + (size_t)gh * v_head_units;
            // (eight steps' loads requested together: one step at a time, the loop is a chain of memory latencies)
            for (int i0 = tid; i0 < v_units; i0 += 8 * 512) {  // (v_units >= n_units)
                u32x4 t[16];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = i0 + 512 * u;
                    t[2 * u] = i < n_units ? kp[i] : u32x4{0u, 0u, 0u, 0u};  // (plain loads: the lines are meant to stay in L2)
                    t[2 * u + 1] = i < v_units ? vp[i] : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int u = 0; u < 16; ++u) x ^= t[u];
            }
        }
        // (keeps the loads alive; the flag word is never all ones)
        if ((x.x & x.y & x.z & x.w) == 0xffffffffu && a.pf_rows < 0) ((volatile uint32_t *)smem)[0] = x.x;
        return;
    }
    const int last_rg = a.n_rg - 1;
    const int col = lane & 15, kg = lane >> 4;
    // byte address of this lane's B chunk for tile t: boff + t * bstride; lanes of columns >= NC
    // (and slots past the wavefront's slice) read the zero chunk at address 0
    const int boff = col < NC ? 16 + (kg * NC + col) * 16 : 0;
    const int bstride = col < NC ? 64 * NC : 0;

    u32x4 buf[NS];
    const u32x4 *base = nullptr;
    auto load_slot = [&](int i) { return __builtin_nontemporal_load(base + (size_t)min(i, nvm1) * 64); };
    auto mma_slot = [&](int i, const u32x4 &av, f32x4 &acc, int live_mask) {
        const int m = (i < nv) ? live_mask : 0;              // all ones or zero, wavefront-uniform
        const int addr = (boff + (t0 + i) * bstride) & m;
        const u32x4 bv = *(const u32x4 *)(smem + addr);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                      acc, 0, 0, 0);
    };
    auto prime = [&](int seg) {
        const int rg = min((seg * W + (int)blockIdx.x) * G + g, last_rg);
        base = Wt + ((size_t)rg * T + t0) * 64 + lane;
#pragma unroll
        for (int u = 0; u < NS; ++u) buf[u] = load_slot(u);
    };

    // ---- stage the split activation (a plain copy: the producer kernel already wrote it in B
    // layout).  Its loads, and those of the norm partials, go out ahead of the weight loads so
    // that they return first; the first weight window is in flight while LDS is filled.
    {
        const u32x4 *src = (const u32x4 *)a.in_s;
        u32x4 *dst = (u32x4 *)(smem + 16);
        const int n_units = T * 4 * NC, real_units = (a.K >> 3) * NC;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        // The residual projections read their norm partials ahead of the weight window and wait for them
        // with an LDS-only barrier, so that the MFMAs start on the first tiles while the rest of the window
        // is still on its way (o_proj 10.7 -> 10.4 us, down_proj 19.0 -> 18.2 us); the other epilogues measured
        // slower that way (q|k|v by 2.7 us) and keep the full barrier.
        constexpr bool kEarlyNorm = EPI == EPI_RESID;
        NormPart np;
        auto side_loads = [&]() {
            if (tid < 4) ((uint32_t *)smem)[tid] = 0u;
            if (EPI == EPI_QKV) {
                // the lines the epilogues of this workgroup's rounds will write values into (wavefront s: round s)
                if (wave < a.S)
                    for (int gg = 0; gg < G; ++gg) mv_touch_value_lines(a, min((wave * W + (int)blockIdx.x) * G + gg, last_rg), lane);
                const int d = a.head_dim, half = d >> 1;
                for (int i = tid; i < R * half; i += 512) {
                    const int r = i / half, e = i - r * half;
                    rot[r * d + e] = a.cos_tab[(size_t)mv_rope_pos(a, r) * half + e];
                    rot[r * d + half + e] = a.sin_tab[(size_t)mv_rope_pos(a, r) * half + e];
                }
            }
        };
        if (n_units <= 4 * 512) {  // depth <= 5461 for one row: four loads per thread cover it
            u32x4 tmp[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = tid + 512 * q;
                tmp[q] = i < real_units ? src[i] : zero;
            }
            if (kEarlyNorm) np = mv_norm_load(a);
            prime(0);
            side_loads();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = tid + 512 * q;
                if (i < n_units) dst[i] = tmp[q];
            }
        } else {
            u32x4 tmp[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int i = tid + 512 * q;
                tmp[q] = i < real_units ? src[i] : zero;
            }
            if (kEarlyNorm) np = mv_norm_load(a);
            prime(0);
            side_loads();
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const int i = tid + 512 * q;
                if (i < n_units) dst[i] = tmp[q];
            }
            for (int i0 = 9 * 512; i0 < n_units; i0 += 4 * 512) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + tid + 512 * q;
                    tmp[q] = i < real_units ? src[i] : zero;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int i = i0 + tid + 512 * q;
                    if (i < n_units) dst[i] = tmp[q];
                }
            }
        }
        if (!kEarlyNorm) np = mv_norm_load(a);
        mv_norm_finish<kEarlyNorm>(a, np, rs, nscratch);
    }

    for (int seg = 0; seg < a.S; ++seg) {
        const int rg = (seg * W + (int)blockIdx.x) * G + g;
        const bool live = rg <= last_rg;
        const int live_mask = live ? -1 : 0;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};

        const int nb16 = (n + NS - 1) / NS;
        // (As compiled, the NS reloads of a block go out together behind its last MFMA.  Pinning each
        // reload behind the MFMA that frees its slot with scheduling barriers measured the same.)
        for (int b = 0; b + 1 < nb16; ++b) {
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_slot(b * NS + u, buf[u], acc, live_mask);
                buf[u] = load_slot((b + 1) * NS + u);
            }
        }
        if (seg + 1 < a.S) {
            // the window rolls on into the next round's row group: the stream never drains
            const int rgn = min(((seg + 1) * W + (int)blockIdx.x) * G + g, last_rg);
            base = Wt + ((size_t)rgn * T + t0) * 64 + lane;
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_slot((nb16 - 1) * NS + u, buf[u], acc, live_mask);
                buf[u] = load_slot(u);
            }
        } else {
#pragma unroll
            for (int u = 0; u < NS; ++u) mma_slot((nb16 - 1) * NS + u, buf[u], acc, live_mask);
        }

        // ---- end of the row group: every wavefront parks its NC result columns in LDS; one
        // wavefront per row group adds terms and K slices and runs the epilogue
        float *rp = red + (size_t)(seg & 1) * (8 * 16 * NC);
        if (col < NC) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) rp[(wave * NC + col) * 16 + 4 * kg + r4] = acc[r4];
        }
        lds_barrier();  // (the next round's tile loads stay in flight)
        if (!live || ks != 0) continue;
        mv_epilogue<EPI>(a, rg, lane, rs, EPI == EPI_QKV ? rot : nullptr, [&](int r, int j) {
            // Slice sums are added per term in groups of kgroup slices (slice order), the three
            // terms of a group are combined, and the groups are added in order.  (Rolled loops: this
            // runs in one wavefront per row group while the load window stays in registers.)
            const int kgroup = a.kgroup;
            const float *w = rp + (g * KS * NC + 3 * r) * 16 + j;
            const int ss = NC * 16;  // from one slice to the next
            float y = 0.f;
#pragma unroll 1
            for (int k0 = 0; k0 < KS; k0 += kgroup) {
                float hi = w[0], mid = w[16], lo = w[32];
                w += ss;
#pragma unroll 1
                for (int k2 = 1; k2 < kgroup; ++k2) {
                    hi += w[0];
                    mid += w[16];
                    lo += w[32];
                    w += ss;
                }
                const float gs = (hi + mid) + lo;
                y = k0 == 0 ? gs : y + gs;
            }
            return y;
        });
    }
}

template <int EPI, int KS, int NS>
static hipError_t launch_mv1_t(const MvArgs &a, int grid, size_t lds, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_mv1<EPI, KS, NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kMvMaxLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    return launch_maybe_timed(k_mv1<EPI, KS, NS>, dim3(grid), dim3(512), lds, s, a);
}

static hipError_t launch_mv1(int epi, MvArgs a, int n_cu, int ks_override, int wg_override, hipStream_t s) {
    const size_t lds = mv1_lds_bytes(a.K, a.R, a.head_dim);
    if (lds > kMvMaxLds) return hipErrorInvalidValue;
    // Work split: KS wavefronts per row group, W workgroups, S rounds, chosen so that every
    // workgroup gets the same number of row groups (a weight stream is only as fast as its
    // slowest wavefront) with at most 16 wavefronts per compute unit.
    int occ = (int)((160 * 1024) / (lds + 512));
    if (occ > 2) occ = 2;
    if (occ < 1) occ = 1;
    const int max_wg = n_cu * occ;
    int best_ks = 8, best_w = 1, best_s = 1;
    double best_score = 1e30;
    // Always 8 K slices per row group (unless a tuning run overrides it): the slice boundaries and
    // the order in which slice sums are added define a row's result bit for bit, and the block kernel
    // for 6-16 rows uses the same ones, so that a token's logits do not depend on how many rows
    // share its pass (speculative output == plain greedy output exactly, not just up to rounding).
    for (int ks = 8; ks >= 1; ks /= 2) {
        if (ks != (ks_override ? ks_override : 8)) continue;
        const int G = 8 / ks;
        for (int S = 1; S <= 64; ++S) {
            int W = (a.n_rg + G * S - 1) / (G * S);
            if (W > max_wg) continue;
            const double waste = (double)W * G * S / a.n_rg;           // >= 1
            const double fill = (double)W / max_wg;                     // fraction of resident slots used
            const double score = waste + (fill < 0.5 ? (0.5 - fill) : 0.0) + 0.002 * S + 0.01 * (8 / ks - 1);
            if (score < best_score) {
                best_score = score;
                best_ks = ks;
                best_w = W;
                best_s = S;
            }
        }
    }
    if (wg_override > 0) {
        const int G = 8 / best_ks;
        best_w = wg_override;
        best_s = (a.n_rg + G * best_w - 1) / (G * best_w);
    }
    a.S = best_s;
    a.n_wg = best_w;
    int grid = best_w;
    // (the warm-up workgroups only pay while they run beside the projection: they take free slots only)
    a.pf_first = (best_w + 7) / 8 * 8;
    a.pf_wgs = std::min((max_wg - a.pf_first) / 8 * 8, (a.pf_heads + 7) / 8 * 8);
    // Only with one workgroup per head, the compute units clearly under-filled (measured with 480 of 512 slots
    // taken: the extra workgroups slow the projection down by more than the attention gains), and a context
    // short enough for a workgroup to read its whole head well before the projection ends: one compute unit
    // takes in about 37 GB/s and the weights stream at about 5 TB/s, so a head may hold 0.6 of what can be
    // read in that time (7B shape: up to about 860 slots; warming only part of a longer head measured worse
    // than not warming at all).
    const double t_us = (double)a.n_rg * a.T * 1024.0 / 5.0e6;
    const double head_bytes = (double)a.pf_rows * a.head_dim * 4.0;  // keys and values, bf16
    if (epi == EPI_QKV && a.pf_heads > 0 && a.pf_rows > 0 && a.pf_wgs >= a.pf_heads &&
        a.pf_first + a.pf_wgs <= max_wg * 85 / 100 && head_bytes <= 0.6 * 37.0e3 * t_us) {
        grid = a.pf_first + a.pf_wgs;
    } else {
        a.pf_heads = 0;
        a.pf_wgs = 0;
    }
    a.kgroup = best_ks == 8 ? mv_slice_group(a, n_cu) : best_ks;
    // Slots per block of the load window (= loads in flight per wavefront): 16 unless another depth
    // cuts a slice of n tiles with fewer wasted slots (n = 43: 3 x 15 instead of 3 x 16; n = 20:
    // 2 x 10 instead of 2 x 16).  Only for the 8-way split, which is what the big shapes use.
    int ns = 16;
    if (best_ks == 8) {
        const int n = (a.T + 7) / 8;
        int best_waste = (n + 15) / 16 * 16 - n;
        for (int c = 15; c >= 10; --c) {
            const int waste = (n + c - 1) / c * c - n;
            if (waste < best_waste && (n + c - 1) / c <= (n + 15) / 16 + 1) {
                best_waste = waste;
                ns = c;
            }
        }
    }
#define SWIFT_MV_CASE(E)                                                                   \
    case E:                                                                                \
        switch (best_ks) {                                                                 \
            case 1: return launch_mv1_t<E, 1, 16>(a, grid, lds, s);                      \
            case 2: return launch_mv1_t<E, 2, 16>(a, grid, lds, s);                      \
            case 4: return launch_mv1_t<E, 4, 16>(a, grid, lds, s);                      \
            default:                                                                       \
                switch (ns) {                                                              \
                    case 10: return launch_mv1_t<E, 8, 10>(a, grid, lds, s);             \
                    case 11: return launch_mv1_t<E, 8, 11>(a, grid, lds, s);             \
                    case 12: return launch_mv1_t<E, 8, 12>(a, grid, lds, s);             \
                    case 13: return launch_mv1_t<E, 8, 13>(a, grid, lds, s);             \
                    case 14: return launch_mv1_t<E, 8, 14>(a, grid, lds, s);             \
                    case 15: return launch_mv1_t<E, 8, 15>(a, grid, lds, s);             \
                    default: return launch_mv1_t<E, 8, 16>(a, grid, lds, s);             \
                }                                                                          \
        }
    switch (epi) {
        SWIFT_MV_CASE(EPI_QKV)
        SWIFT_MV_CASE(EPI_RESID)
        SWIFT_MV_CASE(EPI_SWIGLU)
        SWIFT_MV_CASE(EPI_LOGITS)
    }
#undef SWIFT_MV_CASE
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------------
// a block of up to 64 activation rows: Y = W . X, MFMA, both operands through a ring in LDS, optional split-K
// ------------------------------------------------------------------------------------------
// A workgroup of 8 wavefronts owns 2 WM row groups of W (WM = 4 or 3) and all columns.  Wavefront (w % WM, w / WM), w < 2 WM,
// multiplies two row groups with half of the column blocks, NCW = ceil(NCB / 2) of them.  Weight tiles and the B operand reach LDS
// straight from global memory through a ring of stages of two k tiles each, all eight wavefronts copying; in step t the
// operands of stage t + 1 are read, stage t is multiplied, and what lies further ahead (about 140 KB) is on its way.  One barrier
// per stage.
// What bounds it: the weight stream, and the operand reads (a wavefront reads 2 + NCW KB per k tile; as one row group
// times all columns, which is what this kernel replaces, 1 + NCB KB from chunks of eight tiles that drained the loads in
// flight at every barrier).  Weights are copied non-temporally, so that they do not push the B operand, which every workgroup
// reads, out of L2.  us, before / now, launches back to back: 7B, 31 rows gate/up 54 / 40, down_proj 35.5 / 28 (30 in a pass), LM head 60 / 48; 32 bulk rows gate/up
// 40.5 / 34; 13B, 31 rows gate/up 79 / 57, down_proj 57 / 39; 70B, 31 rows gate/up 231 / 179, LM head 112 / 86.  (One k tile a
// stage 1-3 % slower; weights straight to registers, each tile by two wavefronts: gate/up 54; four wavefronts of 512 registers
// with six row groups each and nothing staged: 62.)
//
// With gridDim.y > 1 the K range is split over workgroups: each wavefront writes the partial results of one row group, and the
// one that arrives last at the row group's counter adds the partials in split order (so the result does
// not depend on arrival order) and runs the epilogue.
//
// CANON (exact layouts: verify blocks of up to 32 rows, 2-6 column blocks; mvn_canon) reproduces the LDS-resident kernel
// bit for bit: the K range of a row group is cut into the same 8 slices of ceil(T/8) tiles, a slice is
// accumulated from zero tile by tile, a workgroup covers a group of 8, 4, 2 or 1 whole slices (mv_slice_group: a
// function of the matrix alone, not of the row count) and adds their sums per term in slice order, combines
// the three terms, and the last workgroup adds the group results in order.  The LDS-resident kernel adds its 8
// slice sums in the same grouping.  The bulk variants (NCB = 4 / 8: layouts of 32 / 64 rows, two-term columns)
// keep their own fixed order.
constexpr int kMvnRing = 144 * 1024;
constexpr int kMvnTiles = 2;       // k tiles of a stage
constexpr int kNonTemporal = 2;    // cache policies: nt; sc1
constexpr int kDeviceScope = 16;
// How k_mvN cuts a matrix over workgroups: grid (row blocks, K parts), tiles per part, row groups per workgroup, six or eight:
// what takes fewer rounds x tiles x cost of a tile, which is about that of (row groups + 20) (7B gate/up, 31 rows, one round
// either way: 40.3 us with six, 42.9 with eight; 13B gate/up, two rounds with six: 88 against 57).
struct MvnPlan {
    int grid_x, ksp, TS, rgs;
};
static MvnPlan mvn_plan(const MvArgs &a, int n_cu, bool canon) {
    MvnPlan best{};
    int64_t least = 0;
    for (int rgs = 6; rgs <= 8; rgs += 2) {
        MvnPlan p;
        p.rgs = rgs;
        p.grid_x = (a.n_rg + rgs - 1) / rgs;
        if (canon) {
            p.TS = ((a.T + 7) / 8) * mv_slice_group(a, n_cu);
        } else {
            // about one workgroup of eight row groups per compute unit, eight tiles each at least (whatever the workgroup's
            // own row groups: the parts are the order of the sums)
            int ksp = std::min(8, std::max(1, n_cu / ((a.n_rg + 7) / 8)));
            while (ksp > 1 && ((a.T + ksp - 1) / ksp < 8 || (int64_t)a.n_rg * ksp > a.part_capacity)) --ksp;
            p.TS = (a.T + ksp - 1) / ksp;
        }
        p.ksp = (a.T + p.TS - 1) / p.TS;  // parts that hold tiles
        const int64_t cost = (int64_t)((p.grid_x * p.ksp + n_cu - 1) / n_cu) * p.TS * (rgs + 20);
        if (rgs == 6 || cost < least) {
            best = p;
            least = cost;
        }
    }
    return best;
}

static int mvn_counters(const MvnPlan &p) { return p.ksp > 1 ? p.grid_x * 8 : 0; }

template <int NCW>
struct MvnOperands {
    u32x4 av[kMvnTiles][2], bv[kMvnTiles][NCW];
};
template <int EPI, int NCB, bool CANON, int WM>
__global__ __launch_bounds__(512) void k_mvN(MvArgs a, int TS) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int KT = kMvnTiles;
    constexpr int NCW = (NCB + 1) / 2;                 // column blocks of a wavefront (two wavefronts side by side)
    constexpr int RGS = 2 * WM;                        // row groups; wavefronts past 2 WM only copy
    constexpr int ST_BYTES = KT * (RGS + NCB) * 1024;
    constexpr int NST = kMvnRing / ST_BYTES;
    constexpr int NP = KT * (RGS + NCB), PW = (NP + 7) / 8;  // 1 KB pieces of a stage; of a wavefront
    static_assert(NST >= 3 && NST * PW < 60, "ring depth against the load counter");
    unsigned char *ring = smem;
    float *rs = (float *)(smem + NST * ST_BYTES + 1024);  // (operand reads of columns past the last run over a stage's end)
    uint32_t *touched = (uint32_t *)(rs + 80);         // [8][64]
    float *nscratch = rs + 80 + 512;                   // [1024]
    constexpr bool kNorm = EPI != EPI_RESID;
    const int R = a.R, NT = block_terms(a.RL), NC = NT * layout_rows(a.RL);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = min(wave / WM, 1);
    const bool worker = wave < 2 * WM;
    const int col = lane & 15, kg = lane >> 4;
    const int T = a.T, rgb = (int)blockIdx.x * RGS;  // first row group
    const int t_lo = (int)blockIdx.y * TS, t_hi = min(T, t_lo + TS), KSP = gridDim.y;
    const int n_c = CANON ? (T + 7) >> 3 : T;  // tiles of a slice
    const bool ragged = (a.K & 31) != 0 && t_hi == T;  // (a last tile past the real depth is not part of the pipeline)
    const int TF = t_hi - t_lo - (ragged ? 1 : 0);

    // (the norm partials go out ahead of the ring's first stages; the scales are read by the epilogue only)
    NormPart np;
    NormPart32 np32;
    NormPart64 np64;
    if (kNorm) {
        if (!CANON)  // (the bulk layouts' own order)
            mv_norm64_load(a, 0, np64);
        else if (a.rp == 16)
            np = mv_norm_load(a);
        else
            mv_norm32_load(a, 0, np32);
    }
    if (EPI == EPI_QKV) {  // the lines this wavefront's epilogue will write values into (see mv_touch_value_lines)
        const int d = a.head_dim, half = d >> 1, gph = half >> 3, rg = min(rgb + wave, a.n_rg - 1);
        const int hh = rg / gph, head = hh - a.n_q_heads - a.n_kv_heads, r = lane >> 1;
        if (a.nb32 > 0 && head >= 0 && r < R) {
            const uint16_t *vp = (const uint16_t *)a.vcache + (kv_vt_index(head, a.nb32, d, a.pos0 + r, 8 * (rg - hh * gph) + (lane & 1) * half) & ~(size_t)1);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)vp,
                                             (__attribute__((address_space(3))) void *)(touched + wave * 64), 4, 0, 0);
        }
    }
    // ---- what this wavefront copies per stage: pieces wave + 8 i (a row group's KT tiles, then KT tiles of B)
    const unsigned char *src[PW];
    int stride[PW];
    uint32_t voff[PW], vend[PW];  // (the last stage of a part may hold tiles past its end, which are not multiplied: cut at the matrix's)
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        const int p = min(wave + 8 * i, NP - 1);
        if (p < KT * RGS) {
            src[i] = (const unsigned char *)a.Wt + (size_t)min(rgb + p / KT, a.n_rg - 1) * T * 1024;
            stride[i] = 1024;
            voff[i] = lane * 16 + (t_lo + p % KT) * 1024;
            vend[i] = lane * 16 + (T - 1) * 1024;
        } else {
            src[i] = (const unsigned char *)a.in_s;
            stride[i] = 64 * NC;
            voff[i] = lane * 16 + t_lo * stride[i] + (p - KT * RGS) * 1024;
            vend[i] = (a.K >> 3) * NC * 16 - 16;
        }
    }
    const bool full_share = (NP % 8 == 0) || wave < NP % 8;
    auto issue = [&](int slot_bytes, auto FULL) {
        unsigned char *dst = ring + slot_bytes + wave * 1024;
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            if (i < PW - 1 || decltype(FULL)::value) {
                const auto from = (const __attribute__((address_space(1))) void *)(src[i] + (size_t)min(voff[i], vend[i]));
                const auto to = (__attribute__((address_space(3))) void *)(dst + i * 8192);
                if (wave + 8 * i < KT * RGS)  // (wavefront-uniform)
                    __builtin_amdgcn_global_load_lds(from, to, 16, 0, kNonTemporal);
                else
                    __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
            }
            voff[i] += KT * stride[i];
        }
    };
    auto wait_all_but = [&](auto N, auto FULL) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(N)::value * (decltype(FULL)::value ? PW : PW - 1)) : "memory");
    };
    auto lds_sync = [&]() {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        asm volatile("s_barrier" ::: "memory");
    };
    f32x4 acc[2][NCW], ssum[CANON ? 2 : 1][CANON ? NCW : 1];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int cb = 0; cb < NCW; ++cb) {
            acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (CANON) ssum[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    int left = n_c;  // tiles to the end of the slice (a workgroup's part begins with a slice)
    const unsigned char *a_base = ring + wm * 2048 * KT + lane * 16;
    const unsigned char *b_base = ring + KT * RGS * 1024 + (kg * NC + 16 * NCW * wn + col) * 16;
    const int tstride = 64 * NC;
    auto read_operands = [&](int slot_bytes, MvnOperands<NCW> &o) {
#pragma unroll
        for (int k = 0; k < KT; ++k) {
#pragma unroll
            for (int g = 0; g < 2; ++g) o.av[k][g] = *(const u32x4 *)(a_base + slot_bytes + (g * KT + k) * 1024);
#pragma unroll
            for (int cb = 0; cb < NCW; ++cb) o.bv[k][cb] = *(const u32x4 *)(b_base + slot_bytes + k * tstride + cb * 256);
        }
    };
    auto slice_end = [&]() {
        if constexpr (CANON) {
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int cb = 0; cb < NCW; ++cb) {
                    ssum[g][cb] += acc[g][cb];
                    acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    auto multiply = [&](const u32x4(&av)[2], const u32x4(&bv)[NCW]) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int cb = 0; cb < NCW; ++cb)
                acc[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[g]), __builtin_bit_cast(bf16x8, bv[cb]),
                                                                     acc[g][cb], 0, 0, 0);
    };
    auto norm = [&]() {
        if (!kNorm) return;
        if (!CANON)
            mv_norm64_finish(a, np64, rs, nscratch);
        else if (a.rp == 16)
            mv_norm_finish<true>(a, np, rs, nscratch);
        else
            mv_norm32_finish(a, np32, rs, nscratch);
    };
    auto pipeline = [&](auto FULL) {
        constexpr auto ALL = std::integral_constant<int, 0>();
        constexpr auto AHEAD = std::integral_constant<int, NST - 2>();
        const int SF = (TF + KT - 1) / KT;  // stages
        const int first = min(SF, NST);
        for (int t = 0; t < first; ++t) issue(t * ST_BYTES, FULL);
        norm();
        if (SF == 0) return;
        if (SF >= NST)
            wait_all_but(std::integral_constant<int, NST - 1>(), FULL);
        else
            wait_all_but(ALL, FULL);
        MvnOperands<NCW> o0, o1;
        lds_sync();
        if (worker) read_operands(0, o0);
        int t = 0, slot = 0, todo = TF;
        auto step = [&](const MvnOperands<NCW> &cur, MvnOperands<NCW> &nxt, auto STEADY) {
            const int nslot = slot + ST_BYTES == NST * ST_BYTES ? 0 : slot + ST_BYTES;
            if (decltype(STEADY)::value)
                wait_all_but(AHEAD, FULL);
            else
                wait_all_but(ALL, FULL);
            lds_sync();
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(STEADY)::value) issue(slot, FULL);
            if (worker) {
                read_operands(nslot, nxt);
#pragma unroll
                for (int k = 0; k < KT; ++k) {
                    if (k > 0 && todo <= k) break;
                    multiply(cur.av[k], cur.bv[k]);
                    if (CANON && --left == 0) {  // (wavefront-uniform)
                        slice_end();
                        left = n_c;
                    }
                }
            }
            todo -= KT;
            slot = nslot;
        };
        constexpr auto GO = std::true_type();
        constexpr auto DRAIN = std::false_type();
        for (; t + NST + 1 < SF; t += 2) {
            step(o0, o1, GO);
            step(o1, o0, GO);
        }
        if (t + NST < SF) {
            step(o0, o1, GO);
            step(o1, o0, DRAIN);
            t += 2;
        }
        for (; t < SF; t += 2) {
            step(o0, o1, DRAIN);
            if (t + 1 < SF) step(o1, o0, DRAIN);
        }
    };
    if (full_share)
        pipeline(std::true_type());
    else
        pipeline(std::false_type());
    if (ragged) {
        const int real_units = (a.K >> 3) * NC;  // 16-byte units of the split activation
        __syncthreads();
        for (int i = tid; i < RGS * 64; i += 512)
            *(u32x4 *)(ring + (i >> 6) * 1024 * KT + (i & 63) * 16) =
                *((const u32x4 *)a.Wt + ((size_t)min(rgb + (i >> 6), a.n_rg - 1) * T + T - 1) * 64 + (i & 63));
        for (int i = tid; i < 4 * NC; i += 512) {
            const int gu = (T - 1) * 4 * NC + i;
            *(u32x4 *)(ring + KT * RGS * 1024 + i * 16) = gu < real_units ? ((const u32x4 *)a.in_s)[gu] : u32x4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        MvnOperands<NCW> o;
        if (worker) {
            read_operands(0, o);
            multiply(o.av[0], o.bv[0]);
        }
        --left;
    }
    if (CANON && left != n_c) slice_end();

    // ---- results to LDS ([row group][column][tile row]), then the epilogue, or with split K the partial
    __syncthreads();  // the ring is no longer read
    float *dump = (float *)ring;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int cb = 0; cb < NCW; ++cb) {
            const int c = 16 * (NCW * wn + cb) + col;
            const f32x4 v = CANON ? ssum[CANON ? g : 0][CANON ? cb : 0] : acc[g][cb];
            if (worker && c < 16 * NCB) *(f32x4 *)(dump + ((2 * wm + g) * (16 * NCB) + c) * 16 + 4 * kg) = v;
        }
    __syncthreads();
    const int rg = rgb + wave;
    const bool live = wave < RGS && rg < a.n_rg;
    const float *dw = dump + wave * (NCB * 256);
    auto y_local = [&](int r, int j) {
        const float y2 = dw[(NT * r) * 16 + j] + dw[(NT * r + 1) * 16 + j];
        return NT == 3 ? y2 + dw[(3 * r + 2) * 16 + j] : y2;
    };
    if (KSP == 1) {
        if (live) mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_local);
        return;
    }
    // ---- every wavefront publishes its row group's partial, terms combined, and counts itself in; of the KSP wavefronts with the
    // same row group the one that arrives last adds the partials in part order and runs the epilogue.  Stores and loads of
    // the partials are device scope (written through, read past this die's L2), so once a wavefront's stores are acknowledged a
    // relaxed count publishes them, and no cache has to be written back or invalidated (as an acquire-release count per
    // workgroup does: 7B, 31 rows, down_proj 30.0 us, 28.0 this way; 64 bulk rows, o_proj 28.6 and 24.3).
    if (!live) return;
    const __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(a.part, 0, 0x7fffffff, 0x00020000);
    auto part_off = [&](int ky, int i) { return (uint32_t)(((ky * a.n_rg + rg) * 4 * R + i) * 16); };  // i: four results of a row
    float *dm = dump + wave * (NCB * 256);
    for (int i = lane; i < 4 * R; i += 64) {
        const float *d = dm + NT * (i >> 2) * 16 + 4 * (i & 3);
        f32x4 y = *(const f32x4 *)d + *(const f32x4 *)(d + 16);
        if (NT == 3) y = y + *(const f32x4 *)(d + 32);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), part, part_off(blockIdx.y, i), 0, kDeviceScope);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int *counter = a.counters + blockIdx.x * 8 + wave;
    int arrived = 0;
    if (lane == 0) arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(arrived) != KSP - 1) return;
    asm volatile("" ::: "memory");
    for (int i = lane; i < 4 * R; i += 64) {
        f32x4 v[8];
#pragma unroll
        for (int s2 = 0; s2 < 8; ++s2)
            v[s2] = s2 < KSP ? __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part, part_off(s2, i), 0, kDeviceScope))
                             : f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 y = v[0];
#pragma unroll
        for (int s2 = 1; s2 < 8; ++s2) y += v[s2];
        *(f32x4 *)(dm + 4 * i) = y;  // [row][16], over what this wavefront alone has read
    }
    // (one wavefront's LDS instructions are carried out in order: only the compiler has to keep it)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    mv_epilogue<EPI>(a, rg, lane, rs, nullptr, [&](int r, int j) { return dm[r * 16 + j]; });
    if (lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int EPI, int NCB, bool CANON, int WM>
static hipError_t launch_mvN_t(const MvArgs &a, int n_cu, hipStream_t s) {
    constexpr int ST = kMvnTiles * (2 * WM + NCB) * 1024;
    const size_t lds = kMvnRing / ST * ST + 1024 + (80 + 512 + 1024) * 4;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_mvN<EPI, NCB, CANON, WM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const MvnPlan p = mvn_plan(a, n_cu, CANON);
    if (mvn_counters(p) > kMvCounters) return hipErrorInvalidValue;
    return launch_maybe_timed(k_mvN<EPI, NCB, CANON, WM>, dim3(p.grid_x, p.ksp), dim3(512), lds, s, a, p.TS);
}

template <int EPI, int NCB, bool CANON>
static hipError_t launch_mvN(const MvArgs &a, int n_cu, hipStream_t s) {
    return mvn_plan(a, n_cu, CANON).rgs == 6 ? launch_mvN_t<EPI, NCB, CANON, 3>(a, n_cu, s) : launch_mvN_t<EPI, NCB, CANON, 4>(a, n_cu, s);
}

// ------------------------------------------------------------------------------------------
// 6..32 activation rows (and any number whose activation is too deep for k_mv1): every wavefront on its own
// ------------------------------------------------------------------------------------------
// As in k_mv1, eight wavefronts share RG row groups of W, each streaming one of the eight K slices through a rolling window
// of NS steps (a step: the tile of each of the RG row groups and the NCB column blocks of B that meet it), and the slice
// sums are added in LDS in the one fixed order.  B is not staged: it comes straight from L2, which holds it (27 columns x
// 4096: 221 KB) and delivers 128 B/ns to a compute unit that takes in about 26 B/ns of weights, so that nothing couples
// the wavefronts between the ends of a round.
// (the slice sums of two rounds, where LDS holds them: one barrier a round)
template <int NCB, int RG>
constexpr bool kMvrTwoBuffers = 2 * 8 * RG * 16 * NCB * 16 * 4 <= 150 * 1024;
template <int EPI, int NCB, int RG, int NS>
__global__ __launch_bounds__(512) void k_mvR(MvArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NCP = 16 * NCB;                 // columns as computed
    constexpr int kRed = 8 * RG * NCP * 16;       // floats of one round's slice sums
    constexpr bool kTwo = kMvrTwoBuffers<NCB, RG>;
    float *red = (float *)smem;                   // [kTwo ? 2 : 1][8 slices][RG][NCP][16]
    float *rs = red + (kTwo ? 2 : 1) * kRed;      // [32]
    float *nscratch = rs + 32;                    // [1024]
    constexpr bool kNorm = EPI != EPI_RESID;
    const int NT = block_terms(a.RL), NC = NT * layout_rows(a.RL);
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kg = lane >> 4;
    const int T = a.T;
    const int n = (T + 7) >> 3;                // k tiles of a slice
    const int t0 = min(ks * n, T - 1);
    const int nv = max(0, min(n, T - ks * n)); // ... of which exist
    const int nvm1 = max(nv - 1, 0);
    const int W = a.n_wg, last_rg = a.n_rg - 1;
    const u32x4 *Wt = (const u32x4 *)a.Wt;
    const unsigned char *bb = (const unsigned char *)a.in_s;
    // this lane's byte offset of B for tile t0 (columns past NC read what lies there: results nobody reads); in a ragged
    // last tile the lanes past the real depth read its last chunk, and meet zero weights
    const uint32_t bstride = 64u * NC;
    const uint32_t boff = ((uint32_t)(4 * t0 + kg) * NC + col) * 16u;
    const uint32_t bmax = ((uint32_t)((a.K >> 3) - 1) * NC + col) * 16u;

    u32x4 A[NS][RG], B[NS][NCB];
    const u32x4 *base[RG];
    auto load_step = [&](int i, u32x4(&Av)[RG], u32x4(&Bv)[NCB]) {
        const int ii = min(i, nvm1);
#pragma unroll
        for (int g = 0; g < RG; ++g) Av[g] = __builtin_nontemporal_load(base[g] + (size_t)ii * 64);
        const uint32_t off = min(boff + (uint32_t)ii * bstride, bmax);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) Bv[cb] = *(const u32x4 *)(bb + off + 256 * cb);
    };
    auto set_base = [&](int seg) {
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const int rg = min((seg * W + (int)blockIdx.x) * RG + g, last_rg);
            base[g] = Wt + ((size_t)rg * T + t0) * 64 + lane;
        }
    };
    // (the norm partials go out first; the scales are read by the epilogue only, so an LDS-only barrier will do)
    NormPart np;
    NormPart32 np32;
    if (kNorm) {
        if (a.rp == 16)
            np = mv_norm_load(a);
        else
            mv_norm32_load(a, 0, np32);
    }
    set_base(0);
#pragma unroll
    for (int u = 0; u < NS; ++u) load_step(u, A[u], B[u]);
    if (EPI == EPI_QKV) {
        // the lines the epilogues of this workgroup's rounds will write values into (wavefront s: round s)
        if (ks < a.S)
            for (int g = 0; g < RG; ++g) mv_touch_value_lines(a, min((ks * W + (int)blockIdx.x) * RG + g, last_rg), lane);
    }
    if (kNorm) {
        if (a.rp == 16)
            mv_norm_finish<true>(a, np, rs, nscratch);
        else
            mv_norm32_finish(a, np32, rs, nscratch);
    }

    f32x4 acc[RG][NCB];
    auto mma_step = [&](int i, const u32x4(&Av)[RG], const u32x4(&Bv)[NCB]) {
        if (i >= nv) return;  // (wavefront-uniform)
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
                acc[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Av[g]), __builtin_bit_cast(bf16x8, Bv[cb]),
                                                                     acc[g][cb], 0, 0, 0);
    };
    const int nb = (n + NS - 1) / NS;
    for (int seg = 0; seg < a.S; ++seg) {
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int b = 0; b + 1 < nb; ++b) {
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_step(b * NS + u, A[u], B[u]);
                load_step((b + 1) * NS + u, A[u], B[u]);
            }
        }
        if (seg + 1 < a.S) {
            // the window rolls on into the next round's row groups: the stream never drains
            set_base(seg + 1);
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_step((nb - 1) * NS + u, A[u], B[u]);
                load_step(u, A[u], B[u]);
            }
        } else {
#pragma unroll
            for (int u = 0; u < NS; ++u) mma_step((nb - 1) * NS + u, A[u], B[u]);
        }
        // ---- end of the round: slice sums to LDS, then all wavefronts share the epilogue
        if (!kTwo && seg > 0) lds_barrier();  // (the previous round's sums are no longer read)
        float *rp = red + (kTwo ? (size_t)(seg & 1) * kRed : 0);
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) *(f32x4 *)(rp + ((ks * RG + g) * NCP + 16 * cb + col) * 16 + 4 * kg) = acc[g][cb];
        lds_barrier();  // (the next round's loads stay in flight)
        constexpr int share = 8 / RG;              // wavefronts per row group
        const int g = ks / share;
        const int rg = (seg * W + (int)blockIdx.x) * RG + g;
        if (g < RG && rg <= last_rg) {
            mv_epilogue<EPI>(a, rg, lane, rs, nullptr, [&](int r, int j) {
                // (the order of k_mv1: per term in groups of kgroup slices, the terms of a group combined, groups in order)
                const int kgroup = a.kgroup;
                const float *w = rp + (g * NCP + NT * r) * 16 + j;
                constexpr int ss = RG * NCP * 16;  // from one slice to the next
                float y = 0.f;
#pragma unroll 1
                for (int k0 = 0; k0 < 8; k0 += kgroup) {
                    float hi = w[0], mid = w[16], lo = NT == 3 ? w[32] : 0.f;
                    w += ss;
#pragma unroll 1
                    for (int k2 = 1; k2 < kgroup; ++k2) {
                        hi += w[0];
                        mid += w[16];
                        if (NT == 3) lo += w[32];
                        w += ss;
                    }
                    const float gs = (hi + mid) + lo;
                    y = k0 == 0 ? gs : y + gs;
                }
                return y;
            }, ks - g * share, share);
        }
    }
}

// Steps in flight per wavefront: what 256 registers hold beside the accumulators (3 x 6 tiles: two steps, three spill).
constexpr int mvr_steps(int ncb, int rg) {
    const int n = ((rg * ncb >= 18 ? 144 : rg * ncb >= 8 ? 184 : 200) - 4 * rg * ncb) / (4 * (rg + ncb));
    return n > 10 ? 10 : n;
}

// A second depth for slices that the first one cuts badly (slots past the end of a slice load its last tile again): 16, 20,
// 32 and 43 tiles are 2 x 8, 2 x 10 or 5 x 4, 4 x 8 and 5 x 9 or 11 x 4.
constexpr int mvr_other_steps(int ns) { return ns > 8 ? 8 : ns == 8 ? 7 : ns > 4 ? 4 : ns == 3 ? 2 : ns; }
// The better of the two depths for a slice of n tiles, and the steps of the slice as walked with it.
static int mvr_depth(int n, int ncb, int rg) {
    const int a = mvr_steps(ncb, rg), b = mvr_other_steps(a);
    return (n + a - 1) / a * a <= (n + b - 1) / b * b ? a : b;
}
static int mvr_slots(int n, int ncb, int rg) {
    const int d = mvr_depth(n, ncb, rg);
    return (n + d - 1) / d * d;
}

template <int EPI, int NCB, int RG, int NS>
static hipError_t launch_mvR_ns(const MvArgs &a, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_mvR<EPI, NCB, RG, NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const size_t lds = (size_t)(kMvrTwoBuffers<NCB, RG> ? 2 : 1) * 8 * RG * 16 * NCB * 16 * 4 + 32 * 4 + 1024 * 4;
    return launch_maybe_timed(k_mvR<EPI, NCB, RG, NS>, dim3(a.n_wg), dim3(512), lds, s, a);
}
template <int EPI, int NCB, int RG>
static hipError_t launch_mvR_t(MvArgs a, int n_cu, hipStream_t s) {
    const int units = (a.n_rg + RG - 1) / RG;
    a.S = (units + n_cu - 1) / n_cu;
    a.n_wg = (units + a.S - 1) / a.S;
    a.kgroup = mv_slice_group(a, n_cu);
    constexpr int NS = mvr_steps(NCB, RG), NS2 = mvr_other_steps(NS);
    return mvr_depth((a.T + 7) / 8, NCB, RG) == NS ? launch_mvR_ns<EPI, NCB, RG, NS>(a, s) : launch_mvR_ns<EPI, NCB, RG, NS2>(a, s);
}

// A line between small blocks and large ones: row groups per workgroup round for k_mvR short of it, 0 beyond.  Two things hang on
// it: which kernel exact blocks take (mvr_row_groups), and how bulk blocks of 32 rows add their sums (mvn_canon).
// It is where k_mvR broke even with the kernel that k_mvN replaces, by what one compute unit had to
// walk, in us per k tile, fitted to 709 sets of launch durations of both (rows 1-32 of both layouts, seven widths
// from 1024 to 8192, matrices of 6 to 1300 MB).  c: column blocks, 0.4 x those computed + 0.6 x the columns' own share.
//   k_mvR   3.7 + rounds x 8 slices x steps of a slice as walked x (weights of 1, 2 or 3 row groups + c columns of B)
//   line    6.1 (+ 2.8 + 0.96 c where K is split over workgroups) + rounds x tiles (a slice's last chunk of eight, where it
//           is partial, counts half of what it lacks) x (row groups + c columns), by the root of the share of units in use
static int mvr_line(const MvArgs &a, int n_cu, int ncb) {
    if (ncb < 1 || ncb > 6 || a.R > kMaxRows) return 0;
    static const double kWeights[3] = {0.0213, 0.0467, 0.0603}, kColumns[3] = {0.0147, 0.0178, 0.0226};
    const bool bulk = (a.RL & kBulkLayout) != 0;
    const double cols = 0.4 * ncb + 0.6 * (block_terms(a.RL) * layout_rows(a.RL)) / 16.0;
    double best = 1e30;
    int rg = 0;
    if (ncb > 1) {  // (one column block: activations too deep for k_mv1, which k_mvN does not take)
        const int n_rb = (a.n_rg + 7) / 8;
        int parts = std::min(8, std::max(1, n_cu / n_rb)), TS = ((a.T + 7) / 8) * mv_slice_group(a, n_cu);
        if (bulk) {
            while (parts > 1 && ((a.T + parts - 1) / parts < 8 || (int64_t)a.n_rg * parts > a.part_capacity)) --parts;
            TS = (a.T + parts - 1) / parts;
        }
        parts = (a.T + TS - 1) / TS;
        const int rgs = n_rb * parts < n_cu ? std::min(8, std::max(4, (a.n_rg * parts + n_cu - 1) / n_cu)) : 8;
        const int n = bulk ? TS : (a.T + 7) / 8;  // tiles of a slice
        const double walked = TS + 0.5 * (TS / n) * ((n + 7) / 8 * 8 - n);
        const int wgs = (a.n_rg + rgs - 1) / rgs * parts, rounds = (wgs + n_cu - 1) / n_cu;
        best = 6.05 + (parts > 1 ? 2.83 + 0.964 * cols : 0.0) +
               rounds * walked * (rgs * 0.0349 + cols * (bulk ? 0.0212 : 0.0284)) * sqrt((double)wgs / (rounds * n_cu));
    }
    for (int c = 1; c <= 3; ++c) {
        if (ncb > 4 && c == 2) continue;
        const int units = (a.n_rg + c - 1) / c, S = (units + n_cu - 1) / n_cu;
        const double us = 3.68 + (double)S * 8 * mvr_slots((a.T + 7) / 8, ncb, c) * (kWeights[c - 1] + cols * kColumns[c - 1]);
        if (us < best) {
            best = us;
            rg = c;
        }
    }
    return rg;
}
// Row groups per workgroup round for k_mvR, or 0: k_mvN.  From eleven exact (17 bulk) rows on, k_mvN takes the matrices that its
// workgroups of six row groups cover in one round with K whole (us, k_mvR / k_mvN, 7B gate/up: 16 rows 35.8 / 33.5, 21 rows 43.0 /
// 35.3, 26 rows 48.1 / 38; 9 rows 33 / 34); elsewhere what lies beyond the line.
// The line prices the predecessor of k_mvN, so it is not where today's two kernels break even (both timed at the 7B, 13B and 70B
// widths, 6-32 rows: profiles/block_projection_sweep.txt, third table).  Beyond it k_mvN is faster throughout (us, k_mvR / k_mvN: 7B, 31
// rows down_proj 41.8 / 28.2, LM head 75 / 47.5; 13B, 24 rows gate/up 82 / 54).  Short of it k_mvR is where the matrix is narrow or
// the rows few (7B, 9 rows q|k|v 20.4 / 23.5, 31 rows o_proj 17 / 20), and k_mvN would be by up to 32 % in a strip along it (13B, 18 rows LM
// head 72.8 / 55.1, 9 rows gate/up 54.9 / 46.9, 21 rows q|k|v 42 / 34.5; 7B, 13 rows down_proj 28.6 / 23.1; 70B, 18 rows gate/up 187 / 160,
// 16 rows down_proj 93 / 75): 3.5 % over all launches of the table.  Exact blocks come out the same bits either way.
static int mvr_row_groups(const MvArgs &a, int n_cu, int ncb) {
    if (ncb > 2 && ncb <= 6) {
        const MvnPlan p = mvn_plan(a, n_cu, true);
        if (p.rgs == 6 && p.ksp == 1) return 0;
    }
    return mvr_line(a, n_cu, ncb);
}
// Whether k_mvN adds the eight slices: exact layouts, and bulk ones of 32 rows short of the line (K whole there), whose sums are
// k_mvR's then.  This is an order of sums and no rule about speed: a short prompt's cache entries hang on it, whichever kernel
// runs, so it stays where it is if the choice between the kernels moves.
static bool mvn_canon(const MvArgs &a, int n_cu, int ncb) { return !(a.RL & kBulkLayout) || mvr_line(a, n_cu, ncb) != 0; }

// Small blocks (in their own exact layout) whose whole activation fits in LDS take the single-pass kernel.
static bool mv_takes_mv1(const MvArgs &a, int ks_override) {
    return !(a.RL & kBulkLayout) && a.R <= kMvSmallRows && ks_override != 16 && mv1_lds_bytes(a.K, a.R, a.head_dim) <= kMvMaxLds;
}
static int mv_column_blocks(const MvArgs &a) { return (block_terms(a.RL) * layout_rows(a.RL) + 15) / 16; }

int mv_path_name(const MvArgs &a, int n_cu, char *out, int capacity) {
    if (mv_takes_mv1(a, 0)) return snprintf(out, (size_t)capacity, "mv1<rows %d>", a.R);
    const int ncb = mv_column_blocks(a), rg = mvr_row_groups(a, n_cu, ncb);
    if (rg == 0) return snprintf(out, (size_t)capacity, "mvN<columns %d, parts %d>", ncb, mvn_plan(a, n_cu, mvn_canon(a, n_cu, ncb)).ksp);
    const int units = (a.n_rg + rg - 1) / rg;
    return snprintf(out, (size_t)capacity, "mvR<columns %d, row groups %d, steps %d, rounds %d>", ncb, rg,
                    mvr_depth((a.T + 7) / 8, ncb, rg), (units + n_cu - 1) / n_cu);
}

int mv_split_slots(const MvArgs &a, int n_cu) {
    if (a.RL & kBulkLayout) return a.part_capacity;  // (bulk layouts: not needed by callers)
    if (mv_takes_mv1(a, 0)) return 0;
    // (what k_mvN needs, also where k_mvR, which needs none, is the faster kernel: what a caller's scratch has to hold does
    // not hang on a rule about speed)
    const int TS = ((a.T + 7) / 8) * mv_slice_group(a, n_cu);
    const int ksp = (a.T + TS - 1) / TS;
    return ksp > 1 ? ksp * a.n_rg : 0;
}

int mv_split_counters(const MvArgs &a, int n_cu) {
    if (mv_split_slots(a, n_cu) == 0) return 0;
    return mvn_counters(mvn_plan(a, n_cu, mvn_canon(a, n_cu, mv_column_blocks(a))));
}

hipError_t launch_mv(int epi, MvArgs a, int n_cu, int ks_override, int wg_override, hipStream_t s) {
    const bool bulk = (a.RL & kBulkLayout) != 0;
    const int lrows = layout_rows(a.RL);
    if (a.R < 1 || a.R > kMaxBlockRows || (a.rp != 16 && a.rp != 64) || a.R > a.rp || a.R > lrows ||
        (bulk ? (lrows != 32 && lrows != 64) : (lrows != a.R || lrows > kMaxRows)) || a.head0 != 0)
        return hipErrorInvalidValue;
    if (mv_takes_mv1(a, ks_override)) return launch_mv1(epi, a, n_cu, ks_override, wg_override, s);
    // exact layouts (up to 32 rows): 2-6 column blocks of three-term columns, the fixed
    // summation order; bulk layouts of 32 / 64 rows (prefill, candidate evaluation): 4 / 8 column blocks of
    // two-term columns
    const int ncb = mv_column_blocks(a);
    if (const int rg = mvr_row_groups(a, n_cu, ncb)) {
#define SWIFT_MVR_RG(E, N)                                          \
    case N:                                                         \
        if (rg == 1) return launch_mvR_t<E, N, 1>(a, n_cu, s);      \
        if (rg == 2) return launch_mvR_t<E, N, 2>(a, n_cu, s);      \
        return launch_mvR_t<E, N, 3>(a, n_cu, s);
#define SWIFT_MVR_CASE(E)                                                                     \
    case E:                                                                                   \
        switch (ncb) {                                                                        \
            SWIFT_MVR_RG(E, 1)                                                                \
            SWIFT_MVR_RG(E, 2)                                                                \
            SWIFT_MVR_RG(E, 3)                                                                \
            SWIFT_MVR_RG(E, 4)                                                                \
            case 5: return rg == 1 ? launch_mvR_t<E, 5, 1>(a, n_cu, s) : launch_mvR_t<E, 5, 3>(a, n_cu, s); \
            case 6: return rg == 1 ? launch_mvR_t<E, 6, 1>(a, n_cu, s) : launch_mvR_t<E, 6, 3>(a, n_cu, s); \
            default: return hipErrorInvalidValue;                                             \
        }
        switch (epi) {
            SWIFT_MVR_CASE(EPI_QKV)
            SWIFT_MVR_CASE(EPI_RESID)
            SWIFT_MVR_CASE(EPI_SWIGLU)
            SWIFT_MVR_CASE(EPI_LOGITS)
        }
#undef SWIFT_MVR_CASE
#undef SWIFT_MVR_RG
        return hipErrorInvalidValue;
    }
    const bool canon = mvn_canon(a, n_cu, ncb);
#define SWIFT_MVN_CASE(E)                                                                \
    case E:                                                                              \
        if (bulk) switch (ncb) {                                                         \
                case 4: return canon ? launch_mvN<E, 4, true>(a, n_cu, s) : launch_mvN<E, 4, false>(a, n_cu, s); \
                case 8: return launch_mvN<E, 8, false>(a, n_cu, s);                      \
                default: return hipErrorInvalidValue;                                    \
            }                                                                            \
        switch (ncb) {                                                                   \
            case 2: return launch_mvN<E, 2, true>(a, n_cu, s);                           \
            case 3: return launch_mvN<E, 3, true>(a, n_cu, s);                           \
            case 4: return launch_mvN<E, 4, true>(a, n_cu, s);                           \
            case 5: return launch_mvN<E, 5, true>(a, n_cu, s);                           \
            case 6: return launch_mvN<E, 6, true>(a, n_cu, s);                           \
            default: return hipErrorInvalidValue;                                        \
        }
    switch (epi) {
        SWIFT_MVN_CASE(EPI_QKV)
        SWIFT_MVN_CASE(EPI_RESID)
        SWIFT_MVN_CASE(EPI_SWIGLU)
        SWIFT_MVN_CASE(EPI_LOGITS)
    }
#undef SWIFT_MVN_CASE
    return hipErrorInvalidValue;
}

}  // namespace swift
