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

constexpr int kNonTemporal = 2;  // cache policies: nt; sc1
constexpr int kDeviceScope = 16;

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
// RMSNorm scale per block row from the producer's partial sums of squares.  A kernel requests the first 256 partials of its rows
// (hidden <= 4096: all of them) ahead of its weights and adds them up once the weights are on their way: no branches
// and no use of a loaded value in between (a partial past the last is the last one again, left out of the sum later), since a
// wait there would hold the weights up.  The summation order is fixed.  One barrier, which orders LDS only, before the final sums.
//
// Up to 16 rows (row pitch 16): thread (q = t / 16, row r = t % 16) adds the partials q + 32 u in order of u, then 16 threads
// add the 32 sums in order.
struct NormPart {
    float v[8];
};
__device__ inline NormPart mv_norm_load(const MvArgs &a, int p0 = 0) {
    NormPart np;
    const uint32_t at = threadIdx.x + 16 * p0, end = 16 * a.n_pss - 1;  // partial p of row r is word 16 p + r
#pragma unroll
    for (int u = 0; u < 8; ++u) np.v[u] = *(const float *)((const char *)a.pss + 4 * min(at + 512 * u, end));
    return np;
}
__device__ inline void mv_norm_finish(const MvArgs &a, const NormPart &np, float *rs /* LDS [16] */, float *scratch /* LDS [512] */) {
    const int tid = threadIdx.x, q = tid >> 4;
    float ss = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u) ss += q + 32 * u < a.n_pss ? np.v[u] : 0.f;
    for (int p0 = 256; p0 < a.n_pss; p0 += 256) {
        const NormPart more = mv_norm_load(a, p0);
#pragma unroll
        for (int u = 0; u < 8; ++u) ss += p0 + q + 32 * u < a.n_pss ? more.v[u] : 0.f;
    }
    scratch[tid] = ss;
    lds_barrier();
    if (tid < 16) {
        float t = 0.f;
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) t += scratch[q2 * 16 + tid];
        rs[tid] = 1.0f / sqrtf(t / (float)a.norm_dim + a.eps);
    }
    // (no barrier here: the scales are read by the epilogue only, and every caller has a barrier between
    // this point and its epilogue)
}

// The same for exact layouts of 17..32 rows (row pitch 64), in the same order -- a row's scale must not depend on the rows it
// shares a pass with: thread (row r, q) adds the partials q + 32 u and q + 16 + 32 u as two sums; then 32 threads add the 32 sums
// in order.
struct NormPart32 {
    float v[2][8];
};
__device__ inline NormPart32 mv_norm32_load(const MvArgs &a, int p0 = 0) {
    NormPart32 np;
    const uint32_t r = threadIdx.x & 31, at = 64 * (p0 + (threadIdx.x >> 5)) + r, end = 64 * (a.n_pss - 1) + r;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int u = 0; u < 8; ++u) np.v[half][u] = *(const float *)((const char *)a.pss + 4 * min(at + 64 * (16 * half + 32 * u), end));
    return np;
}
__device__ inline void mv_norm32_finish(const MvArgs &a, const NormPart32 &np, float *rs /* LDS [32] */, float *scratch /* LDS [1024] */) {
    const int tid = threadIdx.x, r = tid & 31, q0 = tid >> 5;
    float ss[2] = {0.f, 0.f};
    auto add = [&](int p0, const NormPart32 &n) {
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int u = 0; u < 8; ++u) ss[half] += p0 + q0 + 16 * half + 32 * u < a.n_pss ? n.v[half][u] : 0.f;
    };
    add(0, np);
    for (int p0 = 256; p0 < a.n_pss; p0 += 256) add(p0, mv_norm32_load(a, p0));
    scratch[q0 * 32 + r] = ss[0];
    scratch[(q0 + 16) * 32 + r] = ss[1];
    lds_barrier();
    if (tid < 32) {
        float t = 0.f;
#pragma unroll
        for (int q2 = 0; q2 < 32; ++q2) t += scratch[q2 * 32 + tid];
        rs[tid] = 1.0f / sqrtf(t / (float)a.norm_dim + a.eps);
    }
}

// The same for bulk layouts of 64 rows: thread = (partial p mod 8, row r), then 64 threads add the 8 per-thread sums in order.
struct NormPart64 {
    float v[32];
};
__device__ inline NormPart64 mv_norm64_load(const MvArgs &a, int p0 = 0) {
    NormPart64 np;
    const uint32_t at = threadIdx.x + 64 * p0, end = 64 * (a.n_pss - 1) + (threadIdx.x & 63);  // partial p of row r is word 64 p + r
#pragma unroll
    for (int u = 0; u < 32; ++u) np.v[u] = *(const float *)((const char *)a.pss + 4 * min(at + 512 * u, end));
    return np;
}
__device__ inline void mv_norm64_finish(const MvArgs &a, const NormPart64 &np, float *rs /* LDS [64] */, float *scratch /* LDS [512] */) {
    const int tid = threadIdx.x, q = tid >> 6;
    float ss = 0.f;
    auto add = [&](int p0, const NormPart64 &n) {
#pragma unroll
        for (int u = 0; u < 32; ++u) ss += p0 + q + 8 * u < a.n_pss ? n.v[u] : 0.f;
    };
    add(0, np);
    for (int p0 = 256; p0 < a.n_pss; p0 += 256) add(p0, mv_norm64_load(a, p0));
    scratch[tid] = ss;
    lds_barrier();
    if (tid < 64) {
        float t = 0.f;
#pragma unroll
        for (int q2 = 0; q2 < 8; ++q2) t += scratch[q2 * 64 + tid];
        rs[tid] = 1.0f / sqrtf(t / (float)a.norm_dim + a.eps);
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
// launcher picks the depth that cuts the slice with the fewest unused slots), and the window rolls on from one round into the next.
// What bounds it: the weight stream (6.9 TB/s on large matrices) and about 3 us of start and end per launch.  The start: what the
// first loads need travels in the kernel's leading arguments, which are in registers when a wavefront starts; the activation, the
// residual values and the rotary rows go straight to LDS, and loads go out without a branch or a wait between them (a slice is a
// buffer: past its end it reads nothing).  The end: residual values that are there already, and slice sums read all at once in
// the last round.  us, before / now (launches back to back, 7B): one row o_proj 8.8 / 7.8, down_proj 16.8 / 16.3, LM head 41.0 /
// 40.4; two rows down_proj 18.3 / 16.9; five rows q|k|v 22.5 / 20.6, o_proj 10.7 / 9.0, gate/up 32.0 / 31.1, LM head 44.0 / 43.1;
// 13B, one row gate/up 44.3 / 43.2, down_proj 25.8 / 24.3.  7B gate/up of one row stays at 29.7.
// LDS beyond mv1_lds_bytes: the touched lines and what rounds the rotary rows up to whole copies.
constexpr size_t kMv1MoreLds = 256 + 512;
__host__ __device__ inline int mv1_rot_pitch(int R, int head_dim) { return (R * (head_dim >> 1) + 63) & ~63; }
template <int EPI, int KS, int NS>
__global__ __launch_bounds__(512, 4) void k_mv1(const unsigned char *Wt, const unsigned char *in_s, int T, int K, int R, int n_rg, int W,
                                                 int S, MvArgs rest) {  // 4 wavefronts per SIMD: <= 128 VGPRs, two workgroups per CU
    extern __shared__ __align__(16) unsigned char smem[];
    const int NC = 3 * R;
    // LDS: [16 B zeros][4T chunks x NC x 8 bf16][2 x 8 wavefronts x NC x 16 fp32][16 scales][512 scratch][64 touched][R x d rotary]
    float *red = (float *)(smem + 16 + (size_t)T * 64 * NC);
    float *rs = red + 2 * 8 * 16 * NC;
    float *nscratch = rs + 16;
    float *touched = nscratch + 512;  // [64]
    float *rot = touched + 64;        // [R][d/2] cosines, then sines (at mv1_rot_pitch), of the block rows' positions
    constexpr int G = 8 / KS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform from here on
    const int g = wave / KS, ks = wave - g * KS;
    const int n = (T + KS - 1) / KS;           // k-tiles per wavefront and row group
    const int t0 = min(ks * n, T - 1);
    const int nv = max(0, min(n, T - ks * n)); // ... of which exist
    const int last_rg = n_rg - 1;
    const int col = lane & 15, kg = lane >> 4;
    // byte address of this lane's B chunk for tile t: boff + t * bstride; lanes of columns >= NC
    // (and slots past the wavefront's slice) read the zero chunk at address 0
    const int boff = col < NC ? 16 + (kg * NC + col) * 16 : 0;
    const int bstride = col < NC ? 64 * NC : 0;

    u32x4 buf[NS];
    // (the slice as a buffer: slots past its end read nothing and give zeros)
    const uint32_t lane16 = lane * 16;
    __amdgpu_buffer_rsrc_t slice;
    auto set_slice = [&](int seg) {
        const int rg = min((seg * W + (int)blockIdx.x) * G + g, last_rg);
        slice = __builtin_amdgcn_make_buffer_rsrc((void *)(Wt + ((size_t)rg * T + t0) * 1024), 0, nv * 1024, 0x00020000);
    };
    auto load_slot = [&](int i) { return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(slice, lane16, i * 1024, kNonTemporal)); };
    auto mma_slot = [&](int i, const u32x4 &av, f32x4 &acc, int live_mask) {
        const int m = (i < nv) ? live_mask : 0;              // all ones or zero, wavefront-uniform
        const int addr = (boff + (t0 + i) * bstride) & m;
        const u32x4 bv = *(const u32x4 *)(smem + addr);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                      acc, 0, 0, 0);
    };
    // ---- the split activation goes straight to LDS (the producer kernel already wrote it in B layout).  Everything that the
    // prologue and the first epilogue need is requested ahead of the weights (loads return in order), and the barrier at the end
    // orders LDS only: the MFMAs start on the first tiles while the rest of the window is on its way.
    const uint32_t real_bytes = (uint32_t)(K >> 3) * NC * 16, all_bytes = (uint32_t)T * 64 * NC;
    for (uint32_t p = wave * 1024; p < real_bytes; p += 8192)  // (the last piece runs on into the slice sums' place)
        to_lds<16>(in_s + min(p + lane16, real_bytes - 16), smem + 16 + p);
    __builtin_amdgcn_sched_barrier(0);
    const MvArgs &a = late_args<decltype(&k_mv1<EPI, KS, NS>)>();
    NormPart np;
    if (EPI != EPI_RESID) np = mv_norm_load(a);
    // the residual values of the first round's row group (R <= 5: two passes) and their gains, to LDS: wavefronts 0, 1 and 2.  Used where
    // it is the only round; the epilogues of several rounds read their own.  (Left out there: 1024 row groups, depth 4096 22.8 / 22.9 us.)
    auto *resid = (__attribute__((address_space(3))) float *)nscratch;
    if (EPI == EPI_RESID && G == 1 && wave < 3) {
        const int row = min(16 * min((int)blockIdx.x, last_rg) + col, a.O - 1);
        const float *from = wave < 2 ? a.out_f32 + (size_t)min(4 * wave + kg, R - 1) * a.ld_out + row : a.gain_next + row;
        to_lds<4>(from, nscratch + 64 * wave);
    }
    __builtin_amdgcn_sched_barrier(0);
    set_slice(0);
#pragma unroll
    for (int u = 0; u < NS; ++u) buf[u] = load_slot(u);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 4) ((uint32_t *)smem)[tid] = 0u;
    if (EPI == EPI_QKV) {
        // behind the window, to LDS: the rotary rows (wavefront w: elements 64 w .. of [row][d/2]), and a word of each line that the
        // epilogues of this workgroup's rounds will write values into (wavefront s: round s; see mv_value_line)
        const int half = a.head_dim >> 1, lg_half = __builtin_ctz(half), i = min(tid, R * half - 1);
        if (64 * wave < R * half) {
            const uint32_t at = ((uint32_t)mv_rope_pos(a, i >> lg_half) << lg_half) + (i & (half - 1));
            to_lds<4>(a.cos_tab + at, rot + 64 * wave);
            to_lds<4>(a.sin_tab + at, rot + mv1_rot_pitch(R, a.head_dim) + 64 * wave);
        }
        if (G == 1 && wave < S) {
            const uint32_t *line = mv_value_line(a, min(wave * W + (int)blockIdx.x, last_rg), lane);
            if (line) to_lds<4>(line, touched);
        }
    }
    // (the activation has arrived: what was requested after it may be on its way)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NS) : "memory");
    if (EPI != EPI_RESID)
        mv_norm_finish(a, np, rs, nscratch);
    else
        lds_barrier();
    if ((K & 31) != 0) {  // zeros past the real depth
        for (uint32_t i = real_bytes + tid * 16; i < all_bytes; i += 8192) *(u32x4 *)(smem + 16 + i) = u32x4{0u, 0u, 0u, 0u};
        lds_barrier();
    }

    auto round = [&](int seg, auto LAST) {
        constexpr bool kLast = decltype(LAST)::value;
        const int rg = (seg * W + (int)blockIdx.x) * G + g;
        const bool live = rg <= last_rg;
        const int live_mask = live ? -1 : 0;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};

        const int nb16 = (n + NS - 1) / NS;
        // (As compiled, a few reloads of a block follow the MFMA that frees their slot and half of them go out behind the last one.  Pinning
        // each behind its MFMA with scheduling barriers measured the same.)
        for (int b = 0; b + 1 < nb16; ++b) {
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_slot(b * NS + u, buf[u], acc, live_mask);
                buf[u] = load_slot((b + 1) * NS + u);
            }
        }
        if (!kLast) {
            // the window rolls on into the next round's row group: the stream never drains
            // (The last block's addresses are the same in every round.  Kept in registers from round to round, two a slot, they spilled up
            // to eight, whose reloads waited for the window: LM head of depth 3840 43.3 us, 37.8 with the block's number opaque and no
            // register spilled in any instance; depth 7680 83.3 / 72.2, q|k|v of 960 row groups of depth 8192 42.2 / 40.9.)
            int last_block = (nb16 - 1) * NS;
            asm volatile("" : "+s"(last_block));
            set_slice(seg + 1);
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                mma_slot(last_block + u, buf[u], acc, live_mask);
                buf[u] = load_slot(u);
            }
        } else {
#pragma unroll
            for (int u = 0; u < NS; ++u) mma_slot((nb16 - 1) * NS + u, buf[u], acc, live_mask);
        }

        // ---- end of the row group: every wavefront parks its NC result columns in LDS; one
        // wavefront per row group adds terms and K slices and runs the epilogue
        float *rp = red + (size_t)(seg & 1) * (8 * 16 * NC);
        if (col < NC) *(f32x4 *)(rp + (wave * NC + col) * 16 + 4 * kg) = acc;
        if (EPI == EPI_QKV && seg == 0)  // (the rotary rows have arrived)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLast ? 0 : NS) : "memory");
        lds_barrier();  // (the next round's tile loads stay in flight)
        if (!live || ks != 0) return;
        // Slice sums are added per term in groups of kgroup slices (slice order), the three terms of a group are combined, and the
        // groups are added in order.
        const int kgroup = a.kgroup, ss = NC * 16;  // ss: from one slice to the next
        const float *w0 = rp + g * KS * ss;
        if constexpr (!kLast) {
            // (rolled loops: this runs in one wavefront per row group while the load window stays in registers)
            mv_epilogue<EPI>(a, rg, lane, rs, EPI == EPI_QKV ? rot : nullptr, [&](int r, int j) {
                const float *w = w0 + 3 * r * 16 + j;
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
            return;
        }
        // (the last round: the window's registers are free, all slice sums are read at once)
        auto y_last = [&](int r, int j) {
            const float *w = w0 + 3 * r * 16 + j;
            float v[KS][3];
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int t = 0; t < 3; ++t) v[k][t] = w[k * ss + 16 * t];
            float y = 0.f, sum[3];
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const bool first = (k & (kgroup - 1)) == 0;  // (a power of two)
#pragma unroll
                for (int t = 0; t < 3; ++t) sum[t] = first ? v[k][t] : sum[t] + v[k][t];
                if (((k + 1) & (kgroup - 1)) == 0) {
                    const float gs = (sum[0] + sum[1]) + sum[2];
                    y = k < kgroup ? gs : y + gs;
                }
            }
            return y;
        };
        if constexpr (EPI == EPI_RESID) {
            Residuals<2> X;
            if (G == 1 && S == 1)
                X = Residuals<2>{{resid[lane], resid[64 + lane]}, resid[128 + lane]};
            else
                X = mv_residuals<2>(a, rg, lane);
            mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_last, 0, 1, X);
        } else {
            mv_epilogue<EPI>(a, rg, lane, rs, EPI == EPI_QKV ? rot : nullptr, y_last);
        }
    };
    for (int seg = 0; seg + 1 < S; ++seg) round(seg, std::false_type());
    round(S - 1, std::true_type());
}

template <int EPI, int KS, int NS>
static hipError_t launch_mv1_t(const MvArgs &a, int grid, size_t lds, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_mv1<EPI, KS, NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(kMvMaxLds + kMv1MoreLds));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    return launch_maybe_timed(k_mv1<EPI, KS, NS>, dim3(grid), dim3(512), lds + kMv1MoreLds, s, (const unsigned char *)a.Wt,
                              (const unsigned char *)a.in_s, a.T, a.K, a.R, a.n_rg, a.n_wg, a.S, a);
}

// Workgroups of k_mv1 that share a compute unit, by all that a launch asks for.  (Two planned where one fits make two uneven rounds: gate/up of 384
// row groups, depth 12576, one row 31.3 us against 26.6; 512, depth 5984, two rows 20.7 against 18.1.)
static int mv1_per_unit(size_t lds) { return std::max(1, std::min(2, (int)((160 * 1024) / (lds + kMv1MoreLds)))); }
// Work split: KS wavefronts per row group, W workgroups, S rounds, chosen so that every
// workgroup gets the same number of row groups (a weight stream is only as fast as its
// slowest wavefront) with at most 16 wavefronts per compute unit.
struct Mv1Plan {
    int ks, W, S;
};
static Mv1Plan mv1_plan(const MvArgs &a, int n_cu, int ks_override, int wg_override) {
    const int max_wg = n_cu * mv1_per_unit(mv1_lds_bytes(a.K, a.R, a.head_dim));
    // Always 8 K slices per row group (unless a tuning run overrides it): the slice boundaries and
    // the order in which slice sums are added define a row's result bit for bit, and the block kernel
    // for 6-16 rows uses the same ones, so that a token's logits do not depend on how many rows
    // share its pass (speculative output == plain greedy output exactly, not just up to rounding).
    Mv1Plan p{8, 1, 1};
    double best_score = 1e30;
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
                p = Mv1Plan{ks, W, S};
            }
        }
    }
    if (wg_override > 0) {
        const int G = 8 / p.ks;
        p.W = wg_override;
        p.S = (a.n_rg + G * p.W - 1) / (G * p.W);
    }
    return p;
}

static hipError_t launch_mv1(int epi, MvArgs a, int n_cu, int ks_override, int wg_override, hipStream_t s) {
    const size_t lds = mv1_lds_bytes(a.K, a.R, a.head_dim);
    if (lds > kMvMaxLds) return hipErrorInvalidValue;
    const Mv1Plan p = mv1_plan(a, n_cu, ks_override, wg_override);
    const int best_ks = p.ks, grid = p.W;
    a.S = p.S;
    a.n_wg = p.W;
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
// Residual values are requested together, before the count that decides who adds the parts; read one by one in the last wavefront's
// epilogue, a dependent load per pass of four rows, they made up to 7 us of a launch (64 bulk rows o_proj 24.1 / 19.6, down_proj 36.5 /
// 29.5; 31 rows down_proj 27.7 / 25.6; 13B, 31 rows o_proj 22.3 / 19.0, 64 bulk rows down_proj 44.7 / 37.6).
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
            np64 = mv_norm64_load(a);
        else if (NCB <= 3)
            np = mv_norm_load(a);
        else
            np32 = mv_norm32_load(a);
    }
    if (EPI == EPI_QKV) {  // the lines this wavefront's epilogue will write values into (see mv_value_line)
        const uint32_t *line = mv_value_line(a, min(rgb + wave, a.n_rg - 1), lane);
        if (line) to_lds<4>(line, touched + wave * 64);
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
                const unsigned char *from = src[i] + (size_t)min(voff[i], vend[i]);
                if (wave + 8 * i < KT * RGS)  // (wavefront-uniform)
                    to_lds<16, true>(from, dst + i * 8192);
                else
                    to_lds<16>(from, dst + i * 8192);
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
        else if (NCB <= 3)
            mv_norm_finish(a, np, rs, nscratch);
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
    constexpr int kPasses = (NCB == 8 ? 64 : NCB > 3 ? 32 : 16) / 4;  // of an epilogue of as many rows as the columns hold
    if (KSP == 1) {
        if (!live) return;
        if constexpr (EPI == EPI_RESID)
            mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_local, 0, 1, mv_residuals<kPasses>(a, rg, lane));
        else
            mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_local);
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
    // (the residual values are requested with the stores on their way, in case this wavefront is the last)
    Residuals<EPI == EPI_RESID ? kPasses : 1> X;
    if (EPI == EPI_RESID) X = mv_residuals<EPI == EPI_RESID ? kPasses : 1>(a, rg, lane);
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
    auto y_sum = [&](int r, int j) { return dm[r * 16 + j]; };
    if constexpr (EPI == EPI_RESID)
        mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_sum, 0, 1, X);
    else
        mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y_sum);
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
// the wavefronts between the ends of a round.  Slices of W and B are buffers, whose loads cost no address arithmetic and past whose
// ends nothing is read; residual values are requested ahead of the weights.  us, before / now: 7B, 9 rows o_proj 10.2 / 9.7, down_proj
// 23.4 / 22.2; 32 bulk rows q|k|v 25.0 / 23.8, o_proj 13.9 / 13.0; 13B, 9 rows o_proj 16.0 / 14.7, gate/up 54.6 / 53.4; 16 rows o_proj
// 18.9 / 17.6.
// (the slice sums of two rounds, where LDS holds them: one barrier a round)
template <int NCB, int RG>
constexpr bool kMvrTwoBuffers = 2 * 8 * RG * 16 * NCB * 16 * 4 <= 150 * 1024;
template <int EPI, int NCB, int RG, int NS>
__global__ __launch_bounds__(512) void k_mvR(const unsigned char *Wt, const unsigned char *in_s, int T, int K, int NC, int n_rg, int W, int S,
                                              MvArgs rest) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NCP = 16 * NCB;                 // columns as computed
    constexpr int kRed = 8 * RG * NCP * 16;       // floats of one round's slice sums
    constexpr bool kTwo = kMvrTwoBuffers<NCB, RG>;
    float *red = (float *)smem;                   // [kTwo ? 2 : 1][8 slices][RG][NCP][16]
    float *rs = red + (kTwo ? 2 : 1) * kRed;      // [32]
    float *nscratch = rs + 32;                    // [1024]
    constexpr bool kNorm = EPI != EPI_RESID;
    const int tid = threadIdx.x, lane = tid & 63;
    const int ks = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kg = lane >> 4;
    const int n = (T + 7) >> 3;                // k tiles of a slice
    const int t0 = min(ks * n, T - 1);
    const int nv = max(0, min(n, T - ks * n)); // ... of which exist
    const int last_rg = n_rg - 1;
    // Slices of W and of B as buffers: steps past a slice's end, and lanes past the real depth in a ragged last tile, read nothing
    // and get zeros (columns past the last read what lies behind: results nobody reads).
    const uint32_t lane16 = lane * 16, b_at = (uint32_t)(kg * NC + col) * 16, b_step = 64u * NC;
    const uint32_t b_end = (uint32_t)(K >> 3) * NC * 16;
    const __amdgpu_buffer_rsrc_t b_slice =
        __builtin_amdgcn_make_buffer_rsrc((void *)(in_s + (size_t)t0 * b_step), 0, min(nv * b_step, b_end - t0 * b_step), 0x00020000);
    __amdgpu_buffer_rsrc_t slice[RG];
    u32x4 A[NS][RG], B[NS][NCB];
    auto load_step = [&](int i, u32x4(&Av)[RG], u32x4(&Bv)[NCB]) {
#pragma unroll
        for (int g = 0; g < RG; ++g)
            Av[g] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(slice[g], lane16, i * 1024, kNonTemporal));
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            Bv[cb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(b_slice, b_at + 256 * cb, i * b_step, 0));
    };
    auto set_slices = [&](int seg) {
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            const int rg = min((seg * W + (int)blockIdx.x) * RG + g, last_rg);
            slice[g] = __builtin_amdgcn_make_buffer_rsrc((void *)(Wt + ((size_t)rg * T + t0) * 1024), 0, nv * 1024, 0x00020000);
        }
    };
    // (the norm partials go out first; the scales are read by the epilogue only, so an LDS-only barrier will do)
    const MvArgs &a = late_args<decltype(&k_mvR<EPI, NCB, RG, NS>)>();
    constexpr int share = 8 / RG;  // wavefronts per row group in the epilogue
    constexpr int kPasses = ((NCB <= 3 ? 16 : 32) / 4 + share - 1) / share;  // a wavefront's share of an epilogue of up to 16 / 32 rows
    const int eg = min(ks / share, RG - 1);  // this wavefront's row group there
    NormPart np;
    NormPart32 np32;
    if (kNorm) {
        if (NCB <= 3)  // (up to 16 rows: row pitch 16)
            np = mv_norm_load(a);
        else
            np32 = mv_norm32_load(a);
    }
    constexpr bool kAhead = EPI == EPI_RESID && RG * NCB < 15;  // (no registers left in the largest)
    Residuals<kPasses> X;
    if (kAhead) X = mv_residuals<kPasses>(a, min((int)blockIdx.x * RG + eg, last_rg), lane, ks - eg * share, share);
    __builtin_amdgcn_sched_barrier(0);
    set_slices(0);
#pragma unroll
    for (int u = 0; u < NS; ++u) load_step(u, A[u], B[u]);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t v_line[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
        // the lines the epilogues of this workgroup's rounds will write values into (wavefront s: round s)
        v_line[g] = 0u;
        if (EPI == EPI_QKV && ks < S) {
            const uint32_t *line = mv_value_line(a, min((ks * W + (int)blockIdx.x) * RG + g, last_rg), lane);
            if (line) v_line[g] = *line;
        }
    }
    if (kNorm) {
        if (NCB <= 3)
            mv_norm_finish(a, np, rs, nscratch);
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
    for (int seg = 0; seg < S; ++seg) {
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
        if (seg + 1 < S) {
            // the window rolls on into the next round's row groups: the stream never drains
            set_slices(seg + 1);
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
        if (EPI == EPI_QKV && seg == 0)
#pragma unroll
            for (int g = 0; g < RG; ++g) keep_alive(v_line[g]);
        const int g = ks / share;
        const int rg = (seg * W + (int)blockIdx.x) * RG + g;
        if (g < RG && rg <= last_rg) {
            auto y = [&](int r, int j) {
                // (the order of k_mv1: per term in groups of kgroup slices, the terms of a group combined, groups in order)
                const int kgroup = a.kgroup, NT = block_terms(a.RL);
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
            };
            if constexpr (EPI == EPI_RESID) {
                if (!kAhead || seg > 0) X = mv_residuals<kPasses>(a, rg, lane, ks - g * share, share);
                mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y, ks - g * share, share, X);
            } else {
                mv_epilogue<EPI>(a, rg, lane, rs, nullptr, y, ks - g * share, share);
            }
        }
    }
}

// Steps in flight per wavefront: what 256 registers hold beside the accumulators (3 x 6 tiles: two steps, three spill).
constexpr int mvr_steps(int ncb, int rg) {
    const int n = ((rg * ncb >= 18 ? 144 : rg * ncb >= 8 ? 184 : 200) - 4 * rg * ncb) / (4 * (rg + ncb));
    return n > 10 ? 10 : n;
}

// Other depths for slices that the first one cuts badly.  (A step past a slice's end reads nothing and is not multiplied, but it is
// requested, and while it holds its place in the window fewer loads are in flight.)  us, 256 row groups, 9 rows, windows of 8 / 10 / 11 steps: 4 tiles
// 5.2 / 5.7 / 5.7, 16 tiles (7B o_proj) 9.8 / 10.3 / 10.5, 20: 12.0 / 11.6 / 11.8, 24: 13.3 / 14.0 / 14.5, 28: 15.4 / 15.2 / 15.5, 40: 20.1 /
// 20.1 / 20.4, 43 (7B down_proj): 22.1 / 22.3 / 21.6.  Eleven steps only for one row group and up to two column blocks.
constexpr int mvr_other_steps(int ns) { return ns > 8 ? 8 : ns == 8 ? 7 : ns > 4 ? 4 : ns == 3 ? 2 : ns; }
constexpr int mvr_third_steps(int ncb, int rg) { return rg == 1 && ncb <= 2 ? 11 : mvr_steps(ncb, rg); }
static int mvr_walked(int n, int steps) { return (n + steps - 1) / steps * steps; }
// The depth that walks a slice of n tiles in the fewest steps.
static int mvr_depth(int n, int ncb, int rg) {
    const int a = mvr_steps(ncb, rg), b = mvr_other_steps(a), c = mvr_third_steps(ncb, rg);
    const int d = mvr_walked(n, a) <= mvr_walked(n, b) ? a : b;
    return mvr_walked(n, c) < mvr_walked(n, d) ? c : d;
}
// The steps of a slice as mvr_line prices them: as its constants were fitted, with the first two depths.  For one row group and up to two
// column blocks the price is that of eleven steps, and of eight up to 16 tiles.  us, k_mvN or more row groups / one row group in k_mvR, 6-10
// rows: short of 16 tiles at the shallower price, 3072 x 16 row groups 7.9-8.6 / 6.4-7.4, 4096 x 16 8.7-9.4 / 7.7-8.3; beyond them at the
// dearer one, 28672 x 256 40-43 / 47-54, 12288 x 184 17.4-19.2 / 19-23.6, 6144 x 88 11-12.4 / 10.4-12.9; 2560 x 640 12.2-12.7 / 14.3-15.
static int mvr_line_steps(int n, int ncb, int rg) {
    const int a = mvr_steps(ncb, rg), b = mvr_other_steps(a), c = mvr_third_steps(ncb, rg);
    if (c != a) return n > 16 ? mvr_walked(n, c) : std::min(mvr_walked(n, c), mvr_walked(n, b));
    return std::min(mvr_walked(n, a), mvr_walked(n, b));
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
    return launch_maybe_timed(k_mvR<EPI, NCB, RG, NS>, dim3(a.n_wg), dim3(512), lds, s, (const unsigned char *)a.Wt,
                              (const unsigned char *)a.in_s, a.T, a.K, block_terms(a.RL) * layout_rows(a.RL), a.n_rg, a.n_wg, a.S, a);
}
template <int EPI, int NCB, int RG>
static hipError_t launch_mvR_t(MvArgs a, int n_cu, hipStream_t s) {
    const int units = (a.n_rg + RG - 1) / RG;
    a.S = (units + n_cu - 1) / n_cu;
    a.n_wg = (units + a.S - 1) / a.S;
    a.kgroup = mv_slice_group(a, n_cu);
    constexpr int NS = mvr_steps(NCB, RG), NS2 = mvr_other_steps(NS), NS3 = mvr_third_steps(NCB, RG);
    switch (mvr_depth((a.T + 7) / 8, NCB, RG)) {
        case NS: return launch_mvR_ns<EPI, NCB, RG, NS>(a, s);
        case NS3 == NS ? -1 : NS3: return launch_mvR_ns<EPI, NCB, RG, NS3>(a, s);
        default: return launch_mvR_ns<EPI, NCB, RG, NS2>(a, s);
    }
}

// A line between small blocks and large ones: row groups per workgroup round for k_mvR short of it, 0 beyond.  Two things hang on
// it: which kernel exact blocks take (mvr_row_groups), and how bulk blocks of 32 rows add their sums (mvn_canon).
// It is where k_mvR broke even with the kernel that k_mvN replaces, by what one compute unit had to
// walk, in us per k tile, fitted to 709 sets of launch durations of both (rows 1-32 of both layouts, seven widths
// from 1024 to 8192, matrices of 6 to 1300 MB).  c: column blocks, 0.4 x those computed + 0.6 x the columns' own share.
//   k_mvR   3.7 + rounds x 8 slices x steps of a slice (mvr_line_steps) x (weights of 1, 2 or 3 row groups + c columns of B)
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
        const double us = 3.68 + (double)S * 8 * mvr_line_steps((a.T + 7) / 8, ncb, c) * (kWeights[c - 1] + cols * kColumns[c - 1]);
        if (us < best) {
            best = us;
            rg = c;
        }
    }
    return rg;
}
// Row groups per workgroup round for k_mvR, or 0: k_mvN.  From eleven exact (17 bulk) rows on, k_mvN takes the matrices that its
// workgroups of six row groups cover in one round with K whole (us, k_mvR / k_mvN, 7B gate/up: 16 rows 35.9 / 33.3, 21 rows 41.4 /
// 34.5, 26 rows 46.8 / 37.4; 9 rows 32.2 / 32.7); elsewhere what lies beyond the line.
// The line prices the predecessor of k_mvN, and steps past a slice's end as if they carried traffic, so it is not where today's two kernels
// break even (both timed at the 7B, 13B and 70B widths, 6-32 rows: profiles/block_projection_sweep.txt, third table).  Beyond it k_mvN is
// faster throughout (us, k_mvR / k_mvN: 7B, 31 rows down_proj 40.0 / 25.1, LM head 75.3 / 49.5; 13B, 24 rows gate/up 79.5 / 54.3).
// Short of it k_mvR is where the matrix is narrow or the rows few (7B, 9 rows q|k|v 20.0 / 22.9, o_proj 9.7 / 13.3), and k_mvN would be by up
// to 28 % in a strip along it (13B, 18 rows LM head 71.0 / 55.4, 9 rows gate/up 53.6 / 46.5, 21 rows q|k|v 41.0 / 33.5; 7B, 13 rows down_proj
// 26.3 / 21.9; 70B, 18 rows gate/up 183.9 / 156.6, 16 rows down_proj 90.7 / 73.7): 3.3 % over all launches of the table.  Exact blocks come
// out the same bits either way.
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

// Small blocks (in their own exact layout) whose whole activation fits in LDS ..
static bool mv_fits_mv1(const MvArgs &a) {
    return !(a.RL & kBulkLayout) && a.R <= kMvSmallRows && mv1_lds_bytes(a.K, a.R, a.head_dim) <= kMvMaxLds;
}
// .. take the single-pass kernel, but for two kinds of matrices where k_mvR is faster, in rounds of three row groups per compute
// unit.  (All figures: us, k_mv1 / k_mvR; gate/up, the others within 3 % of its ratios.)
//  * 513..768 row groups on 256 units, which it covers in one such round and k_mv1 in an uneven one and a half or two.  One row: depth
//    2048, 640 row groups 11.3 / 9.9; 4096, 520: 18.2 / 15.2, 768: 19.5 / 19.0; 5120, 768: 22.6 / 22.8; 8192, 640: 33.3 / 28.6; next to them
//    4096, 896: 20.9 / 22.7.  Where the activation leaves k_mv1 one workgroup a unit its rounds are even enough: three rows at depth
//    5120, 576: 17.6 / 18.9, 704: 20.5 / 21.4; 6144, 576: 20.2 / 21.8, 768: 25.6 / 26.0; two at 7168, 576: 22.7 / 24.3.  Not so at the depths that
//    k_mvR walks in full windows of eight: three rows at 4096, 544: 16.0 / 15.0, 768: 19.4 / 18.8; two at 8192, 544: 26.7 / 25.9, 768: 34.3 / 33.4.
//  * deep ones (8192 to 10240) whose rounds of three are nine tenths full: one row, 8192, 1536: 63.3 / 62.3, 3584: 140.8 / 136.1, two rows
//    145.8 / 135.7; 10240, 3584: 170.3 / 169.0; 12288, 1536: 89.5 / 91.8, 2304: 130.7 / 133.2.
// The bits are the same either way.
static bool mv_takes_mv1(const MvArgs &a, int n_cu, int ks_override) {
    if (!mv_fits_mv1(a) || ks_override == 16) return false;
    if (ks_override != 0) return true;
    const int per_round = 3 * n_cu, rounds = (a.n_rg + per_round - 1) / per_round;
    if (a.n_rg > 2 * n_cu && rounds == 1)
        return a.T > 128 && a.T < 256 && mv1_per_unit(mv1_lds_bytes(a.K, a.R, a.head_dim)) == 1;
    return !(a.T >= 256 && a.T <= 320 && a.n_rg > per_round && 10 * a.n_rg >= 9 * rounds * per_round);
}
static int mv_column_blocks(const MvArgs &a) { return (block_terms(a.RL) * layout_rows(a.RL) + 15) / 16; }

int mv_path_name(const MvArgs &a, int n_cu, char *out, int capacity) {
    if (mv_takes_mv1(a, n_cu, 0)) {
        const Mv1Plan p = mv1_plan(a, n_cu, 0, 0);
        return snprintf(out, (size_t)capacity, "mv1<rows %d, workgroups %d, rounds %d>", a.R, p.W, p.S);
    }
    const int ncb = mv_column_blocks(a), rg = mvr_row_groups(a, n_cu, ncb);
    if (rg == 0) return snprintf(out, (size_t)capacity, "mvN<columns %d, parts %d>", ncb, mvn_plan(a, n_cu, mvn_canon(a, n_cu, ncb)).ksp);
    const int units = (a.n_rg + rg - 1) / rg;
    return snprintf(out, (size_t)capacity, "mvR<columns %d, row groups %d, steps %d, rounds %d>", ncb, rg,
                    mvr_depth((a.T + 7) / 8, ncb, rg), (units + n_cu - 1) / n_cu);
}

int mv_split_slots(const MvArgs &a, int n_cu) {
    if (a.RL & kBulkLayout) return a.part_capacity;  // (bulk layouts: not needed by callers)
    if (mv_fits_mv1(a)) return 0;
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
        (bulk ? (lrows != 32 && lrows != 64) : (lrows != a.R || lrows > kMaxRows)) || a.head0 != 0 ||
        (epi != EPI_RESID && (!a.pss || a.n_pss < 1)))
        return hipErrorInvalidValue;
    if (mv_takes_mv1(a, n_cu, ks_override)) return launch_mv1(epi, a, n_cu, ks_override, wg_override, s);
    // exact layouts (up to 32 rows): 2-6 column blocks of three-term columns, the fixed
    // summation order; bulk layouts of 32 / 64 rows (prefill, candidate evaluation): 4 / 8 column blocks of
    // two-term columns
    const int ncb = mv_column_blocks(a);
    if ((a.rp == 16) != (ncb <= 3)) return hipErrorInvalidValue;  // (three column blocks: up to 16 rows)
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
