// Causal attention of a block of 17..64 rows over a bf16 cache on the matrix cores (prefill blocks and
// the blocks of candidate evaluation; paper Section 3.1: the verify / prefill pass processes its rows as
// one causal block).  One workgroup per (query head, range of cache slots): its four wavefronts take 16
// block rows each and share every 64-slot chunk of keys and values through LDS, so a chunk is read once
// for all 64 rows instead of once per group of rows.  The values come from a cache that stores eight slots of
// an element together, so they reach LDS as V^T with plain 16-byte copies.
//
// Arithmetic.  Scores: S^T = K Q^T with the fp32 query rows as three bf16 terms (the products are
// exact, the sums fp32).  The transposed form leaves a row's scores in one lane column, so its
// probabilities are, without any data movement, the B operand of O^T = V^T P^T, and the online-softmax
// rescale of O^T is per lane.  Probabilities enter that product as two bf16 terms (relative error
// 2^-17; the values they weight are bf16).  Rows of up to 16-row blocks never come here: their results
// must not depend on how many rows share a pass, and they keep the one fp32 code path that guarantees it.
#include <math.h>

#include "swift_device.h"
#include "swift_kernels.h"

namespace swift {

namespace {

__device__ inline bf16x8 pack_bf16x8(const uint16_t (&v)[8]) {
    u32x4 u;
    u.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
    u.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
    u.z = (uint32_t)v[4] | ((uint32_t)v[5] << 16);
    u.w = (uint32_t)v[6] | ((uint32_t)v[7] << 16);
    return __builtin_bit_cast(bf16x8, u);
}

// What bounds it: a wavefront's 80 matrix instructions per 64-slot chunk (1280 clocks) and the vector arithmetic around them
// (softmax, conversions) hardly overlap, ~3500 clocks a chunk.  Hence hardware bf16 conversions, one fused multiply-add
// per exponent, masks only in the chunk where a range ends, contiguous loads elsewhere and 16-byte stores: 7B, 512-row
// macro blocks, 27 us + 10 us of merging -> 22 us at 512 slots, 69 + 13 -> 64 at 2048.
//
// Lane layout of v_mfma_f32_16x16x32_bf16 (C = A B): lane = 16 g + col.
//   A (16 x 32): row col,    k = 8 g .. 8 g + 7        B (32 x 16): column col, k = 8 g .. 8 g + 7
//   C (16 x 16): column col, rows 4 g .. 4 g + 3
// Scores of one half chunk (32 slots) are two MFMA tiles tt = 0, 1; tile row 4 g + i is slot
// 8 g + 4 tt + i of the half, so that a lane's eight probabilities of the half are slots 8 g .. 8 g + 7:
// the k range of its B operand in the second product.
// A prompt macro block (a.sub_rows = 64) is one launch too: blockIdx.z stands for the sub-block, which is treated as a block
// of its own whose partial results sit at the macro block's row numbers.  Later sub-blocks reach further back and take longer,
// so the order in which they are handed out is theirs from the last one on (they start first, the short ones fill what is left); where
// all workgroups are resident at once, two to a compute unit, only the first half is handed out so and the second from the
// first sub-block on, which pairs long ones with short ones (7B, 1024-row macro blocks over 1024-3072 slots: 95.8 us on average in
// ascending order, 86.5).
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_block(AttnArgs am, int chunk, int paired) {
    constexpr int DC = D / 32;   // k steps of a score tile
    constexpr int DT = D / 16;   // 16-row tiles of O^T
    constexpr int PPR = D / 8;   // 16-byte pieces per cache row
    constexpr int NPC = PPR / 4; // pieces per thread, per chunk and matrix (64 slots, 256 threads)
    constexpr int KP = D + 8;    // LDS pitch of a key row (elements)
    constexpr int VP = 64 + 8;   // LDS pitch of a row of V^T
    __shared__ __align__(16) uint16_t Ks[64 * KP];
    __shared__ __align__(16) uint16_t Vt[D * VP];

    AttnArgs a = am;
    const int n_sub = gridDim.z, zb = blockIdx.z, first = paired ? (n_sub + 1) / 2 : n_sub;
    const int sub = zb < first ? n_sub - 1 - zb : zb - first;
    const int row_base = sub * 64;  // first row of this sub-block in the macro block
    if (am.sub_rows) {
        a.rows = min(64, am.rows - row_base);
        a.n_ctx = am.n_ctx + row_base;
        a.q = am.q + (size_t)sub * am.sub_q;
        if (am.out_s) a.out_s = am.out_s + (size_t)sub * am.sub_out_s;
    }
    const int head = blockIdx.x, sp = blockIdx.y, n_split = gridDim.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, g = lane >> 4;
    const int nq = a.n_q_heads, kvh = head / (nq / a.n_kv_heads);
    const int lo = sp * chunk;
    const int hi_all = min(a.n_ctx + a.rows - 1, lo + chunk);  // end of the longest row's range here
    if (hi_all <= lo) return;
    const uint16_t *kc = (const uint16_t *)a.kcache + (size_t)kvh * a.max_seq * D;
    const uint16_t *vt = (const uint16_t *)a.vcache + (size_t)kvh * a.nb32 * D * 32;
    const int row = 16 * wave + col;
    const int lim = row < a.rows ? a.n_ctx + row : 0;  // rows past the block take part in nothing
    const int tile_lim = a.n_ctx + min(16 * wave + 15, a.rows - 1);
    const bool tile_live = 16 * wave < a.rows;

    bf16x8 qop[DC][3];
    {
        const float *qp = a.q + ((size_t)min(row, a.rows - 1) * nq + head) * D + 8 * g;
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            uint16_t h[8], m[8], l[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) split3(qp[32 * c + j], h[j], m[j], l[j]);
            qop[c][0] = pack_bf16x8(h);
            qop[c][1] = pack_bf16x8(m);
            qop[c][2] = pack_bf16x8(l);
        }
    }

    u32x4 kr[NPC], vr[NPC];
    // Keys: piece p = (slot p / PPR, 8 elements).  Slots past the longest row's range are replaced by its last
    // slot (an unwritten slot may hold anything).  Values come from the cache that groups eight slots per element
    // (kv_vt_index): piece p = (8-slot group p / D of the chunk, element p % D); slots past the range are zeroed in the
    // registers (0 x NaN is NaN in the second product).
    // A chunk that lies wholly inside the range is two runs of contiguous 16-byte pieces.
    auto load_chunk = [&](int k0) {
        if (k0 + 64 <= hi_all) {
            const u32x4 *kp = (const u32x4 *)(kc + (size_t)k0 * D), *vp = (const u32x4 *)(vt + (size_t)k0 * D);
#pragma unroll
            for (int u = 0; u < NPC; ++u) {
                kr[u] = (kp + 256 * u)[tid];
                vr[u] = (vp + 256 * u)[tid];
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < NPC; ++u) {
            const int p = tid + 256 * u, key = p / PPR, dj = p - key * PPR;
            kr[u] = *(const u32x4 *)(kc + (size_t)min(k0 + key, hi_all - 1) * D + 8 * dj);
            const int sg = p / D, dd = p - sg * D;
            const int grp = min((k0 >> 3) + sg, 4 * a.nb32 - 1);
            u32x4 v = *(const u32x4 *)(vt + ((size_t)grp * D + dd) * 8);
            const int n_ok = hi_all - (k0 + 8 * sg);  // slots of this piece inside the range
            if (n_ok < 8) {
                uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j >= n_ok) w[j >> 1] &= (j & 1) ? 0x0000ffffu : 0xffff0000u;
                v = u32x4{w[0], w[1], w[2], w[3]};
            }
            vr[u] = v;
        }
    };
    // V^T in LDS: element (dd, key) at row dd, column 8 ((key / 8) ^ (dd / 8 & 7)) + key % 8
    auto store_chunk = [&]() {
#pragma unroll
        for (int u = 0; u < NPC; ++u) {
            const int p = tid + 256 * u, key = p / PPR, dj = p - key * PPR;
            *(u32x4 *)(Ks + key * KP + 8 * dj) = kr[u];
            const int sg = p / D, dd = p - sg * D;
            *(u32x4 *)(Vt + dd * VP + 8 * (sg ^ ((dd >> 3) & 7))) = vr[u];
        }
    };

    const float scale = 1.0f / sqrtf((float)D), c_exp = scale * 1.4426950408889634f;
    const int first_lim = a.n_ctx + 16 * wave;  // range of the tile's first row
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

    load_chunk(lo);
    for (int k0 = lo; k0 < hi_all; k0 += 64) {
        store_chunk();
        __syncthreads();
        if (k0 + 64 < hi_all) load_chunk(k0 + 64);
        if (tile_live && k0 < tile_lim) {  // wavefront-uniform: some row of the tile reaches this chunk
            // (scores stay unscaled; the scale and log2 e meet them in the exponent: e^(scale (s - max)) = 2^(c s - c max))
            float s[2][2][4];
            float mx = -INFINITY;
            const bool ragged = k0 + 64 > first_lim;  // wavefront-uniform: some row's range ends inside this chunk
            // (the four tiles side by side: four independent chains of matrix instructions)
            f32x4 acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                bf16x8 av[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    av[q] = __builtin_bit_cast(
                        bf16x8, *(const u32x4 *)(Ks + (32 * (q >> 1) + 8 * (col >> 2) + 4 * (q & 1) + (col & 3)) * KP + 8 * g + 32 * c));
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[q], qop[c][t], acc[q], 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int hf = q >> 1, tt = q & 1;
                    if (ragged && k0 + 32 * hf + 8 * g + 4 * tt + i >= lim) acc[q][i] = -INFINITY;
                    s[hf][tt][i] = acc[q][i];
                    mx = fmaxf(mx, acc[q][i]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float mn = fmaxf(m_run, mx);
            const float ms = mn == -INFINITY ? 0.f : mn;  // nothing live yet: every exponential below is 0
            const float mc = ms * c_exp;
            // (not 2^(c m_run - mc): the rounding of mc would stay in it, a factor beside 1 in every chunk with the same sign)
            const float corr = __builtin_amdgcn_exp2f((m_run - ms) * c_exp);
            float ps = 0.f;
            bf16x8 phi[2], plo[2];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                f32x8 p;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    p[j] = __builtin_amdgcn_exp2f(fmaf(s[hf][j >> 2][j & 3], c_exp, -mc));
                    ps += p[j];
                }
                split2(p, phi[hf], plo[hf]);
            }
            l_run = l_run * corr + ps;
            m_run = mn;
            if (!__all(corr == 1.f)) {  // (most chunks leave every row's maximum where it is)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) o[dt] *= corr;
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                for (int d4 = 0; d4 < DT; d4 += 4) {
                    bf16x8 av[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int dd = 16 * (d4 + q) + col;
                        av[q] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(Vt + dd * VP + 8 * ((4 * hf + g) ^ ((dd >> 3) & 7))));
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[d4 + q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[q], phi[hf], o[d4 + q], 0, 0, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) o[d4 + q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[q], plo[hf], o[d4 + q], 0, 0, 0);
                }
        }
        __syncthreads();
    }
    // a row's sum is spread over its four lanes (the running maximum is common to them)
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    const int ns_row = (a.n_ctx + row + chunk - 1) / chunk;  // ranges this row reaches
    const bool mine = row < a.rows && sp < ns_row;
    const float inv = 1.0f / l_run;
    const int orows = a.out_s ? layout_rows(a.out_rows) : 0;
    if (mine && ns_row > 1 && g == 0) {
        const size_t base = ((size_t)(row_base + row) * nq + head) * n_split + sp;
        a.part_ml[base * 2] = m_run * scale;
        a.part_ml[base * 2 + 1] = l_run;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        const int e = head * D + 16 * dt + 4 * g;
        const f32x4 y = o[dt] * inv;
        uint32_t h[4], m[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = f32_to_bf16_rne_finite(y[i]);
            m[i] = f32_to_bf16_rne_finite(y[i] - __uint_as_float(h[i] << 16));
        }
        // (the lane with the even g ends up with eight elements' first terms, its neighbour with their second terms)
        const u32x4 u = join8(pack2(h[0], h[1]), pack2(h[2], h[3]), pack2(m[0], m[1]), pack2(m[2], m[3]));
        if (!mine) continue;
        if (ns_row == 1) {  // the row ends in the first range: write the result
            if (a.out) *(f32x4 *)(a.out + (size_t)row * nq * D + e) = y;
            if (a.out_s) *(u32x4 *)(a.out_s + ((size_t)(e >> 3) * (2 * orows) + 2 * row + (g & 1)) * 8) = u;
        } else {            // partial result of this range; k_attn_combine merges the ranges in order
            const size_t base = ((size_t)(row_base + row) * nq + head) * n_split + sp;
            *(f32x4 *)(a.part_o + base * D + 16 * dt + 4 * g) = o[dt];
        }
    }
}

}  // namespace

bool attn_block_applies(int dtype, const AttnArgs &a) {
    return dtype == BF16 && !a.tree && a.rows > kMaxRows && a.rows <= 64 && (a.head_dim == 64 || a.head_dim == 128);
}

hipError_t launch_attn_block(const AttnArgs &a, int n_cu, hipStream_t s) {
    const int n_sub = a.sub_rows ? (a.rows + 63) / 64 : 1;
    if (a.tree || a.rows < 1 || a.rows > 64 * n_sub || (a.sub_rows != 0 && a.sub_rows != 64) || n_sub > kMacroSub ||
        (a.sub_rows && a.out) || (a.head_dim != 64 && a.head_dim != 128) || a.n_ctx < 1 ||
        a.n_kv_heads < 1 || a.n_q_heads % a.n_kv_heads != 0 || a.n_ctx + a.rows - 1 > a.max_seq || (!a.out && !a.out_s) || (a.out_s && block_terms(a.out_rows) != 2) ||
        a.nb32 < (a.max_seq + 31) / 32 ||
        !a.part_o || !a.part_ml)
        return hipErrorInvalidValue;
    const int ctx = a.n_ctx + a.rows - 1;
    // ranges: about one workgroup per compute unit (a second one takes as much longer as it adds: 7B, 512 rows at 2048
    // slots 69 us in two ranges + 13 us to merge them, 73 us in one), at least two chunks each, and no more partial
    // results than the buffers hold (they are sized for kMaxRows rows times max_split ranges)
    int want = (n_cu + a.n_q_heads * n_sub - 1) / (a.n_q_heads * n_sub);
    const int cap = kMaxRows * a.max_split / a.rows;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    int chunk = ((ctx + want - 1) / want + 63) / 64 * 64;
    if (chunk < 128) chunk = 128;
    const int n_split = (ctx + chunk - 1) / chunk;
    if ((int64_t)n_split * a.rows > (int64_t)kMaxRows * a.max_split) return hipErrorInvalidValue;
    const dim3 grid(a.n_q_heads, n_split, n_sub), block(256);
    const int paired = a.n_q_heads * n_split * n_sub <= 2 * n_cu;
    if (a.head_dim == 128)
        hipLaunchKernelGGL(k_attn_block<128>, grid, block, 0, s, a, chunk, paired);
    else
        hipLaunchKernelGGL(k_attn_block<64>, grid, block, 0, s, a, chunk, paired);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_split == 1) return e;
    return launch_attn_combine(a, chunk, n_split, s);
}

}  // namespace swift
