// Attention of decode, draft and verify rows over a bf16 cache with heads of 64 or 128 on the matrix
// cores (paper Sections 3.1 and 4.2: a draft or plain decoding pass has one row, a verify pass the pending
// token and its k drafts as one causal block, dynamic verification the rows of a token tree).
//
// All rows of a block and all query heads of a kv head's group are the columns ("members") of one MFMA
// tile, so a workgroup reads every key/value chunk of its cache range once for up to 16 members -- once
// per block for a block of up to 16 rows on one kv head per query head.  The operands come straight from
// global memory in MFMA layout with 128-bit loads: the keys as stored, the values from a cache that holds
// eight slots of an element together (kv_vt_index), so nothing is transposed or staged on the way.
//
// What a row computes (the same for a row decoded alone, a row of a chain block and a row of a tree, bit for
// bit, because every step below is per member and its order does not depend on the other members):
//  * the row's prefix -- logical slots [0, P), P = its position -- is walked in chunks of 32 slots.  A
//    workgroup owns a range of the cache capacity fixed by the configuration alone; its wavefronts take the
//    range's chunks round-robin, each folding its chunks in order into a running (max, sum, weighted values)
//    with S^T = K Q^T and O^T += V^T P^T (queries and probabilities as two bf16 terms each: relative error
//    2^-17 against the 2^-9 of the bf16 keys and values; fp32 sums); the wavefronts' results are merged in
//    wavefront order, the ranges' in range order (by the last workgroup of a head, by one workgroup that walks them all, or by
//    k_attn_mfma_combine: the same bits);
//  * the row's own slot (its key and value, written to the cache by the projection kernel of the same pass)
//    is merged last, in fp32 vector arithmetic.  For a tree row the prefix beyond the committed slots is
//    the first candidates of the levels above it: one mapping for all rows, so tree rows share the loads
//    too, and only the own slot differs from row to row.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <type_traits>

#include "swift_device.h"
#include "swift_kernels.h"

namespace swift {

namespace {

constexpr int kAmPad = 4;         // floats of padding per member row of the merge area
constexpr int kDeviceScope = 16;  // cache policy sc1
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ inline bf16x8 am_pack(const uint16_t (&v)[8]) {
    u32x4 u;
    u.x = (uint32_t)v[0] | ((uint32_t)v[1] << 16);
    u.y = (uint32_t)v[2] | ((uint32_t)v[3] << 16);
    u.z = (uint32_t)v[4] | ((uint32_t)v[5] << 16);
    u.w = (uint32_t)v[6] | ((uint32_t)v[7] << 16);
    return __builtin_bit_cast(bf16x8, u);
}

// Logical slots [0, this) are launch row r's prefix; its own slot holds the row's key and value.
template <bool TREE>
__device__ inline int am_prefix_end(const AttnArgs &a, int r) {
    return TREE ? a.n_base + (int)a.tt.depth[(a.row_base + r) & (kMaxRows - 1)] : a.n_ctx - 1 + r;
}
template <bool TREE>
__device__ inline int am_own_slot(const AttnArgs &a, int r) {
    return TREE ? a.n_base + a.row_base + r : a.n_ctx - 1 + r;
}
// Cache slot of logical prefix slot p.  Tree rows: beyond the committed slots the prefix is the block's
// first row, then the first candidates of the levels in between.
template <bool TREE>
__device__ inline int am_phys(const AttnArgs &a, int p) {
    if (TREE && p >= a.n_base) return a.n_base + (int)a.tt.spine[(p - a.n_base) & (kMaxRows - 1)];
    return p;
}

__device__ inline float am_bf(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// q . k of a row's own slot, by one wavefront: lane l takes elements 2l, 2l+1 (+128 ...), then a butterfly.
__device__ inline float am_own_score(const float *q, const uint16_t *k, int d, int lane, float scale) {
    float s = 0.f;
    for (int e = 2 * lane; e < d; e += 128) {
        s = fmaf(q[e], am_bf(k[e]), s);
        s = fmaf(q[e + 1], am_bf(k[e + 1]), s);
    }
    return wave_sum(s) * scale;
}

// Merges the own slot (score s_own, value v_own) into the prefix's (max mn, sum ls, weighted value os) and
// normalises.  An empty prefix has mn = -inf, ls = os = 0.  (Of two products in a sum one is
// rounded: which one is spelt out, here and in am_fold.  The compiler's own choice hangs on the instance, and a row's bits would.)
__device__ inline float am_finish(float mn, float ls, float os, float s_own, float v_own) {
    const float m2 = fmaxf(mn, s_own);
    const float c1 = mn == -INFINITY ? 0.f : __expf(mn - m2);
    const float c2 = __expf(s_own - m2);
    return fmaf(c2, v_own, os * c1) / fmaf(ls, c1, c2);
}

// Folds the next range's (max m, sum l, weighted value o) into a running merge.  (A range's maximum is -inf only if its rows see
// nothing there.)
template <typename V>
__device__ inline void am_fold(float &mn, float &ls, V &os, float m, float l, const V &o) {
    const float m2 = fmaxf(mn, m);
    const float c1 = mn == -INFINITY ? 0.f : __expf(mn - m2);
    const float c2 = m == -INFINITY ? 0.f : __expf(m - m2);
    ls = fmaf(ls, c1, l * c2);
    if constexpr (std::is_same_v<V, float>) {
        os = fmaf(os, c1, o * c2);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) os[i] = fmaf(os[i], c1, o[i] * c2);
    }
    mn = m2;
}

__device__ inline void am_write(const AttnArgs &a, int row, int e, float y) {
    if (a.out) a.out[(size_t)row * a.n_q_heads * a.head_dim + e] = y;
    if (a.out_s) {
        uint16_t hi, mid, lo;
        split3(y, hi, mid, lo);
        const int ocode = a.out_rows ? a.out_rows : a.rows, orows = layout_rows(ocode), nt = block_terms(ocode);
        uint16_t *p = a.out_s + ((size_t)(e >> 3) * (nt * orows) + nt * row) * 8 + (e & 7);
        p[0] = hi;
        p[8] = mid;
        if (nt == 3) p[16] = lo;
    }
}

// Four consecutive elements, the first a multiple of four.
__device__ inline void am_write4(const AttnArgs &a, int row, int e, const f32x4 &y) {
    if (a.out) *(f32x4 *)(a.out + (size_t)row * a.n_q_heads * a.head_dim + e) = y;
    if (a.out_s) {
        uint16_t t[3][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) split3(y[i], t[0][i], t[1][i], t[2][i]);
        const int ocode = a.out_rows ? a.out_rows : a.rows, orows = layout_rows(ocode), nt = block_terms(ocode);
        uint16_t *p = a.out_s + ((size_t)(e >> 3) * (nt * orows) + nt * row) * 8 + (e & 7);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < nt) *(u32x2 *)(p + 8 * k) = u32x2{pack2(t[k][0], t[k][1]), pack2(t[k][2], t[k][3])};
    }
}

// Who merges a row's ranges: a launch of its own; the workgroup that arrives last; the one workgroup that walks them all.
enum AmMerge : int { kOwnLaunch, kLastWorkgroup, kSerial };

// Lane layout of v_mfma_f32_16x16x32_bf16 (C = A B): lane = 16 g + col.
//   A (16 x 32): row col,    k = 8 g .. 8 g + 7        B (32 x 16): column col, k = 8 g .. 8 g + 7
//   C (16 x 16): column col, rows 4 g .. 4 g + 3
// Scores of a 32-slot chunk are two tiles tt = 0, 1; tile row 4 g + i is slot 8 g + 4 tt + i of the chunk, so
// that a lane's eight probabilities are slots 8 g .. 8 g + 7: the k range of its B operand in O^T = V^T P^T.
//
// Workgroup (kv head, cache range sp, member tile z), NW wavefronts.  range: slots per workgroup, a multiple of 32.  hi_all: end of the
// longest prefix of the block.  lg_group: log2 of the query heads per kv head.  MERGE: who finishes the rows whose prefix spans several
// ranges: k_attn_mfma_combine, the workgroup that arrives last at their (kv head, member tile), or the only one there is (range: the
// whole cache; the ranges in which it walks it, a chunk per wavefront, are those of kLastWorkgroup).
//
// What bounds it at short contexts: a chain of latencies (launch, first loads, chunks, merge).  So the arguments of the first loads
// are the kernel's leading ones, which are in registers at its start, and nothing on the way to the first product waits for a load
// that is not part of it (100 slots, one row: 5.8 us, 4.5 without such waits and with the wavefronts' results read all at once).
template <int D, bool TREE, int NW, AmMerge MERGE>
__global__ __launch_bounds__(64 * NW, 2) void k_attn_mfma(const uint16_t *kcache, const uint16_t *vcache, const uint16_t *q_s, int max_seq,
                                                          int nb32, int range, int hi_all, int rows, int lg_group, AttnArgs a) {
    constexpr int DC = D / 32;      // k steps of a score tile
    constexpr int DT = D / 16;      // 16-row tiles of O^T
    constexpr int MP = D + kAmPad;  // pitch of a member's values in the merge area
    extern __shared__ __align__(16) float am_sh[];
    const int kvh = blockIdx.x, sp = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M_total = rows << lg_group;
    const int m0 = 16 * blockIdx.z;  // first member of this workgroup's tile; member m = (row m / group, head m % group)
    const int lo = sp * range, hi = min(hi_all, lo + range);
    const float scale = 1.0f / sqrtf((float)D);
    const uint16_t *kc = kcache + (size_t)kvh * max_seq * D;
    const uint16_t *vt = vcache + (size_t)kvh * nb32 * D * 32;

    // ---- operands of a chunk, straight from the cache in MFMA A layout
    // Chunks that lie below safe_end hold 32 prefix slots that sit where their numbers say: keys as stored,
    // values one 16-byte load per eight slots.  In the chunk in which the longest prefix ends, the keys of the
    // slots past it are replaced by its last slot's and their values by zeros (an unwritten slot may hold
    // anything, and 0 x NaN is NaN in an MFMA); a tree's chunks beyond the committed slots go slot by slot
    // through the mapping.
    const int safe_end = TREE ? min(a.n_base, hi_all) : hi_all;
    auto load_keys = [&](int c, u32x4(&kA)[2][DC]) {
        const bool plain = 32 * (c + 1) <= safe_end;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int slot = 32 * c + 8 * (col >> 2) + 4 * tt + (col & 3);
            const int ps = plain ? slot : am_phys<TREE>(a, min(slot, hi_all - 1));
            const uint16_t *kp = kc + (size_t)ps * D + 8 * g;
#pragma unroll
            for (int cc = 0; cc < DC; ++cc) kA[tt][cc] = *(const u32x4 *)(kp + 32 * cc);
        }
    };
    auto load_values = [&](int c, u32x4(&vA)[DT]) {
        const bool plain = 32 * (c + 1) <= safe_end;
        if (!TREE || plain) {
            const uint16_t *vp = vt + ((size_t)(4 * c + g) * D + col) * 8;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) vA[dt] = *(const u32x4 *)(vp + dt * (16 * 8));
        } else {
            // a tree's chunks beyond the committed slots: slot by slot through the mapping
            int ps[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) ps[j] = am_phys<TREE>(a, min(32 * c + 8 * g + j, hi_all - 1));
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                uint16_t e[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) e[j] = vt[((size_t)(ps[j] >> 3) * D + 16 * dt + col) * 8 + (ps[j] & 7)];
                vA[dt] = __builtin_bit_cast(u32x4, am_pack(e));
            }
        }
    };
    // (at their use, so that nothing waits for them earlier)
    auto mask_values = [&](int c, u32x4(&vA)[DT]) {
        if (TREE || 32 * (c + 1) <= safe_end) return;
        // the chunk in which the longest prefix ends: the slots past it are zeroed in the registers
        const int n_ok = hi_all - (32 * c + 8 * g);  // slots of this lane's eight that belong to the prefix
        const uint32_t m0 = n_ok >= 2 ? 0xffffffffu : n_ok == 1 ? 0x0000ffffu : 0u;
        const uint32_t m1 = n_ok >= 4 ? 0xffffffffu : n_ok == 3 ? 0x0000ffffu : 0u;
        const uint32_t m2 = n_ok >= 6 ? 0xffffffffu : n_ok == 5 ? 0x0000ffffu : 0u;
        const uint32_t m3 = n_ok >= 8 ? 0xffffffffu : n_ok == 7 ? 0x0000ffffu : 0u;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            vA[dt].x &= m0;
            vA[dt].y &= m1;
            vA[dt].z &= m2;
            vA[dt].w &= m3;
        }
    };

    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int c_end = (hi + 31) >> 5;
    u32x4 kA[2][DC], kB[2][DC], vA[DT];
    int c = (lo >> 5) + wave;
    // the first chunk's operands are requested before anything else, so that the set-up below (query operands,
    // own slots) runs while they are on their way
    if (c < c_end) {
        load_keys(c, kA);
        load_values(c, vA);
    }

    // query operands of this lane's member (column col of the tile): two bf16 terms per value (relative error 2^-17; the keys they
    // meet are bf16), written in this form by the projection kernel
    const int nq = a.n_q_heads, group = 1 << lg_group;
    const int mem = min(m0 + col, M_total - 1), mrow = mem >> lg_group, mhead = mem & (group - 1);
    bf16x8 qop[DC][2];
    {
        const uint16_t *qp = q_s + ((size_t)(mrow * nq + kvh * group + mhead) * 2) * D + 8 * g;
#pragma unroll
        for (int c = 0; c < DC; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t) qop[c][t] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(qp + t * D + 32 * c));
    }
    const int lim = m0 + col < M_total ? min(am_prefix_end<TREE>(a, mrow), lo + range) : 0;  // the prefix slots it sees here

    // ---- the rows' own slots (MERGE: any workgroup may be the one that finishes a row), requested before
    // the prefix is walked so that their latency is not paid at the end: what this wavefront's scores need (16 / NW members,
    // by whole wavefronts, lane l elements 2 l and 2 l + 1; reduced after the walk) and the value elements each thread will need
    // in the last phase, four in a row, each as the word that holds it.  (Trees with four wavefronts have no registers for the
    // second unit's, which are loaded when the unit is finished.  us a launch, spilling three / now, trees of 31: 64 / 8 heads of 128, 100
    // slots 9.9 / 9.2, 2048 slots 41.2 / 40.6; 32 heads, 60 slots 10.9 / 10.6.)
    constexpr int kUnits = (16 * D / 4 + 64 * NW - 1) / (64 * NW);  // units of four elements per thread in the last phase
    constexpr int kEarlyUnits = TREE && NW == 4 ? 1 : kUnits;
    constexpr int kScores = 16 / NW;
    constexpr int kArea = NW * 16 * (MP + 2);  // floats of the merge area; kSerial uses two in turn
    float *s_own = am_sh + (MERGE == kSerial ? 2 : 1) * kArea;
    const bool finishes = MERGE != kOwnLaunch || sp == 0;
    const int n_here = finishes ? min(16, M_total - m0) : 0;  // members that may be finished here
    // (member of score i: the last wavefronts have the fewest chunks to walk)
    auto own_member = [&](int i) { return NW - 1 - wave + NW * i; };
    auto unit_member = [&](int u) { return (tid + u * 64 * NW) / (D / 4); };
    auto unit_elem = [&](int u) { return 4 * ((tid + u * 64 * NW) % (D / 4)); };
    uint32_t v_own[kEarlyUnits][4];
    auto load_own_values = [&](int u, uint32_t(&v)[4]) {
        const int row = min(m0 + unit_member(u), M_total - 1) >> lg_group, own = am_own_slot<TREE>(a, row);
        const uint16_t *vp = vt + ((size_t)(own >> 3) * D + unit_elem(u)) * 8 + (own & 6);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = *(const uint32_t *)(vp + 8 * i);
    };
    float q_own[kScores][2];
    uint32_t k_own[kScores];
#pragma unroll
    for (int i = 0; i < kScores; ++i) {
        q_own[i][0] = q_own[i][1] = 0.f;
        k_own[i] = 0u;
        const int mm = own_member(i), row = (m0 + mm) >> lg_group, head = (m0 + mm) & (group - 1);
        if (mm >= n_here) continue;  // (wavefront-uniform)
        if (2 * lane < D) {
            const float *q = a.q + ((size_t)row * nq + kvh * group + head) * D + 2 * lane;
            q_own[i][0] = q[0];
            q_own[i][1] = q[1];
            k_own[i] = *(const uint32_t *)(kc + (size_t)am_own_slot<TREE>(a, row) * D + 2 * lane);
        }
    }
    if (finishes) {
#pragma unroll
        for (int u = 0; u < kEarlyUnits; ++u) load_own_values(u, v_own[u]);
    }

    // ---- this wavefront's chunks: every NW-th of the range, folded in order.  The keys of the next chunk are
    // requested before the current chunk's scores are computed (two sets of key registers, used in turn); the
    // value operands are dead once they are multiplied, so the next chunk's values are requested right after
    // the second product, into the same registers.
    auto step = [&](int c, const u32x4(&kCur)[2][DC], u32x4(&kNxt)[2][DC]) {
        const bool more = c + NW < c_end;  // wavefront-uniform
        if (more) load_keys(c + NW, kNxt);
        float s[8];
        float mx = -INFINITY;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cc = 0; cc < DC; ++cc)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kCur[tt][cc]), qop[cc][t], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int slot = 32 * c + 8 * g + 4 * tt + i;
                const float v = slot < lim ? acc[i] * scale : -INFINITY;
                s[4 * tt + i] = v;
                mx = fmaxf(mx, v);
            }
        }
        mx = column_reduce(mx, [](float x, float y) { return fmaxf(x, y); });
        const float mn = fmaxf(m_run, mx);
        const float ms = mn == -INFINITY ? 0.f : mn;  // nothing live yet: every exponential below is 0
        const float corr = __expf(m_run - ms);
        float ps = 0.f;
        uint16_t ph[8], pl[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float p = __expf(s[j] - ms);
            ps += p;
            const uint32_t hb = f32_to_bf16_rne_finite(p);
            ph[j] = (uint16_t)hb;
            pl[j] = (uint16_t)f32_to_bf16_rne_finite(p - __uint_as_float(hb << 16));
        }
        const bf16x8 phi = am_pack(ph), plo = am_pack(pl);
        l_run = l_run * corr + ps;
        m_run = mn;
        mask_values(c, vA);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            o[dt] *= corr;
            o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vA[dt]), phi, o[dt], 0, 0, 0);
            o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vA[dt]), plo, o[dt], 0, 0, 0);
        }
        if (more) load_values(c + NW, vA);
    };
    // ---- merge the wavefronts (in wavefront order): every wavefront parks its (max, sum, weighted values) of a range in LDS ..
    int area = 0;
    auto park = [&]() {
        float *wbase = am_sh + area + wave * (16 * (MP + 2));
        l_run = column_reduce(l_run, [](float x, float y) { return x + y; });
        if (g == 0) {
            wbase[col] = m_run;
            wbase[16 + col] = l_run;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) *(f32x4 *)(wbase + 32 + col * MP + 16 * dt + 4 * g) = o[dt];
    };
    // .. and a thread takes four elements of a member: the wavefronts' weights are worked out once for them
    auto merged = [&](int mm, int dd, float &mn, float &ls, f32x4 &os) {
        float mw[NW], lw[NW];
        f32x4 ow[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float *wb = am_sh + area + w * (16 * (MP + 2));
            mw[w] = wb[mm];
            lw[w] = wb[16 + mm];
            ow[w] = *(const f32x4 *)(wb + 32 + mm * MP + dd);
        }
        mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mn = fmaxf(mn, mw[w]);
        ls = 0.f;
        os = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float cw = mw[w] == -INFINITY ? 0.f : __expf(mw[w] - mn);
            ls += lw[w] * cw;
            os += ow[w] * cw;
        }
    };
    auto own_scores = [&]() {
#pragma unroll
        for (int i = 0; i < kScores; ++i) {
            const int mm = own_member(i);
            if (mm >= n_here) continue;  // (wavefront-uniform)
            const float sc = fmaf(q_own[i][1], am_bf((uint16_t)(k_own[i] >> 16)), fmaf(q_own[i][0], am_bf((uint16_t)k_own[i]), 0.f));
            const float sum = wave_sum(sc) * scale;
            if (lane == 0) s_own[mm] = sum;
        }
    };
    auto finish = [&](int u, int row, int qh, float mn, float ls, const f32x4 &os) {
        const int shift = (am_own_slot<TREE>(a, row) & 1) * 16;
        uint32_t late[4];
        if (u >= kEarlyUnits) load_own_values(u, late);
        f32x4 y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t v = u < kEarlyUnits ? v_own[u < kEarlyUnits ? u : 0][i] : late[i];
            y[i] = am_finish(mn, ls, os[i], s_own[unit_member(u)], am_bf((uint16_t)(v >> shift)));
        }
        am_write4(a, row, qh * D + unit_elem(u), y);
    };
    if constexpr (MERGE == kSerial) {
        // ---- one range after the other, a chunk of each per wavefront, folded in range order as they come.  The next range's chunk is on
        // its way while a range is merged: one barrier a range, which orders LDS only, and two merge areas in turn.
        float r_mn[kUnits], r_ls[kUnits];
        f32x4 r_os[kUnits];
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            r_mn[u] = -INFINITY;
            r_ls[u] = 0.f;
            r_os[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        own_scores();
        auto one = [&](int sp, const u32x4(&kCur)[2][DC], u32x4(&kNxt)[2][DC]) {
            m_run = -INFINITY;
            l_run = 0.f;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (c < c_end) step(c, kCur, kNxt);
            c += NW;
            park();
            lds_barrier();
#pragma unroll
            for (int u = 0; u < kUnits; ++u) {
                const int mm = unit_member(u), m = m0 + mm;
                if (mm >= 16 || m >= M_total) continue;
                if (sp * 32 * NW >= am_prefix_end<TREE>(a, m >> lg_group)) continue;  // the row's prefix does not reach this range
                float mn, ls;
                f32x4 os;
                merged(mm, unit_elem(u), mn, ls, os);
                am_fold(r_mn[u], r_ls[u], r_os[u], mn, ls, os);
            }
            area = kArea - area;
        };
        const int n = (hi_all + 32 * NW - 1) / (32 * NW);  // ranges
        for (int sp = 0; sp < n; sp += 2) {
            one(sp, kA, kB);
            if (sp + 1 < n) one(sp + 1, kB, kA);
        }
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int mm = unit_member(u), m = m0 + mm;
            if (mm >= 16 || m >= M_total) continue;
            finish(u, m >> lg_group, kvh * group + (m & (group - 1)), r_mn[u], r_ls[u], r_os[u]);
        }
        return;
    }
    for (; c < c_end; c += 2 * NW) {
        step(c, kA, kB);
        if (c + NW < c_end) step(c + NW, kB, kA);
    }
    // ---- then finish the rows whose prefix ends in the first range with their own slot, or leave the range's partial result
    park();
    own_scores();
    __syncthreads();
    const int n_split = gridDim.y;
    const __amdgpu_buffer_rsrc_t part_o = __builtin_amdgcn_make_buffer_rsrc(a.part_o, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t part_ml = __builtin_amdgcn_make_buffer_rsrc(a.part_ml, 0, 0x7fffffff, 0x00020000);
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const int mm = unit_member(u), dd = unit_elem(u), m = m0 + mm;
        if (mm >= 16 || m >= M_total) continue;
        const int row = m >> lg_group, qh = kvh * group + (m & (group - 1));
        const int pe = am_prefix_end<TREE>(a, row);
        const int nsr = (pe + range - 1) / range;  // ranges the row's prefix reaches (0: an empty prefix)
        if (sp >= max(nsr, 1)) continue;
        float mn, ls;
        f32x4 os;
        merged(mm, dd, mn, ls, os);
        if (nsr <= 1) {
            finish(u, row, qh, mn, ls, os);
        } else {
            const size_t slot = ((size_t)row * nq + qh) * n_split + sp;
            if constexpr (MERGE == kLastWorkgroup) {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, os), part_o, (uint32_t)((slot * D + dd) * 4), 0, kDeviceScope);
                if (dd == 0)
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(mn), __float_as_uint(ls)}, part_ml, (uint32_t)(slot * 8), 0,
                                                          kDeviceScope);
            } else {
                *(f32x4 *)(a.part_o + slot * D + dd) = os;
                if (dd == 0) {
                    a.part_ml[slot * 2] = mn;
                    a.part_ml[slot * 2 + 1] = ls;
                }
            }
        }
    }
    if constexpr (MERGE == kLastWorkgroup) {
        if (n_split == 1) return;
        // ---- the workgroup that arrives last merges the ranges, in range order.  Partial results are stored and loaded at device
        // scope (written through, read past this die's L2): once a workgroup's stores are acknowledged, a relaxed count
        // publishes them, and no cache is written back or invalidated.
        __shared__ int arrived;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int *counter = a.counters + kvh * (int)gridDim.z + (int)blockIdx.z;
        if (tid == 0) arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (arrived != n_split - 1) return;
        asm volatile("" ::: "memory");
        if (tid == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const int mm = unit_member(u), dd = unit_elem(u), m = m0 + mm;
            if (mm >= 16 || m >= M_total) continue;
            const int row = m >> lg_group, qh = kvh * group + (m & (group - 1));
            const int nsr = (am_prefix_end<TREE>(a, row) + range - 1) / range;
            if (nsr <= 1) continue;
            const uint32_t base = (uint32_t)(((size_t)row * nq + qh) * n_split);
            float mn = -INFINITY, ls = 0.f;
            f32x4 os = {0.f, 0.f, 0.f, 0.f};
            for (int s0 = 0; s0 < nsr; s0 += 8) {
                u32x2 ml[8];
                u32x4 ov[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t slot = base + (uint32_t)min(s0 + k, nsr - 1);
                    ml[k] = __builtin_amdgcn_raw_buffer_load_b64(part_ml, slot * 8, 0, kDeviceScope);
                    ov[k] = __builtin_amdgcn_raw_buffer_load_b128(part_o, (slot * D + dd) * 4, 0, kDeviceScope);
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (s0 + k >= nsr) break;
                    am_fold(mn, ls, os, __uint_as_float(ml[k].x), __uint_as_float(ml[k].y), __builtin_bit_cast(f32x4, ov[k]));
                }
            }
            finish(u, row, qh, mn, ls, os);
        }
    }
}

// Rows whose prefix spans several ranges: merges the ranges' partial results in range order, then the own
// slot.  One workgroup of two wavefronts per (query head, row): thread t owns value element t; the first
// wavefront also computes the own slot's score.
template <bool TREE>
__global__ __launch_bounds__(128) void k_attn_mfma_combine(AttnArgs a, int range, int n_split) {
    __shared__ float sh_own;
    const int head = blockIdx.x, row = blockIdx.y, tid = threadIdx.x, d = a.head_dim;
    const int pe = am_prefix_end<TREE>(a, row);
    const int nsr = (pe + range - 1) / range;
    if (nsr <= 1) return;  // finished by the attention kernel itself
    const int kvh = head / (a.n_q_heads / a.n_kv_heads);
    const uint16_t *kc = (const uint16_t *)a.kcache + (size_t)kvh * a.max_seq * d;
    const uint16_t *vt = (const uint16_t *)a.vcache + (size_t)kvh * a.nb32 * d * 32;
    const int own = am_own_slot<TREE>(a, row);
    const size_t base = ((size_t)row * a.n_q_heads + head) * n_split;
    const float *__restrict__ ml = a.part_ml + base * 2;
    const float *__restrict__ po = a.part_o + base * d + tid;
    // everything this thread needs, requested together: the ranges' (max, sum) pairs and its element of their
    // weighted values, eight ranges at a time
    const bool live = tid < d;
    const float v_own = live ? am_bf(vt[((size_t)(own >> 3) * d + tid) * 8 + (own & 7)]) : 0.f;
    float mn = -INFINITY, ls = 0.f, os = 0.f;
    for (int s0 = 0; s0 < nsr; s0 += 8) {
        float m8[8], l8[8], o8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int sidx = min(s0 + u, nsr - 1);
            m8[u] = ml[2 * sidx];
            l8[u] = ml[2 * sidx + 1];
            o8[u] = live ? po[(size_t)sidx * d] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (s0 + u >= nsr) break;
            am_fold(mn, ls, os, m8[u], l8[u], o8[u]);
        }
    }
    if (tid < 64) {
        const float sc = am_own_score(a.q + ((size_t)row * a.n_q_heads + head) * d, kc + (size_t)own * d, d, tid,
                                      1.0f / sqrtf((float)d));
        if (tid == 0) sh_own = sc;
    }
    __syncthreads();
    if (live) am_write(a, row, head * d + tid, am_finish(mn, ls, os, sh_own, v_own));
}

// The launch shape.  Everything that shapes a row's arithmetic (wavefronts per workgroup, slots per range)
// follows from the cache capacity and the head counts alone.
struct AmPlan {
    int nw;        // wavefronts per workgroup
    int range;     // cache slots per workgroup
    int hi_all;    // end of the longest prefix of the block
    int n_split;   // ranges that prefix reaches
    int n_tiles;   // member tiles (16 members each) = workgroups per (kv head, range)
    AmMerge merge;
};
AmPlan am_plan(const AttnArgs &a, int n_cu) {
    AmPlan p{};
    // Short caches of many-headed models: workgroups of eight wavefronts, ranges of a chunk each.  (us a launch, 32 heads of 128, cold caches;
    // before: one workgroup per head and range, three to six chunks in a row per wavefront.  640 slots: one row 10.2 / 8.5, 9 rows
    // 12.8 / 9.6, 31 rows 13.6 / 10.6; 1400 slots: 21.5 / 11.7, 21.3 / 11.8, 21.8 / 17.9; one range as before, with this kernel 10.2, 11.9,
    // 12.5 and 21.0, 20.6, 21.5; ranges of 128 with four wavefronts: 14 at 9 rows and 640 slots; ranges of 512: 10.8, 11.8, 12.7 and
    // 13.6, 13.2, 14.3.)  Where a full block's partial results would not fit the static scratch, one range.
    const bool short_cache = attn_uses_head_kernel(a.max_seq, a.n_kv_heads);
    if (short_cache) {
        p.nw = 8;
        p.range = 256;
        const size_t slots = (size_t)kMaxRows * a.n_q_heads * ((a.max_seq + p.range - 1) / p.range);
        if (slots * (a.head_dim + 2) * 4 + 256 > kStaticAttnBytes) p.range = (a.max_seq + 31) / 32 * 32;
    } else {
        // otherwise the capacity is cut into enough ranges for about two workgroups per compute unit with one member tile, and a
        // launch of its own merges them (7B, 8150 slots: 30.4 us for both, one row; 9 rows 31.2.  By the last workgroup, 16 ranges
        // of 9 rows: 40)
        p.nw = 4;
        int want = (2 * n_cu + a.n_kv_heads - 1) / a.n_kv_heads;
        if (want > a.max_split) want = a.max_split;
        if (want < 1) want = 1;
        // (whole chunks; a range need not hold the same number of chunks for every wavefront)
        p.range = std::max(32 * p.nw, ((a.max_seq + want - 1) / want + 31) / 32 * 32);
    }
    if (a.tree) {
        int deepest = 0;
        for (int r = 0; r < a.rows; ++r) deepest = std::max(deepest, (int)a.tt.depth[(a.row_base + r) & (kMaxRows - 1)]);
        p.hi_all = a.n_base + deepest;
    } else {
        p.hi_all = a.n_ctx - 1 + a.rows - 1;
    }
    p.n_split = std::max(1, (p.hi_all + p.range - 1) / p.range);
    p.n_tiles = (a.rows * (a.n_q_heads / a.n_kv_heads) + 15) / 16;
    // Who merges the ranges of a short cache changes no bit.  Up to a workgroup per compute unit: the last one of a head.  Beyond, those that
    // wait for a unit arrive late; with enough heads and tiles to occupy the units by themselves (three eighths of them) a
    // workgroup each walks all of its ranges, with fewer a launch of its own merges four ranges and more.  us, last workgroup / own launch /
    // one for all: 192 workgroups (32 heads, 1400 slots, 16 rows) 12.6 / 13.3 / -, 256 (1000 slots, 24 rows) 11.2 / 12.9 / -; 64 heads x
    // tiles, 384 (1400 slots, 31 rows) 19.5 / 17.9 / 24.5; 80, 400 (40 heads, 1100 slots) 19.0 / 18.1 / 21.2, 240 (700 slots) 11.1 / 12.7 / -;
    // 96, 288 and 480 (64 / 32 heads, 500 and 1100 slots, 24 rows) 11.7 / 13.5 / 12.4 and 19.2 / 19.7 / 19.7; 104, 416 (52 heads, 800 slots, 31
    // rows) - / 18.9 / 16.9; 128, 640 (64 heads, 1100 slots) 28.4 / 25.2 / 21.2; 256, 768 (128 / 32 heads, 600 slots) 27.4 / - / 14.2, 1280
    // (1100 slots) 44 / 39.4 / 20.2.
    const int groups = a.n_kv_heads * p.n_tiles;
    if (!short_cache)
        p.merge = kOwnLaunch;
    else if (p.n_split == 1 || groups * p.n_split <= n_cu)
        p.merge = kLastWorkgroup;
    else if (8 * groups >= 3 * n_cu)
        p.merge = kSerial;
    else
        p.merge = p.n_split <= 3 ? kLastWorkgroup : kOwnLaunch;
    return p;
}

}  // namespace

size_t attn_mfma_partial_floats(const AttnArgs &a, int n_cu) {
    const AmPlan p = am_plan(a, n_cu);
    const int max_splits = (a.max_seq + p.range - 1) / p.range;
    return max_splits > 1 ? (size_t)a.rows * a.n_q_heads * max_splits * a.head_dim : 0;
}

int attn_mfma_path_name(const AttnArgs &a, int n_cu, char *out, int capacity) {
    const AmPlan p = am_plan(a, n_cu);
    return snprintf(out, (size_t)capacity, "mfma<d %d, group %d, %d wavefronts, range %d, tiles %d%s%s>", a.head_dim,
                    a.n_q_heads / a.n_kv_heads, p.nw, p.range, p.n_tiles, a.tree ? ", tree" : "",
                    p.nw != 8 || p.merge == kLastWorkgroup ? "" : p.merge == kSerial ? ", serial" : ", merge launch");
}

hipError_t launch_attn_mfma(const AttnArgs &a, int n_cu, hipStream_t s) {
    if ((a.head_dim != 64 && a.head_dim != 128) || a.rows < 1 || a.rows > kAttnMfmaMaxRows || a.nb32 < (a.max_seq + 31) / 32 ||
        a.n_kv_heads < 1 || a.n_q_heads % a.n_kv_heads != 0 || !a.q || !a.q_s || !a.kcache || !a.vcache || (!a.out && !a.out_s) ||
        !a.part_o || !a.part_ml)
        return hipErrorInvalidValue;
    if (a.tree ? (a.row_base < 0 || a.row_base + a.rows > kMaxRows || a.n_base < 0 || a.n_base + a.row_base + a.rows > a.max_seq)
               : (a.n_ctx < 1 || a.n_ctx - 1 + a.rows > a.max_seq))
        return hipErrorInvalidValue;
    const AmPlan p = am_plan(a, n_cu);
    const int group = a.n_q_heads / a.n_kv_heads;
    if (p.n_split > a.max_split || (group & (group - 1)) != 0 ||
        (p.merge == kLastWorkgroup && p.n_split > 1 && (!a.counters || a.n_kv_heads * p.n_tiles > kMvCounters)))
        return hipErrorInvalidValue;
    const int D = a.head_dim;
    const size_t lds = ((size_t)(p.merge == kSerial ? 2 : 1) * p.nw * 16 * (D + kAmPad + 2) + 16) * sizeof(float);
    const dim3 grid(a.n_kv_heads, p.merge == kSerial ? 1 : p.n_split, p.n_tiles), block(64 * p.nw);
    const int range = p.merge == kSerial ? (a.max_seq + 31) / 32 * 32 : p.range;
    const int lg_group = __builtin_ctz(a.n_q_heads / a.n_kv_heads);
#define SWIFT_AM(DD, TR, WV, MG)                                                                                \
    do {                                                                                                        \
        static bool attr_set = false;                                                                           \
        if (!attr_set) {                                                                                        \
            hipError_t e = hipFuncSetAttribute((const void *)k_attn_mfma<DD, TR, WV, MG>,                       \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 144 * 1024);         \
            if (e != hipSuccess) return e;                                                                      \
            attr_set = true;                                                                                    \
        }                                                                                                       \
        hipLaunchKernelGGL((k_attn_mfma<DD, TR, WV, MG>), grid, block, lds, s, (const uint16_t *)a.kcache,      \
                           (const uint16_t *)a.vcache, a.q_s, a.max_seq, a.nb32, range, p.hi_all, a.rows, lg_group, a); \
    } while (0)
#define SWIFT_AM_D(DD)                                                                                          \
    if (p.merge == kLastWorkgroup) {                                                                            \
        if (a.tree) SWIFT_AM(DD, true, 8, kLastWorkgroup); else SWIFT_AM(DD, false, 8, kLastWorkgroup);         \
    } else if (p.merge == kSerial) {                                                                            \
        if (a.tree) SWIFT_AM(DD, true, 8, kSerial); else SWIFT_AM(DD, false, 8, kSerial);                       \
    } else if (p.nw == 8) {                                                                                     \
        if (a.tree) SWIFT_AM(DD, true, 8, kOwnLaunch); else SWIFT_AM(DD, false, 8, kOwnLaunch);                 \
    } else {                                                                                                    \
        if (a.tree) SWIFT_AM(DD, true, 4, kOwnLaunch); else SWIFT_AM(DD, false, 4, kOwnLaunch);                 \
    }
    if (D == 128) {
        SWIFT_AM_D(128)
    } else {
        SWIFT_AM_D(64)
    }
#undef SWIFT_AM_D
#undef SWIFT_AM
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.n_split == 1 || p.merge != kOwnLaunch) return e;
    const dim3 cgrid(a.n_q_heads, a.rows);
    if (a.tree)
        hipLaunchKernelGGL(k_attn_mfma_combine<true>, cgrid, dim3(128), 0, s, a, p.range, p.n_split);
    else
        hipLaunchKernelGGL(k_attn_mfma_combine<false>, cgrid, dim3(128), 0, s, a, p.range, p.n_split);
    return hipGetLastError();
}

}  // namespace swift
