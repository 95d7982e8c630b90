// Projections of a prompt macro block: up to kMacroSub sub-blocks of 64 rows through one weight matrix in
// one launch, as a blocked matrix product on the matrix cores (paper Section 4.2: the pass over the input
// that fills the cache before drafting starts; Section 3.1: the rows of a block are independent given the
// cache, so any number of them may share one sweep over the weights).
//
// A workgroup of 8 wavefronts owns a tile of WM RGW 16-row groups of W times WN / 2 sub-blocks (a sub-block: 64 rows x 2
// bf16 terms = 128 columns; WM WN = 8, WN = 4 or 2).  Wavefront (wm, wn) = (w % WM, w / WM) owns RGW row groups
// times 64 columns, half wn % 2 of sub-block wn / 2 (32 of its rows): 4 RGW accumulator tiles.  Both operands reach LDS straight
// from global memory (no registers in between) through a ring of NST stages of one 32-deep k tile each: WM RGW weight tiles
// of 1 KB (already in A-operand order) and the sub-blocks' 8 KB of split activations each (already in B-operand
// order).  LDS moves 128 bytes a clock, and it is what bounds all but the 256 x 256 tile: a wavefront reads RGW + 4 KB a stage,
// so its tile is kept near a square (as RGW / 2 row groups times 128 columns, it read RGW / 2 + 8 KB for the same products).  In step t the operands of stage t + 1 are read from LDS and stage t is multiplied while stages
// t + 2 .. t + NST - 1 are on their way and stage t + NST is requested: what a compute unit can take in is
// bounded by the bytes it keeps in flight, and the ring is what keeps most of LDS in flight.  One barrier per
// stage.
//
// The workgroups that share a weight tile (the other column tiles of the macro block) and those that
// share activations (the other row tiles) are given consecutive positions on one die, so that what one of
// them pulls from memory the others find in that die's L2.
//
// The epilogue works on the accumulators in registers and leaves every sub-block exactly as laid out for a 64-row block
// of the bulk layout.
//
// Workgroups come in rounds of one per compute unit.  Where the last round (or the only one: a matrix of few rows, a
// macro block of few sub-blocks) would leave compute units idle, its tiles are split in depth over up to four
// workgroups each: every wavefront publishes its results, and of the wavefronts that share a piece of a tile the one
// that arrives last adds them in part order and runs the epilogue.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <type_traits>

#include "swift_device.h"
#include "swift_kernels.h"
#include "swift_mv.h"

namespace swift {

namespace {

constexpr int kRingBytes = 144 * 1024;   // most of LDS: what is in flight bounds what a compute unit takes in
constexpr int kDeviceScope = 16;              // cache policy of buffer loads and stores: sc1
constexpr int kNormFloats = 2 * 16 * 64;  // scratch of gemm_norm_scales

// RMSNorm scales of the workgroup's two sub-blocks: rs[64 wn + r].  Thread (wn, q, r4) adds the partials q, q + 16,
// .. of rows 4 r4 .. 4 r4 + 3 of sub-block wn (16 loads of 16 bytes in flight at a time); then one thread per row
// adds the sixteen sums in order.  The first 256 partials are requested ahead of the ring's first stages, so that they do not queue
// behind 140 KB of tiles, and added up once those are on their way, where registers allow (kLateNorm; else before); the scales are read by
// the epilogue only, so no barrier here waits for more than LDS.
struct GemmNorm {
    f32x4 v[16];
};
__device__ inline GemmNorm gemm_norm_load(const MvArgs &a, const MacroArgs &ma, int sub0, int p0 = 0) {
    const int tid = threadIdx.x, q = (tid >> 4) & 15;
    const float *p = a.pss + (size_t)min(sub0 + (tid >> 8), ma.S - 1) * ma.pss + 4 * (tid & 15);
    GemmNorm n;
#pragma unroll
    for (int u = 0; u < 16; ++u) n.v[u] = *(const f32x4 *)(p + (size_t)min(p0 + q + 16 * u, a.n_pss - 1) * a.rp);
    return n;
}
__device__ inline f32x4 gemm_norm_sum(const MvArgs &a, const MacroArgs &ma, int sub0, const GemmNorm &first) {
    const int q = (threadIdx.x >> 4) & 15;
    f32x4 ss = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](int p0, const GemmNorm &n) {
#pragma unroll
        for (int u = 0; u < 16; ++u) ss += p0 + q + 16 * u < a.n_pss ? n.v[u] : f32x4{0.f, 0.f, 0.f, 0.f};
    };
    add(0, first);
    for (int p0 = 256; p0 < a.n_pss; p0 += 256) add(p0, gemm_norm_load(a, ma, sub0, p0));
    return ss;
}
__device__ inline void gemm_norm_scales(const MvArgs &a, const f32x4 &ss, float *rs, float *scratch) {
    const int tid = threadIdx.x, r4 = tid & 15, q = (tid >> 4) & 15, wn = tid >> 8;
    *(f32x4 *)(scratch + (wn * 16 + q) * 64 + 4 * r4) = ss;
    lds_barrier();
    if (tid < 128) {
        const int w2 = tid >> 6, r2 = tid & 63;
        float sum = 0.f;
#pragma unroll
        for (int q2 = 0; q2 < 16; ++q2) sum += scratch[(w2 * 16 + q2) * 64 + r2];
        rs[tid] = 1.0f / sqrtf(sum / (float)a.norm_dim + a.eps);
    }
}

// ------------------------------------------------------------------------------------------
// epilogue
// ------------------------------------------------------------------------------------------
// It works on the accumulators where they are: a wavefront's 4 accumulator tiles of a row group hold column 16 cb + col
// = 2 r + term in lane column col, tile rows 4 kg .. 4 kg + 3 in the lane's four registers.  The two terms of a block
// row sit in neighbouring lanes; the even lane keeps the even column blocks, the odd lane the odd ones, so that a lane
// ends up with two block rows r(c) = r0 + 16 c + 8 (col & 1) + col / 2, c = 0, 1 (r0: first row of the wavefront's half of
// the sub-block), and four consecutive tile rows of each: 16-byte reads and writes of everything that is laid out along the rows of W, and no trip through LDS.  (The
// block kernel's epilogue, which this replaces here, walks a row group in sixteen dependent rounds of a load, a few
// LDS reads and 2-byte stores: about 10 us per row group and wavefront, 20-43 us per workgroup, a third of a 512-row
// launch; now 4-9 us.)
__device__ inline float dpp_xor1(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));  // quad_perm [1,0,3,2]
}
__device__ inline int gemm_row(int c, int col) { return 16 * c + 8 * (col & 1) + (col >> 1); }  // within the wavefront's 32 rows
__device__ inline void fold_terms(const f32x4 (&acc)[4], int col, f32x4 (&y)[2]) {
    const bool odd = col & 1;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float own = odd ? acc[2 * c + 1][i] : acc[2 * c][i], other = odd ? acc[2 * c][i] : acc[2 * c + 1][i];
            y[c][i] = own + dpp_xor1(other);
        }
}
// Exchanges the upper 32 lanes of a with the lower ones of b.
__device__ inline void swap32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// The two-term split of the four values of lanes kg, kg ^ 1 (values 4 (kg & 1) .. of eight), to unit
// [chunk][128 columns][8]: columns 2 r and 2 r + 1.
__device__ inline void store_split(uint16_t *out_s, int chunk, int r, int kg, bool ok, const f32x4 &v) {
    uint32_t h[4], m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = f32_to_bf16_rne_finite(v[i]);
        m[i] = f32_to_bf16_rne_finite(v[i] - __uint_as_float(h[i] << 16));
    }
    const u32x4 u = join8(pack2(h[0], h[1]), pack2(h[2], h[3]), pack2(m[0], m[1]), pack2(m[2], m[3]));
    if (ok) *(u32x4 *)(out_s + ((size_t)chunk * 128 + 2 * r + (kg & 1)) * 8) = u;
}

// x += y for RGW row groups from rg0 and rows r0 .. r0 + 31: the residual values and gains of up to four of them are
// requested together.  y(g, out): finished sums of row group g.
template <int RGW, typename YF>
__device__ inline void gemm_resid(const MvArgs &a, int rg0, int r0, int lane, YF y) {
    const int col = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int g0 = 0; g0 < RGW; g0 += 4) {
        constexpr int G = RGW < 4 ? RGW : 4;
        f32x4 x[G][2], gain[G];
#pragma unroll
        for (int g = 0; g < G && g0 + g < RGW; ++g) {
            const int row = 16 * (rg0 + g0 + g) + 4 * kg;
            const bool in = row < a.O;  // (O is a multiple of 8: a lane's four rows are all real or all padding)
            gain[g] = in ? *(const f32x4 *)(a.gain_next + row) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int r = r0 + gemm_row(c, col);
                x[g][c] = in && r < a.R ? *(const f32x4 *)(a.out_f32 + (size_t)r * a.ld_out + row) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int g = 0; g < G && g0 + g < RGW; ++g) {
            const int rg = rg0 + g0 + g, row = 16 * rg + 4 * kg;
            if (rg >= a.n_rg) return;  // (wavefront-uniform)
            const bool in = row < a.O;
            f32x4 v[2];
            y(g0 + g, v);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int r = r0 + gemm_row(c, col);
                const bool ok = in && r < a.R;
                const f32x4 xn = x[g][c] + v[c];
                if (ok) *(f32x4 *)(a.out_f32 + (size_t)r * a.ld_out + row) = xn;
                store_split(a.out_s, 2 * rg + (kg >> 1), r, kg, ok, xn * gain[g]);
                float ss = in ? (xn[0] * xn[0] + xn[1] * xn[1]) + (xn[2] * xn[2] + xn[3] * xn[3]) : 0.f;
                ss = column_reduce(ss, [](float x, float y) { return x + y; });
                if (kg == 0 && r < a.R) a.pss_out[(size_t)rg * a.rp + r] = ss;
            }
        }
    }
}

// A lane's two block rows paired up: the first eight tile rows (gate, or the first half of rotary pairs) of c =
// kg >> 1 end up in lo, the other eight of the same block row in hi (tile rows 4 (kg & 1) .. of each), scaled.
__device__ inline void pair_halves(const f32x4 (&v)[2], const float (&sc)[2], f32x4 &lo, f32x4 &hi) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = v[0][i] * sc[0], y = v[1][i] * sc[1];
        swap32(x, y);
        lo[i] = x;
        hi[i] = y;
    }
}

__device__ inline void gemm_swiglu(const MvArgs &a, int rg, int r0, int lane, const float (&sc)[2], const f32x4 (&v)[2]) {
    const int col = lane & 15, kg = lane >> 4;
    f32x4 ga, up, h;
    pair_halves(v, sc, ga, up);
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = ga[i] / (1.0f + expf(-ga[i])) * up[i];
    const int r = r0 + gemm_row(kg >> 1, col);
    store_split(a.out_s, rg, r, kg, r < a.R && 16 * rg < a.O, h);
}

// Queries to fp32 rows, keys to their slots, values to the grouped layout: there, eight consecutive slots of an element
// are one 16-byte unit, so the values cross the lanes through a wavefront's own 1.3 KB of LDS (vsh).
template <int RGW, typename YF>
__device__ inline void gemm_qkv(const MvArgs &a, int rg0, int r0, int lane, const float (&sc)[2], uint16_t *vsh, YF y) {
    constexpr int VP = 32 + 8;  // pitch of an element's slots in vsh
    const int col = lane & 15, kg = lane >> 4;
    const int d = a.head_dim, half = d >> 1, gph = half >> 3, nq = a.n_q_heads, nkv = a.n_kv_heads;
    const int rl = gemm_row(kg >> 1, col), r = r0 + rl, pos = a.pos0 + r;  // the lane's block row, once paired up
    const bool ok = r < a.R;
    f32x4 cs[RGW], sn[RGW];
#pragma unroll
    for (int g = 0; g < RGW; ++g) {
        const int rg = min(rg0 + g, a.n_rg - 1), i0 = 8 * (rg % gph) + 4 * (kg & 1);
        cs[g] = *(const f32x4 *)(a.cos_tab + (size_t)(a.pos0 + min(r, a.R - 1)) * half + i0);
        sn[g] = *(const f32x4 *)(a.sin_tab + (size_t)(a.pos0 + min(r, a.R - 1)) * half + i0);
    }
#pragma unroll
    for (int g = 0; g < RGW; ++g) {
        const int rg = rg0 + g;
        if (rg >= a.n_rg) break;  // (wavefront-uniform)
        const int hl = rg / gph, hh = a.head0 + hl, e0 = 8 * (rg - hl * gph);  // head; first element of the row group's eight pairs
        f32x4 v[2], ya, yb;
        y(g, v);
        pair_halves(v, sc, ya, yb);
        if (hh < nq + nkv) {
            const f32x4 qa = ya * cs[g] - yb * sn[g], qb = yb * cs[g] + ya * sn[g];
            if (hh < nq) {
                float *qp = a.out_f32 + (size_t)r * a.ld_out + hh * d + e0 + 4 * (kg & 1);
                if (ok) {
                    *(f32x4 *)qp = qa;
                    *(f32x4 *)(qp + half) = qb;
                }
                continue;
            }
            ya = qa;
            yb = qb;
        }
        uint32_t ha[4], hb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ha[i] = f32_to_bf16_rne(ya[i]);
            hb[i] = f32_to_bf16_rne(yb[i]);
        }
        if (hh < nq + nkv || a.nb32 <= 0) {
            const int head = hh < nq + nkv ? hh - nq : hh - nq - nkv;
            uint16_t *plane = (uint16_t *)(hh < nq + nkv ? a.kcache : a.vcache);
            const u32x4 u = join8(pack2(ha[0], ha[1]), pack2(ha[2], ha[3]), pack2(hb[0], hb[1]), pack2(hb[2], hb[3]));
            if (ok) *(u32x4 *)(plane + ((size_t)head * a.max_seq + pos) * d + e0 + (kg & 1) * half) = u;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vsh[(4 * (kg & 1) + i) * VP + rl] = (uint16_t)ha[i];
                vsh[(8 + 4 * (kg & 1) + i) * VP + rl] = (uint16_t)hb[i];
            }
            // (one wavefront's LDS instructions are carried out in order: only the compiler has to keep it)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int e = lane & 15, elem = e0 + (e & 7) + (e >> 3) * half;
            const int u8 = 8 * (lane >> 4), ru = r0 + u8;  // eight slots from block row ru on
            const u32x4 w = *(const u32x4 *)(vsh + e * VP + u8);
            uint16_t *vp = (uint16_t *)a.vcache;
            if ((a.pos0 & 7) == 0 && ru + 8 <= a.R) {
                *(u32x4 *)(vp + kv_vt_index(hh - nq - nkv, a.nb32, d, a.pos0 + ru, elem)) = w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (ru + i < a.R)
                        vp[kv_vt_index(hh - nq - nkv, a.nb32, d, a.pos0 + ru + i, elem)] = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Which workgroups do what.  Row tiles [0, MTF) are computed whole, one workgroup each per column tile (grid ids below
// n_full); the rest are split in depth over ksp workgroups of TS k tiles each.  fold_rg, fold_TS: a tile that is computed whole
// adds the sums of its row groups from fold_rg on in parts of fold_TS k tiles all the same (see gemm_sums).
struct GemmPlan {
    int MT, NN, MTF, n_full, ksp, TS, fold_rg, fold_TS;
};

template <int RGW>
struct GemmOperands {
    u32x4 av[RGW], bv[4];
};

template <int EPI, int WN, int RGW, bool FOLD>
__global__ __launch_bounds__(512) void k_gemm(MvArgs a, MacroArgs ma, GemmPlan pl) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int WM = 8 / WN, SB = WN / 2;       // wavefronts along the rows; SB sub-blocks side by side
    constexpr int TRG = WM * RGW;                 // row groups of the workgroup's tile
    constexpr int A_BYTES = TRG * 1024;
    constexpr int ST_BYTES = A_BYTES + SB * 8192;
    constexpr int NST = kRingBytes / ST_BYTES;   // stages of the ring
    constexpr int NP = TRG + 8 * SB;              // 1 KB pieces of a stage
    constexpr int PW = (NP + 7) / 8;              // pieces a wavefront copies per stage (PW - 1 past the remainder)
    constexpr bool kLateNorm = !FOLD && RGW != 7 && !(EPI == EPI_QKV && RGW == 8);  // (the others have no registers for the partials behind the first requests)
    constexpr bool kNorm = EPI != EPI_RESID;      // the input is a normalised one: scales from the producer's partial sums
    static_assert(NST >= 3 && NST * PW < 64, "ring depth against the load counter");
    unsigned char *ring = smem;
    float *rs = (float *)(smem + kRingBytes);     // [2][64]
    float *nscratch = rs + 128;                   // [kNormFloats]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM, ws = wn >> 1, wh = wn & 1;  // its sub-block of the tile, its half of that
    // workgroup -> tile: the NN column tiles of a row tile (for tiles split in depth: of one of its parts) sit next to
    // each other on one die (consecutive workgroup ids go round the 8 dies)
    const int NN = pl.NN, id = (int)blockIdx.x < pl.n_full ? blockIdx.x : blockIdx.x - pl.n_full;
    const int die = id & 7, qd = id >> 3;
    const int nt = qd % NN, pair = (qd / NN) * 8 + die;
    int mt = pair, kz = 0, KSP = 1, TS = a.T;
    if ((int)blockIdx.x < pl.n_full) {
        if (mt >= pl.MTF) return;
    } else {
        const int tail = pl.MT - pl.MTF;
        if (pair >= tail * pl.ksp) return;
        kz = pair / tail;
        mt = pl.MTF + pair - kz * tail;
        KSP = pl.ksp;
        TS = pl.TS;
    }
    const int sub0 = SB * nt;
    const int T = a.T;
    const int col = lane & 15, kg = lane >> 4;
    const int t_lo = kz * TS, t_hi = min(T, t_lo + TS);  // (every part holds tiles: the launcher)

    // A ragged last k tile (depth not a multiple of 32) is not part of the pipeline: it is handled at the end (by
    // the part that holds it).  TF: full tiles of this workgroup's part; TR: the ragged tile's number, if it is here.
    const bool ragged = (a.K & 31) != 0 && t_hi == T;
    const int TF = t_hi - t_lo - (ragged ? 1 : 0), TR = T - 1;
    // ---- what this wavefront copies per stage: pieces p = wave + 8 i, each 64 lanes x 16 bytes from a
    // wavefront-uniform address
    const unsigned char *src[PW];   // tile 0 of the piece (wavefront-uniform)
    int stride[PW];                 // bytes from one k tile to the next
    int seg64[PW];                  // B pieces: first 16-byte unit of the piece inside its tile (A pieces: -1)
    uint32_t voff[PW];              // this lane's byte offset from src[i] in the next stage to be issued
#pragma unroll
    for (int i = 0; i < PW; ++i) {
        const int p = wave + 8 * i;
        if (p < TRG) {
            const int rg = min(mt * TRG + p, a.n_rg - 1);  // row groups past the end repeat the last one
            src[i] = (const unsigned char *)a.Wt + (size_t)rg * T * 1024;
            stride[i] = 1024;
            seg64[i] = -1;
        } else {
            const int q = min(p, NP - 1) - TRG, sb = min(sub0 + (q >> 3), ma.S - 1), seg = q & 7;
            src[i] = (const unsigned char *)(a.in_s + (size_t)sb * ma.in_s) + seg * 1024;
            stride[i] = 8192;
            seg64[i] = seg * 64;
        }
        voff[i] = lane * 16 + t_lo * stride[i];
    }
    const bool full_share = (NP % 8 == 0) || wave < NP % 8;  // this wavefront copies PW pieces (else PW - 1)
    // FULL: whether this wavefront copies PW pieces (a compile-time copy of full_share)
    auto issue = [&](int slot_bytes, auto FULL) {
        unsigned char *dst = ring + slot_bytes + wave * 1024;
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            if (i < PW - 1 || decltype(FULL)::value)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src[i] + (size_t)voff[i]),
                                                 (__attribute__((address_space(3))) void *)(dst + i * 8192), 16, 0, 0);
            voff[i] += stride[i];
        }
    };
    // waits until at most N stages' worth of this wavefront's loads are in flight (loads complete in order; every
    // stage is the same number of loads per lane)
    auto wait_all_but = [&](auto N, auto FULL) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(N)::value * (decltype(FULL)::value ? PW : PW - 1)) : "memory");
    };
    // (the wait as a builtin: the compiler follows it, unlike one inside inline assembly, and so does not add a
    // wait of its own for the operand reads of the previous step in front of the matrix instructions)
    auto lds_sync = [&]() {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wavefront's LDS reads and writes are done
        asm volatile("s_barrier" ::: "memory");
    };

    f32x4 acc[RGW][4];
    f32x4 done[FOLD ? RGW : 1][2];  // FOLD: the finished parts of the sums, the two terms combined
    auto clear = [&]() {            // (once the registers of the norm partials are free)
#pragma unroll
        for (int g = 0; g < RGW; ++g)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < (FOLD ? RGW : 1); ++g)
#pragma unroll
            for (int c = 0; c < 2; ++c) done[g][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    auto fold_part = [&]() {
#pragma unroll
        for (int g = 0; g < (FOLD ? RGW : 0); ++g)
            if ((mt * WM + wm) * RGW + g >= pl.fold_rg) {  // (wavefront-uniform)
                f32x4 v[2];
                fold_terms(acc[g], col, v);
#pragma unroll
                for (int c = 0; c < 2; ++c) done[g][c] += v[c];
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };

    const unsigned char *a_base = ring + (wm * RGW) * 1024 + lane * 16;
    const unsigned char *b_base = ring + A_BYTES + ws * 8192 + (kg * 128 + 64 * wh + col) * 16;
    auto read_operands = [&](int slot_bytes, GemmOperands<RGW> &o) {
#pragma unroll
        for (int g = 0; g < RGW; ++g) o.av[g] = *(const u32x4 *)(a_base + slot_bytes + g * 1024);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) o.bv[cb] = *(const u32x4 *)(b_base + slot_bytes + cb * 256);
    };
    auto multiply = [&](const GemmOperands<RGW> &o) {
#pragma unroll
        for (int g = 0; g < RGW; ++g)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                acc[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, o.av[g]),
                                                                     __builtin_bit_cast(bf16x8, o.bv[cb]), acc[g][cb], 0, 0, 0);
    };

    // The order of a step's instructions: two matrix instructions, the copies, then the next stage's operand reads one by
    // one between the other matrix instructions.  (All reads in front, as it was: they queue up at LDS, 88 KB per step
    // of a compute unit, and hold the matrix cores up; all behind: LDS and the matrix cores take turns.  7B, 512 rows, this
    // change alone: gate/up 184 -> 163 us, q|k|v 117 -> 107.)
    auto interleave = [&]() {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, PW, 0);
#pragma unroll
        for (int i = 0; i < RGW + 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The pipeline.  Step t: the operands of stage t are in registers (read during step t - 1).  Once stage t + 1
    // has landed for everybody -- and everybody's reads of stage t have completed: the barrier waits for them --
    // stage t + NST is requested into the slot stage t leaves, the operands of stage t + 1 are read into the other
    // register set, and the matrix cores work on stage t meanwhile.  `slot`: byte offset of stage t's ring slot.
    // The loop body is kept free of conditions: a wavefront issues at most one scalar instruction every few cycles,
    // and whatever the loop needs beyond the matrix instructions is paid for in full.
    GemmNorm np;
    f32x4 norm_ss = {0.f, 0.f, 0.f, 0.f};
    auto start = [&](auto FULL) {  // requests the first stages and waits for the first one
        const int first = min(TF, NST);
        if (TF >= NST) {
#pragma unroll
            for (int t = 0; t < NST; ++t) issue(t * ST_BYTES, FULL);
        } else {
            for (int t = 0; t < first; ++t) issue(t * ST_BYTES, FULL);
        }
        if (kNorm && kLateNorm) norm_ss = gemm_norm_sum(a, ma, sub0, np);
        if (kNorm) gemm_norm_scales(a, norm_ss, rs, nscratch);
        if (TF >= NST)
            wait_all_but(std::integral_constant<int, NST - 1>(), FULL);
        else
            wait_all_but(std::integral_constant<int, 0>(), FULL);
    };
    auto next_slot = [&](int sl) { return sl + ST_BYTES == NST * ST_BYTES ? 0 : sl + ST_BYTES; };
    constexpr auto ALL = std::integral_constant<int, 0>();
    constexpr auto AHEAD = std::integral_constant<int, NST - 2>();  // stages t + 2 .. t + NST - 1 may stay in flight
    // A wavefront whose half of a sub-block holds no row copies its share and keeps the others' barriers, no more (its products cost
    // the others power and LDS: 13 rows in the last of 4 sub-blocks, 13B: gate/up 133.7 / 130.5 us, down_proj 86.6 / 83.9, q|k|v 92.0 /
    // 88.6; of 2, 70B gate/up 238 / 214).
    auto copy_only = [&](auto FULL) {
        start(FULL);
        if (TF == 0) return;
        lds_sync();
        for (int t = 0, slot = 0; t < TF; ++t) {
            if (t + NST < TF) {
                wait_all_but(AHEAD, FULL);
                lds_sync();
                issue(slot, FULL);
            } else {
                wait_all_but(ALL, FULL);
                lds_sync();
            }
            slot = next_slot(slot);
        }
    };
    auto pipeline = [&](auto FULL) {
        start(FULL);
        clear();
        if (TF == 0) return;
        GemmOperands<RGW> o0, o1;
        lds_sync();
        read_operands(0, o0);
        int t = 0, slot = 0;
        auto steady = [&](const GemmOperands<RGW> &cur, GemmOperands<RGW> &nxt) {
            const int nslot = next_slot(slot);
            wait_all_but(AHEAD, FULL);
            lds_sync();
            __builtin_amdgcn_sched_barrier(0);
            issue(slot, FULL);
            read_operands(nslot, nxt);
            multiply(cur);
            interleave();
            slot = nslot;
        };
        // (the last step reads a slot nobody needs: no harm)
        auto drain = [&](const GemmOperands<RGW> &cur, GemmOperands<RGW> &nxt) {
            const int nslot = next_slot(slot);
            wait_all_but(ALL, FULL);
            lds_sync();
            __builtin_amdgcn_sched_barrier(0);
            read_operands(nslot, nxt);
            multiply(cur);
            interleave();
            slot = nslot;
        };
        for (int end = FOLD ? pl.fold_TS : TF;; end += pl.fold_TS) {  // a part of the sums (an even number of stages but for the last)
            const int e = min(end, TF), both = min(e, TF - NST - 1);
            for (; t < both; t += 2) {  // both steps issue a stage
                steady(o0, o1);
                steady(o1, o0);
            }
            if (t < e && t + NST < TF) {  // an odd number of issuing steps: one more, then the operands sit in the other set
                steady(o0, o1);
                drain(o1, o0);
                t += 2;
            }
            for (; t < e; t += 2) {
                drain(o0, o1);
                if (t + 1 < e) drain(o1, o0);
            }
            if (!FOLD) break;
            if (e < TF || (ragged && end == TF)) fold_part();
            if (e == TF) break;
        }
    };
    const int sub = min(sub0 + ws, ma.S - 1), r0 = 32 * wh;  // the wavefront's sub-block, and its rows of it: r0 .. r0 + 31
    const bool wave_live = sub0 + ws < ma.S && r0 < (sub == ma.S - 1 ? ma.rows_last : 64);
    if (kNorm) {
        np = gemm_norm_load(a, ma, sub0);
        if (!kLateNorm) norm_ss = gemm_norm_sum(a, ma, sub0, np);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (!wave_live) {
        if (full_share)
            copy_only(std::true_type());
        else
            copy_only(std::false_type());
    } else if (full_share) {
        pipeline(std::true_type());
    } else {
        pipeline(std::false_type());
    }
    if (ragged) {
        // the ragged tile: copied with ordinary loads, zeros past the real depth (a piece lies wholly inside or
        // wholly outside it), into the first ring slot
        const int real_units = (a.K >> 3) * 128;  // 16-byte units of a sub-block's split activation
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            if (i < PW - 1 || full_share) {
                const bool past = seg64[i] >= 0 && seg64[i] + TR * 512 >= real_units;
                const unsigned char *sp = src[i] + (size_t)TR * stride[i];
                const u32x4 v = past ? u32x4{0u, 0u, 0u, 0u} : *(const u32x4 *)(sp + lane * 16);
                *(u32x4 *)(ring + wave * 1024 + i * 8192 + lane * 16) = v;
            }
        }
        __syncthreads();
        if (wave_live) {
            GemmOperands<RGW> o;
            read_operands(0, o);
            multiply(o);
        }
    }

    // ---- epilogue on the sub-block's own buffers
    __syncthreads();  // the ring is no longer read (and the scales are visible where no step had a barrier)
    if (!wave_live) return;
    MvArgs as = a;
    as.R = sub == ma.S - 1 ? ma.rows_last : 64;
    as.pos0 = a.pos0 + 64 * sub;
    if (a.out_f32) as.out_f32 = a.out_f32 + (size_t)sub * ma.out_f32;
    if (a.out_s) as.out_s = a.out_s + (size_t)sub * ma.out_s;
    if (a.pss_out) as.pss_out = a.pss_out + (size_t)sub * ma.pss_out;
    const int rg0 = (mt * WM + wm) * RGW;
    // (the epilogue of G row groups from rg1 on; y(g, v): finished sums of the g-th of them)
    auto finish = [&](auto G, int rg1, auto y) {
        constexpr int kG = decltype(G)::value;
        if (EPI == EPI_RESID) {
            gemm_resid<kG>(as, rg1, r0, lane, y);
        } else {
            float sc[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) sc[c] = rs[64 * ws + r0 + gemm_row(c, col)];
            if (EPI == EPI_QKV) {
                gemm_qkv<kG>(as, rg1, r0, lane, sc, (uint16_t *)ring + (size_t)wave * 1024, y);
            } else {
#pragma unroll
                for (int g = 0; g < kG; ++g) {
                    if (rg1 + g >= a.n_rg) break;
                    f32x4 v[2];
                    y(g, v);
                    gemm_swiglu(as, rg1 + g, r0, lane, sc, v);
                }
            }
        }
    };
    constexpr auto WHOLE = std::integral_constant<int, RGW>();
    if (FOLD || KSP == 1) {
        finish(WHOLE, rg0, [&](int g, f32x4(&v)[2]) {
            fold_terms(acc[g], col, v);
            if (FOLD) {
#pragma unroll
                for (int c = 0; c < 2; ++c) v[c] = done[g][c] + v[c];
            }
        });
        return;
    }
    // ---- depth split over workgroups.  Every wavefront publishes its results, the two terms combined, as
    // part[kz][row group][sub-block] (lane by lane: its partners in the other parts read them back into the same lanes),
    // and counts itself in; the one that arrives last of its KSP partners adds the parts in part order (so the result
    // does not depend on who is last) and runs the epilogue.  No barrier: the wavefronts of a tile are independent, and
    // partners arrive in any order, so the adding is spread over the parts.  Stores and loads of the parts are device
    // scope (sc1: written through, read past this die's L2), so once a wavefront's stores are acknowledged (vmcnt 0) a
    // relaxed count publishes them, and no cache has to be written back or invalidated.  (One counter per workgroup,
    // 8-byte stores and an acquire-release count cost 25-30 us per launch; this ~10.)
    const int rgt0 = rg0 - pl.MTF * TRG, n_rgt = a.n_rg - pl.MTF * TRG;  // row groups of the split tiles
    const __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(a.part, 0, 0x7fffffff, 0x00020000);
    auto part_off = [&](int k2, int g, int c) { return (uint32_t)((((k2 * n_rgt + rgt0 + g) * ma.S + sub) * 4 + 2 * wh + c) * 1024 + lane * 16); };
#pragma unroll
    for (int g = 0; g < RGW; ++g) {
        if (rg0 + g >= a.n_rg) break;
        f32x4 v[2];
        fold_terms(acc[g], col, v);
#pragma unroll
        for (int c = 0; c < 2; ++c)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[c]), part, part_off(kz, g, c), 0, kDeviceScope);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int *counter = a.counters + ((mt - pl.MTF) * NN + nt) * 8 + wave;
    int arrived = 0;
    if (lane == 0) arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(arrived) != KSP - 1) return;
    asm volatile("" ::: "memory");
    // (the parts of two row groups are requested together: one by one, each was a round trip of its own.  us, before / now: 13B, 4
    // sub-blocks o_proj 41 / 37; 7B, 2 sub-blocks o_proj 21.8 / 20.5)
    auto batch = [&](auto G, int g0) {
        constexpr int kG = decltype(G)::value;
        f32x4 w[4][kG][2];
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2)
#pragma unroll
            for (int g = 0; g < kG; ++g)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    if (k2 < KSP && rg0 + g0 + g < a.n_rg)  // (wavefront-uniform)
                        w[k2][g][c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part, part_off(k2, g0 + g, c), 0, kDeviceScope));
        finish(G, rg0 + g0, [&](int g, f32x4(&v)[2]) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                v[c] = w[0][g][c];
#pragma unroll
                for (int k2 = 1; k2 < 4; ++k2)
                    if (k2 < KSP) v[c] += w[k2][g][c];
            }
        });
    };
    constexpr int kB = RGW < 2 || (EPI == EPI_QKV && RGW == 8) ? 1 : 2;
#pragma unroll 1
    for (int g0 = 0; g0 + kB <= RGW; g0 += kB) batch(std::integral_constant<int, kB>(), g0);
    if constexpr (RGW % kB != 0) batch(std::integral_constant<int, 1>(), RGW - 1);
    if (lane == 0) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int EPI, int WN, int RGW, bool FOLD>
hipError_t launch_gemm_f(const MvArgs &a, const MacroArgs &ma, const GemmPlan &pl, hipStream_t s) {
    static bool attr_set = false;
    const size_t lds = kRingBytes + 128 * 4 + kNormFloats * 4;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)k_gemm<EPI, WN, RGW, FOLD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tail = pl.MT - pl.MTF;
    const int grid = pl.n_full + (tail * pl.ksp + 7) / 8 * 8 * pl.NN;
    hipLaunchKernelGGL((k_gemm<EPI, WN, RGW, FOLD>), dim3(grid), dim3(512), lds, s, a, ma, pl);
    return hipGetLastError();
}
constexpr int kFoldMaxRgw = 6;  // (beside more accumulators, the finished parts do not fit the registers)
template <int EPI, int WN, int RGW>
hipError_t launch_gemm_t(const MvArgs &a, const MacroArgs &ma, const GemmPlan &pl, hipStream_t s) {
    if constexpr (RGW <= kFoldMaxRgw)
        if (pl.fold_TS > 0) return launch_gemm_f<EPI, WN, RGW, true>(a, ma, pl, s);
    return launch_gemm_f<EPI, WN, RGW, false>(a, ma, pl, s);
}

// Tilings: wavefronts along the columns (4: two sub-blocks side by side, 2: one) and row groups per wavefront.  Codes 1..4:
// workgroup tiles of 64, 128, 192, 256 rows x 256 columns; 5, 6: 128, 256 rows x 128 columns (for matrices with few rows, where
// the narrower tile gives as many workgroups with fewer bytes to copy per product); 7..9: 96, 160, 224 rows x 256 columns; 10:
// 192 rows x 128 columns.  The odd heights fit more matrices into whole rounds of workgroups: without them the fastest launches
// of the sweep below add up to 1.8 % more.
struct GemmTiling {
    int wn, rgw;
};
constexpr int kGemmCodes = 10;
constexpr GemmTiling kGemmTilings[kGemmCodes + 1] = {{0, 0}, {4, 2}, {4, 4}, {4, 6}, {4, 8}, {2, 2}, {2, 4}, {4, 3}, {4, 5}, {4, 7}, {2, 3}};

// What a workgroup costs, measured with all compute units at work (7B, 13B and 70B shapes, 128-1024 rows): us per k tile, and us
// per workgroup for its start, the first stages' arrival and the epilogue.  Over 105 launches (profiles/blocked_product_sweep.txt)
// the shapes and splits chosen by them, were any order of the sums allowed, add up to 0.3 % more than the fastest of each launch;
// single launches up to 11 % (13B q|k|v).  With the order kept (gemm_sums) it is 3.2 %.  (A 256 x 256 tile's matrix instructions take 0.54 us per k tile at 1.9 GHz; a whole chip of them is held to less by
// its power, 1.6 PFLOP/s.)
struct GemmCost {
    double stage, fixed;
};
constexpr GemmCost kGemmCosts[kGemmCodes + 1] = {{0, 0},       {0.286, 5.4}, {0.393, 5.6}, {0.513, 8.3}, {0.670, 6.1}, {0.276, 4.6},
                                                {0.425, 4.8}, {0.329, 5.0}, {0.445, 7.3}, {0.594, 6.7}, {0.347, 5.1}};
constexpr double kPartBytesPerUs = 1.43e6;  // publishing and adding the parts of tiles split in depth

// The order of the sums.  Row groups from `first` on are summed in parts of TS k tiles (each from zero, the two terms combined,
// then the parts in order), the others in one go.  It is a function of the matrix and the number of sub-blocks alone, not of
// the tile shape or of who computes what, so that the cache entries that a prompt leaves are the same bits whatever the plan below
// makes of them (a sampled continuation may hang on them); macro blocks of more than eight sub-blocks follow the order of
// eight, so that a prompt may be cut into either.  The shapes and costs below are those of a launcher of earlier kernels, whose last round
// of workgroups was split in depth: they stand for nothing but the order it left, which caches and continuations follow.
// What it costs: row groups summed in parts exclude tiles whose edges do not meet the first of them, and, inside a workgroup, tiles of more
// than kFoldMaxRgw row groups per wavefront (7B gate/up, 1024 rows: 309 us, 280 with 256 x 256 tiles; k|v of 70B at 6-8
// sub-blocks 69, 43-47).
struct GemmSums {
    int first, parts, TS;
};
GemmSums gemm_sums(int n_rg, int T, int S, int n_cu) {
    static const struct { int wn, rgw; double stage, fixed; } kShapes[6] = {{2, 1, 0.305, 9.0}, {2, 2, 0.37, 10.0}, {2, 3, 0.54, 12.0},
                                                                            {2, 4, 0.58, 14.0}, {1, 1, 0.26, 8.0},  {1, 2, 0.385, 9.0}};
    S = std::min(S, 8);
    GemmSums best{n_rg, 1, T};
    double least = 1e30;
    for (const auto &h : kShapes)
        for (int ksp = 1; ksp <= 4; ++ksp) {
            const int trg = 8 / h.wn * h.rgw, MT = (n_rg + trg - 1) / trg, NN = (S + h.wn - 1) / h.wn;
            const int per_round = std::max(1, n_cu / NN / 8) * 8, MTF = ksp == 1 ? MT : MT / per_round * per_round;
            const int TS = (T + ksp - 1) / ksp, parts = (T + TS - 1) / TS, tail = MT - MTF;
            double us = (double)((MTF * NN + n_cu - 1) / n_cu) * (T * h.stage + h.fixed);
            if (tail == 0 || parts == 1) {
                if (ksp != 1) continue;
            } else {
                const int64_t slots = (int64_t)parts * (n_rg - MTF * trg) * S;
                if (TS < 16 || slots > 8192 || tail * NN * 8 > 4096) continue;
                us += (double)((tail * NN * parts + n_cu - 1) / n_cu) * (TS * h.stage + h.fixed) + (double)slots * 4096.0 / 1.3e6;
            }
            if (us >= least) continue;
            least = us;
            best = parts == 1 || tail == 0 ? GemmSums{n_rg, 1, T} : GemmSums{MTF * trg, parts, TS};
        }
    return best;
}

// The plan of a tiling, and what it costs.  Row groups that are summed in parts are either split over workgroups, a part each
// (fold = false; their first one has to begin a tile, and the partial results have to fit the scratch), or added part by part in the
// workgroup that computes the whole depth (fold = true; parts of an even number of k tiles, up to six row groups per wavefront).
bool gemm_plan(const MvArgs &a, const MacroArgs &ma, int n_cu, int code, const GemmSums &sums, bool fold, GemmPlan &pl, double &us) {
    const int wn = kGemmTilings[code].wn, rgw = kGemmTilings[code].rgw, trg = (8 / wn) * rgw, sb = wn / 2;
    const bool split = sums.parts > 1 && !fold;
    if (fold && (sums.parts == 1 || (sums.TS & 1) != 0 || rgw > kFoldMaxRgw)) return false;
    if (split && sums.first % trg != 0) return false;
    pl.MT = (a.n_rg + trg - 1) / trg;
    pl.NN = (ma.S + sb - 1) / sb;
    pl.MTF = split ? sums.first / trg : pl.MT;
    pl.ksp = sums.parts;
    pl.TS = sums.TS;
    pl.n_full = (pl.MTF + 7) / 8 * 8 * pl.NN;
    pl.fold_rg = sums.first;
    pl.fold_TS = fold ? sums.TS : 0;
    const int tail = pl.MT - pl.MTF;
    const GemmCost c = kGemmCosts[code];
    // (rounds by the fullest die: all column tiles of a row tile, or of one of its parts, are on one)
    auto rounds = [&](int groups) { return (double)(((groups + 7) / 8 * pl.NN + n_cu / 8 - 1) / std::max(1, n_cu / 8)); };
    us = rounds(pl.MTF) * (a.T * c.stage + c.fixed);
    if (tail == 0) return true;
    const int64_t slots = (int64_t)pl.ksp * (a.n_rg - sums.first) * ma.S;
    us += rounds(tail * pl.ksp) * (pl.TS * c.stage + c.fixed) + (double)slots * 4096.0 / kPartBytesPerUs;
    return a.part && a.counters && slots <= ma.part_slots && tail * pl.NN * 8 <= 4096;
}

// The plan with the least cost: the tile shape and the way of adding the parts that finish first, among those that keep the order
// of the sums.  Workgroups come in rounds of one per compute unit, and splitting the last round's tiles in depth fills the units
// that would idle in it, for the price of the parts' results.  code 0: none keeps it.
struct GemmChoice {
    int code;
    GemmPlan pl;
};
GemmChoice gemm_choose(const MvArgs &a, const MacroArgs &ma, int n_cu, int tiling_override, const GemmSums &sums) {
    GemmChoice ch{};
    double best = 1e30;
    for (int c = 1; c <= kGemmCodes; ++c) {
        if (tiling_override && c != tiling_override) continue;
        for (const bool fold : {false, true}) {
            GemmPlan p;
            double us;
            if (!gemm_plan(a, ma, n_cu, c, sums, fold, p, us) || us >= best) continue;
            best = us;
            ch = GemmChoice{c, p};
        }
    }
    return ch;
}
// The order of the sums of a launch's row groups: that of their matrix.
GemmSums launch_sums(const MvArgs &a, const MacroArgs &ma, int n_cu) {
    GemmSums sums = gemm_sums(ma.matrix_rg > 0 ? ma.matrix_rg : a.n_rg, a.T, ma.S, n_cu);
    sums.first = std::max(0, sums.first - ma.first_rg);
    return sums.first >= a.n_rg ? GemmSums{a.n_rg, 1, a.T} : sums;
}

}  // namespace

bool gemm_keeps_order(const MvArgs &a, const MacroArgs &ma, int n_cu) {
    return gemm_choose(a, ma, n_cu, 0, launch_sums(a, ma, n_cu)).code != 0;
}

int gemm_path_name(const MvArgs &a, const MacroArgs &ma, int n_cu, char *out, int capacity) {
    const GemmChoice ch = gemm_choose(a, ma, n_cu, 0, launch_sums(a, ma, n_cu));
    if (ch.code == 0) return snprintf(out, (size_t)capacity, "none");
    const GemmPlan &p = ch.pl;
    return snprintf(out, (size_t)capacity, "gemm<tile %d, parts %d, %s>", ch.code, p.fold_TS > 0 || p.MTF < p.MT ? p.ksp : 1,
                    p.fold_TS > 0 ? "inside" : p.MTF < p.MT ? "workgroups" : "whole");
}

hipError_t launch_gemm(int epi, const MvArgs &a, const MacroArgs &ma, int n_cu, int tiling_override, hipStream_t s) {
    if (ma.S < 1 || ma.S > kMacroSub || ma.rows_last < 1 || ma.rows_last > 64 || a.RL != (64 | kBulkLayout) || a.rp != 64 ||
        (a.K & 7) != 0 || a.T != (a.K + 31) / 32 || a.n_rg < 1 || !a.Wt || !a.in_s || a.tree || a.q_s ||
        (epi == EPI_RESID ? !a.gain_next || !a.pss_out || (a.O & 7) != 0 : !a.pss || a.n_pss < 1))
        return hipErrorInvalidValue;
    GemmChoice ch = gemm_choose(a, ma, n_cu, tiling_override, launch_sums(a, ma, n_cu));
    // (a tile shape asked for by a tuning run, or scratch that is not there, may not allow the order: then the sums are added in one go,
    // which every shape can)
    if (ch.code == 0) ch = gemm_choose(a, ma, n_cu, tiling_override, GemmSums{a.n_rg, 1, a.T});
    const int code = ch.code;
    const GemmPlan &pl = ch.pl;
    if (code == 0) return hipErrorInvalidValue;
#define SWIFT_GEMM_CASE(E)                                                \
    case E:                                                               \
        switch (code) {                                                   \
            case 1: return launch_gemm_t<E, 4, 2>(a, ma, pl, s);         \
            case 2: return launch_gemm_t<E, 4, 4>(a, ma, pl, s);         \
            case 3: return launch_gemm_t<E, 4, 6>(a, ma, pl, s);         \
            case 4: return launch_gemm_t<E, 4, 8>(a, ma, pl, s);         \
            case 5: return launch_gemm_t<E, 2, 2>(a, ma, pl, s);         \
            case 6: return launch_gemm_t<E, 2, 4>(a, ma, pl, s);         \
            case 7: return launch_gemm_t<E, 4, 3>(a, ma, pl, s);         \
            case 8: return launch_gemm_t<E, 4, 5>(a, ma, pl, s);         \
            case 9: return launch_gemm_t<E, 4, 7>(a, ma, pl, s);         \
            default: return launch_gemm_t<E, 2, 3>(a, ma, pl, s);        \
        }
    switch (epi) {
        SWIFT_GEMM_CASE(EPI_QKV)
        SWIFT_GEMM_CASE(EPI_RESID)
        SWIFT_GEMM_CASE(EPI_SWIGLU)
    }
#undef SWIFT_GEMM_CASE
    return hipErrorInvalidValue;
}

}  // namespace swift
