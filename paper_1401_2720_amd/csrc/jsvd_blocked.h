// The one-sided Jacobi method on a matrix that one workgroup owns: the
// helpers and the two-level (blocked) sweep loop shared by the batched path
// (a whole small problem per workgroup) and by the inner level of the dense
// path's widest blocks (the third blocking level: a block Jacobi with
// 16-column sub-blocks on the Cholesky factor of a 128-column pivot block).
#pragma once

#include <type_traits>

#include "jsvd_device.h"

namespace jsvd {

namespace {

__device__ __forceinline__ double hw_sum(double v) {
    v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);  // row_half_mirror
    v += dpp_mov<0x140>(v);  // row_mirror
    const long long x = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_ds_swizzle((int)x, 0x401F);         // lane ^ 16
    const int hi = __builtin_amdgcn_ds_swizzle((int)(x >> 32), 0x401F);
    return v + __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Order the LDS accesses of one wave around this point: what the wave
// wrote before is what its lanes read after (the wave's LDS operations
// complete in order).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Relative orthogonality test (subphase 2, reading: <= skips) and the
// trigonometric rotation, eqs. (4.3)-(4.6) with t = +1 and cs_2: refined
// reciprocal and square roots inside [2^-900, 2^900], IEEE outside.
__device__ __forceinline__ bool trig_pair(double hpp, double hqq, double hpq, double tol,
                                          double &tn, double &cs) {
    bool clamped;
    if (in_fast_range(hpp) && in_fast_range(hqq) && in_fast_range(fabs(hpq))) {
        if (fabs(hpq) <= tol * nsqrt(hpp) * nsqrt(hqq)) return false;
        rotation_fast(hpp, hqq, hpq, 1, tn, cs, clamped);
    } else {
        if (!(hpq != 0.0) || fabs(hpq) <= tol * sqrt(hpp) * sqrt(hqq)) return false;
        rotation(hpp, hqq, hpq, 1, tn, cs, clamped);
    }
    return true;
}

// ---------------------------------------------------------------- blocked
// Problems with many columns take the two-level method of the dense path
// inside their workgroup: block-columns of kBlkW columns, the closest
// parallel strategy of order nb on the blocks, and for every pivot
// block-pair the Gram matrix (2.7), one sweep of the pointwise method on it
// accumulating V' (Section 4.3, block-oriented) and [G_p G_q] V',
// [V_p V_q] V' (2.9), skipped when the pair did not rotate (Section 4.4).  A
// pair whose Gram matrix already passes the relative orthogonality test
// everywhere is left alone.  Up to kBlkPairs pivot pairs are in flight: two
// waves per pair form the Gram matrix (rows split, FP64 MFMA) and apply V'
// (FP64 MFMA).  G and V stay in their global buffers; H and V' live in LDS,
// small enough for two workgroups (two problems) per CU, which hide each
// other's latencies.
constexpr int kBlkW = 16, kBlkBW = 2 * kBlkW, kBlkLD = kBlkBW + 1, kBlkPairs = 4;
constexpr int kBlkThreads = 512;  // 8 waves: two per pivot pair in the Gram and update phases
typedef double d2a __attribute__((ext_vector_type(2), aligned(8)));  // a 16-byte load
constexpr int kBlkMat = kBlkBW * kBlkLD;  // doubles of one H or V'

// The lane number, opaque to the compiler, so that what is computed from it
// is computed where it is used: hoisted out of the group loop, the addresses
// of all phases together spill (128 registers).
__device__ __forceinline__ int fresh_lane() {
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

// X[0:rows, cols of pq] <- X[0:rows, cols of pq] V' for the rows of one
// wave (16-row slices from row 16 sub, stride 16 nsub), V' row-major in LDS
// with leading dimension kBlkLD.  All loads of a slice precede its stores.
__device__ __forceinline__ void blk_rows_update(double *X, int ldx, int rows, int2 pq, int n,
                                                const double *vs, int sub, int nsub) {
    constexpr int KS = kBlkBW / 4;
    const int lane = fresh_lane(), i16 = lane & 15, grp = lane >> 4;
    auto load = [&](int base, double (&bx)[KS]) __attribute__((always_inline)) {
        const int row = base + i16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int gc = (int)pair_col(4 * ks + grp, kBlkW, pq);
            bx[ks] = (row < rows && gc < n) ? X[gc * ldx + row] : 0.0;
        }
    };
    double bx[KS];
    if (16 * sub < rows) load(16 * sub, bx);
    for (int base = 16 * sub; base < rows; base += 16 * nsub) {
        // V' is re-read from LDS in every slice rather than held in registers
        asm volatile("" ::: "memory");
        const int row = base + i16;
        const bool rv = row < rows;
        double by[KS] = {};
        if (base + 16 * nsub < rows) load(base + 16 * nsub, by);
#pragma unroll
        for (int jt = 0; jt < kBlkBW / 16; ++jt) {
            d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                acc = mfma16(vs[(4 * ks + grp) * kBlkLD + jt * 16 + i16], bx[ks], acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int gc = (int)pair_col(jt * 16 + grp + 4 * v, kBlkW, pq);
                if (rv && gc < n) X[gc * ldx + row] = acc[v];
            }
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bx[ks] = by[ks];
    }
}

// The inner sweep works on the 32 x 32 Gram matrices of the group's pivot
// pairs as jacobi_kernel does on its one (two-sided rotations, positions,
// slots; see there), with the roles spread over the workgroup so that the
// four matrices fill them: wave 0 computes the rotations of all four (16
// lanes each, a step ahead), waves 1-3 rotate H, waves 4-7 V'.  Both copies
// of an H share one array: even steps keep entry (x, y) at (min, max), odd
// ones at (max, min).
struct BlkLds {
    double H[kBlkPairs][kBlkMat];                         // then V', row-major
    __align__(16) double xch[kBlkPairs][2][kBlkW * kBlkBW];  // columns of V' on their way;
                                                          // before that the Gram sums
    double diag[kBlkPairs][kBlkBW];
    double2 prm[2][kBlkPairs][kBlkW];                     // published rotations: tan, +-cos
    unsigned dst[2][kBlkPairs][kBlkW];                    // next positions (times 8)
    uint2 tbl[(kBlkBW - 1) * kBlkW];                      // position_tables' entries
    unsigned vctl[(kBlkBW - 1) * kBlkW];                  // V waves' control words
};
constexpr int kBlkLdsDoubles = (int)(sizeof(BlkLds) / sizeof(double));
static_assert(sizeof(BlkLds) % sizeof(double) == 0, "whole doubles");
static_assert(3 * 4 * 64 <= 2 * kBlkW * kBlkBW, "Gram partial sums fit in xch");
static_assert(kBlkLdsDoubles == kBatchBlockLds, "host LDS bound of the blocked method");
static_assert(kBlkBW == kBatchInnerOrder && kBlkPairs == 4 && kBlkThreads == 512, "wave roles");

// pair bytes of the largest block strategy (order 16)
constexpr int kBlkMaxTable = (kBatchMaxN / kBlkW - 1) * (kBatchMaxN / kBlkW);
static_assert(kBlkMaxTable <= kBlkThreads, "one pair byte per thread");
constexpr int kBlkConverged = 1 << 16, kBlkNonfinite = 1 << 17;

// Wave 0 of blk_inner_sweep: lane 16 mx + k has pair k of matrix mx.
struct BlkRotations {
    static constexpr int NP = kBlkW, NS = kBlkBW - 1, LD = kBlkLD;
    BlkLds &L;
    const int mx, k, cm;
    const bool act;
    double off = 0.0;  // h_pq after the pair's rotation,
    unsigned off_at = 0;  // and where it goes
    // the next step's columns, as in jacobi_kernel
    unsigned h00 = 0, h01 = 0, h10 = 0, h11 = 0, Ia = 0, Jb = 0;
    bool fa = false, fb = false;
    int rots = 0, prop = 0;

    __device__ __forceinline__ BlkRotations(BlkLds &lds, int lane, const int *need, const int *cmax)
        : L(lds), mx(lane / NP), k(lane % NP), cm(cmax[lane / NP]), act(need[lane / NP] == 1) {}

    template <int PAR>
    static __device__ __forceinline__ unsigned at(unsigned x8, unsigned y8) {
        return PAR ? max(x8, y8) * LD + min(x8, y8) : min(x8, y8) * LD + max(x8, y8);
    }

    // decide, compute and publish the pair's rotation in the step of parity
    // PAR and table entry t; nxt: the next step's entry
    template <int PAR>
    __device__ __forceinline__ void rotate(uint2 t, uint2 nxt, double hpp, double hqq, double hpq) {
        constexpr double tol2 = kEps * kEps * kBlkBW;  // c(eps)^2 = 2w eps^2, exact
        const int cp = t.y & 0xff, cq = (t.y >> 8) & 0xff;
        hpp = act ? hpp : 1.0;
        hqq = act ? hqq : 1.0;
        hpq = act ? hpq : 0.0;
        const unsigned flip = (t.y & 0x10000u) << 15;
        const double up = __builtin_bit_cast(
            double, __builtin_bit_cast(unsigned long long, hqq - hpp) ^ ((unsigned long long)flip << 32));
        const bool swap = (up > 0.0) & (max(cp, cq) < cm);
        const unsigned mine = (unsigned)(__builtin_amdgcn_ballot_w64(swap) >> (NP * mx));
        const unsigned dp8 = ((t.x >> 16) & 0xff) * 8, dq8 = (t.x >> 24) * 8;
        const unsigned np8 = swap ? dq8 : dp8, nq8 = swap ? dp8 : dq8;
        bool rot = !(hpq * hpq <= tol2 * hpp * hqq);
        double tn, cs;
        bool clamped;
        rotation_h(hpp, hqq, hpq, false, tn, cs, clamped);
        if (!in_trig_range_bits(hpp, hqq)) {  // IEEE operations, as in jacobi_kernel
            const double tol = kEps * sqrt((double)kBlkBW);
            rot = hpq != 0.0 && !(fabs(hpq) <= tol * sqrt(hpp) * sqrt(hqq));
            rotation(hpp, hqq, hpq, 1, tn, cs, clamped);
        }
        tn = rot ? tn : 0.0;
        cs = rot ? cs : 1.0;
        off = rot ? 0.0 : hpq;
        rots += rot ? 1 : 0;
        prop += (rot && cs != 1.0) ? 1 : 0;
        char *const db = reinterpret_cast<char *>(L.diag[mx]);
        L.prm[PAR][mx][k] = make_double2(tn, swap ? -cs : cs);
        L.dst[PAR][mx][k] = np8 | nq8 << 16;
        *reinterpret_cast<double *>(db + np8) = fma(-tn, hpq, hpp);
        *reinterpret_cast<double *>(db + nq8) = fma(tn, hpq, hqq);
        off_at = at<1 - PAR>(dp8, dq8);
        const unsigned sp = nxt.x & 0xff, sq = (nxt.x >> 8) & 0xff;
        Ia = sp % NP;
        Jb = sq % NP;
        const unsigned r8 = (sp ^ ((mine >> Ia) & 1u) * NP) * 8, c8 = (sq ^ ((mine >> Jb) & 1u) * NP) * 8;
        const unsigned r8o = r8 ^ (NP * 8), c8o = c8 ^ (NP * 8);
        fa = r8 >= NP * 8;
        fb = c8 >= NP * 8;
        h00 = at<PAR>(r8, c8);
        h01 = at<PAR>(r8, c8o);
        h10 = at<PAR>(r8o, c8);
        h11 = at<PAR>(r8o, c8o);
        asm volatile("" : "+v"(h00), "+v"(h01), "+v"(h10), "+v"(h11), "+v"(off_at));
    }

    // step st of parity PAR: the rotation of step st + 1
    template <int PAR>
    __device__ __forceinline__ void ahead(int st, uint2 &t0, uint2 &t1) {
        char *const hb = reinterpret_cast<char *>(L.H[mx]);
        auto ld = [&](unsigned o) { return *reinterpret_cast<const double *>(hb + o); };
        const double x00 = ld(h00), x01 = ld(h01), x10 = ld(h10), x11 = ld(h11);
        const double2 ra = L.prm[PAR][mx][Ia], rb = L.prm[PAR][mx][Jb];
        const double hpp = L.diag[mx][k], hqq = L.diag[mx][k + NP];
        *reinterpret_cast<double *>(hb + off_at) = off;
        const uint2 t = t0;
        t0 = t1;
        t1 = L.tbl[min(st + 3, NS - 1) * NP + k];
        const double ga = fa ? ra.x : -ra.x, gb = fb ? rb.x : -rb.x;
        const double x0 = fma(gb, x01, x00), x1 = fma(gb, x11, x10);
        rotate<1 - PAR>(t, t0, hpp, hqq, fabs(ra.y * rb.y) * fma(ga, x1, x0));
    }
};

// H waves of blk_inner_sweep: the 2 x 2 block of pairs (I, J), I < J, of one
// matrix in a step of parity PAR.
template <int PAR>
__device__ __forceinline__ void blk_rotate_block(BlkLds &L, int m, int I, int J) {
    constexpr int NP = kBlkW, LD = kBlkLD;
    char *const hb = reinterpret_cast<char *>(L.H[m]);
    auto ld = [&](int x, int y) {  // x < y
        return *reinterpret_cast<const double *>(hb + 8 * (PAR ? y * LD + x : x * LD + y));
    };
    const double b00 = ld(I, J), b01 = ld(I, J + NP), b10 = ld(J, I + NP), b11 = ld(I + NP, J + NP);
    const double2 ri = L.prm[PAR][m][I], rj = L.prm[PAR][m][J];
    const unsigned di = L.dst[PAR][m][I], dj = L.dst[PAR][m][J];
    const double cc = fabs(ri.y * rj.y);
    const double x0 = fma(-rj.x, b01, b00), y0 = fma(rj.x, b00, b01);
    const double x1 = fma(-rj.x, b11, b10), y1 = fma(rj.x, b10, b11);
    const unsigned A0 = di & 0xffff, A1 = di >> 16, B0 = dj & 0xffff, B1 = dj >> 16;
    auto put = [&](unsigned x8, unsigned y8, double v) {
        *reinterpret_cast<double *>(hb + BlkRotations::at<1 - PAR>(x8, y8)) = v;
    };
    put(A0, B0, cc * fma(-ri.x, x1, x0));
    put(A1, B0, cc * fma(ri.x, x0, x1));
    put(A0, B1, cc * fma(-ri.x, y1, y0));
    put(A1, B1, cc * fma(ri.x, y0, y1));
}

// V waves of blk_inner_sweep: one slot of matrix m in step st of parity PAR;
// vk the kept column, vr the other one, ctl the slot's control word.
template <int PAR>
__device__ __forceinline__ void blk_rotate_v(BlkLds &L, int m, int sl, int vrow, int st, double2 &vk,
                                             double2 &vr, unsigned &ctl) {
    constexpr int NP = kBlkW, NS = kBlkBW - 1, BW = kBlkBW;
    if (st > 0) vr = *reinterpret_cast<const double2 *>(&L.xch[m][1 - PAR][sl * BW + vrow]);
    const double2 r = L.prm[PAR][m][sl];
    const unsigned long long mask = (unsigned long long)(ctl & 0x80000000u) << 32;
    const double tk = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, r.x) ^ mask);
    const double c = fabs(r.y);
    const double2 k1 = make_double2(c * fma(-tk, vr.x, vk.x), c * fma(-tk, vr.y, vk.y));
    const double2 r1 = make_double2(c * fma(tk, vk.x, vr.x), c * fma(tk, vk.y, vr.y));
    const bool same = ((ctl & 0x40000000u) != 0) != (r.y < 0.0);
    vk = make_double2(same ? k1.x : r1.x, same ? k1.y : r1.y);
    vr = make_double2(same ? r1.x : k1.x, same ? r1.y : k1.y);
    if (st + 1 < NS) {
        *reinterpret_cast<double2 *>(reinterpret_cast<char *>(&L.xch[m][PAR][vrow]) + (ctl & 0xffff)) = vr;
        ctl = L.vctl[(st + 1) * NP + sl];
    }
}

// One inner sweep on the matrices k with need[k] == 1 (H and diag set); V' into
// H, row-major; their rotations added to rotk, the proper ones of this lane
// to prop.  cmax[k]: columns of pair k from there on are padding.  All 512
// threads; each role has its own loop, with the same barriers.
__device__ __forceinline__ void blk_inner_sweep(BlkLds &L, const int *need, const int *cmax,
                                                int *rotk, int &prop) {
    constexpr int NP = kBlkW, NS = kBlkBW - 1, LD = kBlkLD;
    static_assert(NS % 2 == 1, "the last step is an even one");
    const int lane = fresh_lane();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        BlkRotations r(L, lane, need, cmax);
        const int k = r.k;
        uint2 t0 = L.tbl[NP + k], t1 = L.tbl[2 * NP + k];
        r.rotate<0>(L.tbl[k], t0, L.diag[r.mx][k], L.diag[r.mx][k + NP],
                    L.H[r.mx][k * LD + k + NP]);
        __syncthreads();
        for (int st = 0; st + 1 < NS; st += 2) {
            r.ahead<0>(st, t0, t1);
            __syncthreads();
            r.ahead<1>(st + 1, t0, t1);
            __syncthreads();
        }
        __syncthreads();
        if (r.rots) atomicAdd(&rotk[r.mx], r.rots);
        prop += r.prop;
        __builtin_amdgcn_s_setprio(0);
    } else if (wave < 4) {
        // both halves of matrix wave - 1 (64 blocks each), and of waves 1 and
        // 2 half of matrix 3
        int bI[2], bJ[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int ht = lane + 64 * u, g = ht / NP, l = ht % NP;
            const bool first = l < NP - 1 - g;
            bI[u] = first ? g : NP - 2 - g;
            bJ[u] = first ? g + 1 + l : l;
        }
        const int m = wave - 1;
        const bool on = need[m] == 1, on3 = wave < 3 && need[3] == 1;
        const int I3 = wave == 2 ? bI[1] : bI[0], J3 = wave == 2 ? bJ[1] : bJ[0];
        auto step = [&](auto par) __attribute__((always_inline)) {
            constexpr int PAR = decltype(par)::value;
            if (on) {
                blk_rotate_block<PAR>(L, m, bI[0], bJ[0]);
                blk_rotate_block<PAR>(L, m, bI[1], bJ[1]);
            }
            if (on3) blk_rotate_block<PAR>(L, 3, I3, J3);
            __syncthreads();
        };
        __syncthreads();
        for (int st = 0; st + 1 < NS; st += 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
        __syncthreads();
    } else {
        // matrix vm, slots 4 u + lane / 16, two rows per lane
        const int vm = wave == 4 ? 3 : wave - 5, vrow = 2 * (lane % NP), vq = lane / NP;
        const bool on = need[vm] == 1;
        double2 vk[4], vr[4];
        unsigned ctl[4];
        auto kept_col = [&](int e, int &ck, int &cr) __attribute__((always_inline)) {
            const unsigned t = L.tbl[e].y;
            const bool ky = (t & 0x20000u) != 0;
            ck = (ky ? t >> 8 : t) & 0xff;
            cr = (ky ? t : t >> 8) & 0xff;
        };
        auto step = [&](auto par, int st) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (on) blk_rotate_v<decltype(par)::value>(L, vm, 4 * u + vq, vrow, st, vk[u], vr[u], ctl[u]);
            __syncthreads();
        };
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // V' = I
            const int sl = 4 * u + vq;
            int ck, cr;
            kept_col(sl, ck, cr);
            vk[u] = make_double2(vrow == ck ? 1.0 : 0.0, vrow + 1 == ck ? 1.0 : 0.0);
            vr[u] = make_double2(vrow == cr ? 1.0 : 0.0, vrow + 1 == cr ? 1.0 : 0.0);
            ctl[u] = L.vctl[sl];
        }
        __syncthreads();
        for (int st = 0; st + 1 < NS; st += 2) {
            step(std::integral_constant<int, 0>{}, st);
            step(std::integral_constant<int, 1>{}, st + 1);
        }
        step(std::integral_constant<int, 0>{}, NS - 1);
        double *const v = L.H[vm];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int ck, cr;
            kept_col((NS - 1) * NP + 4 * u + vq, ck, cr);
            v[vrow * LD + ck] = vk[u].x;
            v[(vrow + 1) * LD + ck] = vk[u].y;
            v[vrow * LD + cr] = vr[u].x;
            v[(vrow + 1) * LD + cr] = vr[u].y;
        }
    }
    __syncthreads();
}

// The sweep loop of the blocked method on one problem (G: m x n, ld m; V:
// n x n, ld n, identity on entry, or null).  lds holds kBlkLdsDoubles; jac:
// position_tables' tables of order 32.  Columns from n_real on are the caller's
// padding, orthogonal to all others: they keep their places.
// Returns the sweeps performed (max_sweeps <= 0xffff), plus kBlkConverged
// when a sweep performed no proper rotation and kBlkNonfinite when a pivot
// Gram matrix held a NaN or an infinity.  stats (LDS, three ints the caller
// zeroes, or null) accumulates the rotations, the proper rotations and the
// pivot pairs whose V' was applied.
__device__ __forceinline__ int blocked_sweeps(double *G, double *V, int m, int n, int n_real,
                                              int max_sweeps,
                                              const int *tbl_order, const int64_t *tbl_off,
                                              const unsigned char *tbls, const unsigned char *jac,
                                              double *lds, int *stats = nullptr) {
    __shared__ int2 s_pq[kBlkPairs];
    __shared__ int s_need[kBlkPairs], s_rotk[kBlkPairs], s_cmax[kBlkPairs], s_prop, s_bad;
    __shared__ unsigned char s_pos0[kBlkBW], s_row[kBlkMaxTable];
    BlkLds &L = *reinterpret_cast<BlkLds *>(lds);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = (n + kBlkW - 1) / kBlkW;
    const int NB = tbl_order[nb];
    const unsigned char *btbl = tbls + tbl_off[NB >> 1];
    const double tol = kEps * sqrt((double)kBlkBW);  // c(eps) at the inner level, n^ = 2w
    const double tol2 = kEps * kEps * kBlkBW;
    const int wk = wave >> 1, sub = wave & 1;  // pair and half of a wave's Gram / update work

    constexpr int kEntries = (kBlkBW - 1) * kBlkW;
    static_assert(kEntries <= kBlkThreads, "one table entry per thread");
    if (tid < kEntries) {
        const uint2 t = reinterpret_cast<const uint2 *>(jac)[tid];
        L.tbl[tid] = t;
        // where the sent column goes (bytes in xch); bit 31: the kept column is
        // y; bit 30: it is kept again
        L.vctl[tid] = (t.y >> 24) * (kBlkBW * 8) | (t.y & 0x20000u) << 14 | (t.y & 0x40000u) << 12;
    }
    if (tid < kBlkBW) s_pos0[tid] = jac[8 * kEntries + tid];
    if (tid < (NB - 1) * NB) s_row[tid] = btbl[tid];  // the block strategy

    int sweeps = 0, result = 0;
    if (tid == 0) s_bad = 0;
    while (sweeps < max_sweeps) {
        if (tid == 0) s_prop = 0;
        int prop = 0;  // proper rotations of this lane's pivot pairs (wave 0)
        for (int st = 0; st < NB - 1; ++st) {
            const unsigned char *row = s_row + st * NB;
            int slot = 0;
            for (;;) {
                // the next pivot pairs of the step with a block inside the
                // problem (the same walk in every thread)
                __syncthreads();  // the previous group is done with s_pq, s_rotk
                int npg = 0;
                while (slot < NB / 2 && npg < kBlkPairs) {
                    const int p = row[2 * slot], q = row[2 * slot + 1];
                    ++slot;
                    if (p < nb || q < nb) {
                        if (tid == 0) s_pq[npg] = make_int2(p, q);
                        ++npg;
                    }
                }
                if (npg == 0) break;
                if (tid < kBlkPairs) s_need[tid] = s_rotk[tid] = 0;
                __syncthreads();
                const int lane = fresh_lane(), i16 = lane & 15, grp = lane >> 4;

                // (1) Gram matrices: each wave sums its 16-row slices, the next
                // slice's loads issued before the products of the current one;
                // the two partial sums of a pair are added in wave order.
                // positions of the columns i and j of this lane's entries of H
                int pos_i[2][2], pos_j[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
#pragma unroll
                    for (int v = 0; v < 2; ++v) pos_i[t][v] = s_pos0[16 * t + grp + 4 * (v + 2 * sub)];
                    pos_j[t] = s_pos0[16 * t + i16];
                }
                d4 acc[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) acc[t] = d4{0.0, 0.0, 0.0, 0.0};
                int2 pq = make_int2(0, 0);
                double *const red = &L.xch[wk][0][0];
                if (wk < npg) {
                    pq = s_pq[wk];
                    const double *col[2];
                    bool valid[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int gc = (int)pair_col(16 * t + i16, kBlkW, pq);
                        valid[t] = gc < n;
                        col[t] = G + (valid[t] ? gc : 0) * m + 4 * grp;
                    }
                    const bool allv = (pq.y + 1) * kBlkW <= n;
                    auto load = [&](int base, double (&x)[2][4]) __attribute__((always_inline)) {
                        if (allv && base + 16 <= m) {
#pragma unroll
                            for (int t = 0; t < 2; ++t)
#pragma unroll
                                for (int s2 = 0; s2 < 2; ++s2) {
                                    const d2a v = *reinterpret_cast<const d2a *>(col[t] + base + 2 * s2);
                                    x[t][2 * s2] = v.x;
                                    x[t][2 * s2 + 1] = v.y;
                                }
                        } else {
#pragma unroll
                            for (int t = 0; t < 2; ++t)
#pragma unroll
                                for (int s2 = 0; s2 < 4; ++s2)
                                    x[t][s2] = (valid[t] && base + 4 * grp + s2 < m) ? col[t][base + s2] : 0.0;
                        }
                    };
                    double x[2][4];
                    if (16 * sub < m) load(16 * sub, x);
                    for (int base = 16 * sub; base < m; base += 32) {
                        double y[2][4] = {};
                        if (base + 32 < m) load(base + 32, y);
#pragma unroll
                        for (int s2 = 0; s2 < 4; ++s2) {
                            acc[0] = mfma16(x[0][s2], x[0][s2], acc[0]);
                            acc[1] = mfma16(x[0][s2], x[1][s2], acc[1]);
                            acc[2] = mfma16(x[1][s2], x[1][s2], acc[2]);
                        }
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int s2 = 0; s2 < 4; ++s2) x[t][s2] = y[t][s2];
                    }
                    // each wave passes on the half that the other one sums
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int v = 0; v < 2; ++v)
                            red[(6 * sub + 2 * t + v) * 64 + lane] = sub ? acc[t][v] : acc[t][v + 2];
                }
                __syncthreads();
                // entries (i, j), i <= j, of H to their places, v = 0, 1 by the
                // first wave, 2, 3 by the second; padding columns become unit vectors
                double hs[3][2];
                if (wk < npg) {
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int v = 0; v < 2; ++v) {
                            const double o = red[(6 * (1 - sub) + 2 * t + v) * 64 + lane];
                            const double h = sub ? o + acc[t][v + 2] : acc[t][v] + o;
                            const int i = (t == 2 ? 16 : 0) + grp + 4 * (v + 2 * sub);
                            const int j = (t == 0 ? 0 : 16) + i16;
                            const bool ok = pair_col(i, kBlkW, pq) < n && pair_col(j, kBlkW, pq) < n;
                            hs[t][v] = ok ? h : (i == j ? 1.0 : 0.0);
                            const int pi = pos_i[t == 2][v], pj = pos_j[t != 0];
                            if (i < j) L.H[wk][min(pi, pj) * kBlkLD + max(pi, pj)] = hs[t][v];
                            if (i == j) L.diag[wk][pi] = hs[t][v];
                        }
                    if (lane == 0) {
                        const int nq = n_real - pq.y * kBlkW;
                        s_cmax[wk] = nq > 0 ? kBlkW + min(kBlkW, nq) : min(kBlkW, n_real - pq.x * kBlkW);
                    }
                }
                __syncthreads();

                // (2) which pairs need the inner sweep: some (i, j) fails the
                // relative orthogonality test on H (reading: <= passes), on
                // squares where they cannot leave the normal range
                if (wk < npg) {
                    bool need = false, bad = false, wide = false;
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int v = 0; v < 2; ++v) {
                            const bool up = (t == 2 ? 16 : 0) + grp + 4 * (v + 2 * sub) < (t == 0 ? 0 : 16) + i16;
                            const double hii = L.diag[wk][pos_i[t == 2][v]], hjj = L.diag[wk][pos_j[t != 0]];
                            bad = bad || !(fabs(hs[t][v]) <= 0x1.fffffffffffffp+1023);
                            need = need || (up && !(hs[t][v] * hs[t][v] <= tol2 * hii * hjj));
                            wide = wide || (up && !in_trig_range_bits(hii, hjj));
                        }
                    if (__builtin_amdgcn_ballot_w64(wide)) {
                        need = false;
#pragma unroll
                        for (int t = 0; t < 3; ++t)
#pragma unroll
                            for (int v = 0; v < 2; ++v) {
                                const bool up = (t == 2 ? 16 : 0) + grp + 4 * (v + 2 * sub) < (t == 0 ? 0 : 16) + i16;
                                const double hii = L.diag[wk][pos_i[t == 2][v]], hjj = L.diag[wk][pos_j[t != 0]];
                                need = need || (up && hs[t][v] != 0.0 &&
                                                !(fabs(hs[t][v]) <= tol * sqrt(hii) * sqrt(hjj)));
                            }
                    }
                    const bool any_need = __builtin_amdgcn_ballot_w64(need) != 0;
                    const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
                    if (lane == 0 && (any_need || any_bad))
                        atomicOr(&s_need[wk], (any_need ? 1 : 0) | (any_bad ? 2 : 0));
                }
                __syncthreads();
                int any = 0;
#pragma unroll
                for (int u = 0; u < kBlkPairs; ++u) {
                    const int f = u < npg ? s_need[u] : 0;
                    any |= f == 1;
                    // a NaN or infinity in a pair that is not left alone ends the
                    // problem after this sweep
                    if (tid == 0 && f == 3) s_bad = 1;
                }
                if (!any) continue;

                // (3) one inner sweep on H, V' into H's place
                blk_inner_sweep(L, s_need, s_cmax, s_rotk, prop);

                // (4) [G_p G_q] V' and [V_p V_q] V' for the pairs that rotated
                if (wk < npg && s_rotk[wk] > 0) {
                    const double *vs = L.H[wk];
                    blk_rows_update(G, m, m, pq, n, vs, sub, 2);
                    if (V) blk_rows_update(V, n, n, pq, n, vs, sub, 2);
                }
                if (stats && tid < npg && s_rotk[tid] > 0) {
                    atomicAdd(&stats[0], s_rotk[tid]);
                    atomicAdd(&stats[2], 1);
                }
            }
        }
        if (prop) atomicAdd(&s_prop, prop);
        __syncthreads();
        const int all = s_prop, bad = s_bad;
        if (stats && tid == 0) stats[1] += all;
        ++sweeps;
        __syncthreads();
        if (bad) {
            result = kBlkNonfinite;
            break;
        }
        if (all == 0) {
            result = kBlkConverged;
            break;
        }
    }
    return sweeps | result;
}

}  // namespace

}  // namespace jsvd
