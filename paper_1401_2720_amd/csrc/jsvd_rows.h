// The transformation of eq. (2.9) on a range of rows of one pivot
// block-pair: [X_p X_q] <- [X_p X_q] V'_pq, on FP64 MFMA, in place.  Used by
// the update kernel (rows of G and of V) and by the extra workgroups of the
// inner kernel's launch that update V for the previous p-step.
#pragma once

#include "jsvd_device.h"

namespace jsvd {

namespace {

// NW waves take 16-row slices of rows [r0, r1) and compute
// (X V')^T = V'^T X^T tile by tile: V' (staged by rows in LDS, vs holds at
// least BW * BW doubles: row i at vs + i BW, its column j at position
// j ^ (i mod 16), so that the staging stores of 16 consecutive rows of one
// column fall in 16 distinct banks, and the MFMA operand loads of 16
// consecutive columns of one row too) supplies the A operand, a slice of X
// the B operand (lane l reads row l%16 of local column 4*ks + l/16), and each
// result column is written back as 16 consecutive rows.  All loads of a
// slice precede its stores, so the update is in place.  The pair's columns
// are w consecutive columns of block P, then w of block Q; local columns
// past n (padding) are neither loaded nor stored.  JB of the BW/16 result
// tiles are accumulated at a time (fewer live registers for smaller JB).
// NTV: non-temporal loads and stores, for V, which is not read again before
// the next block sweep, so that it does not push G (read by the next Gram
// and update kernels) out of the caches.
// All 64 NW threads of the workgroup must call it (it contains a barrier).
template <int BW, int NW, int JB, bool NTV = false>
__device__ __forceinline__ void update_rows(double *X, int64_t ldx, int64_t r0, int64_t r1,
                                            int2 pq, int w, int64_t n, const double *vpr,
                                            double *vs) {
    constexpr int KS = BW / 4, JT = BW / 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, grp = lane >> 4;
    for (int e = threadIdx.x; e < BW * BW; e += 64 * NW) {
        const int i = e % BW, j = e / BW;
        vs[i * BW + (j ^ (i & 15))] = vpr[e];
    }
    __syncthreads();

    // Column addresses are recomputed per slice rather than kept in
    // registers, which keeps four waves per SIMD resident.
    double *XP = X + (int64_t)pq.x * w * ldx, *XQ = X + (int64_t)pq.y * w * ldx;
    const int64_t np = n - (int64_t)pq.x * w, nq = n - (int64_t)pq.y * w;
    for (int64_t base = r0 + wave * 16; base < r1; base += 16 * NW) {
        // re-read V' from LDS in every slice instead of pinning it in 2w^2/64
        // registers per lane (keeps the occupancy of this streaming code up)
        asm volatile("" ::: "memory");
        const int64_t row = base + i16;
        const bool rv = row < r1;
        double b[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int c = 4 * ks + grp;
            const bool in_p = c < w;
            const int lc = in_p ? c : c - w;
            const double *src = (in_p ? XP : XQ) + (int64_t)lc * ldx + row;
            b[ks] = (rv && lc < (in_p ? np : nq))
                        ? (NTV ? __builtin_nontemporal_load(src) : *src)
                        : 0.0;
        }
#pragma unroll
        for (int j0 = 0; j0 < JT; j0 += JB) {
            d4 acc[JB];
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) acc[jb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int jb = 0; jb < JB; ++jb)
                    acc[jb] = mfma16(vs[(4 * ks + grp) * BW + (j0 + jb) * 16 + (i16 ^ ((4 * ks + grp) & 15))],
                                     b[ks], acc[jb]);
#pragma unroll
            for (int jb = 0; jb < JB; ++jb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int c = (j0 + jb) * 16 + grp + 4 * v;
                    const bool in_p = c < w;
                    const int lc = in_p ? c : c - w;
                    if (rv && lc < (in_p ? np : nq)) {
                        double *dst = (in_p ? XP : XQ) + (int64_t)lc * ldx + row;
                        if (NTV)
                            __builtin_nontemporal_store(acc[jb][v], dst);
                        else
                            *dst = acc[jb][v];
                    }
                }
        }
    }
}

// The same for the pivot pairs of two consecutive p-steps at once, on the four
// blocks of a quad (step_quads; w = 32): (a0 a1) and (b0 b1) by the first
// p-step's V', then a pair of {a0, a1} x {b0, b1} and the other one by the
// second's.  The results of the first product of a 16-row slice are, lane by
// lane, the B operands of the second (lane l holds row l%16 of columns
// l/16 + 4v), so X is read and written once.  vs holds the four V' (16384
// doubles) laid out as in update_rows; the columns of the first two, and rows
// and columns of the last two, are taken round by w where it takes that to
// bring a0 (b0; a0, a1) first.  A pair that did not rotate takes part with the
// identity.  Bound by the MFMAs: 256 per wave and slice (64 cycles each: 16384, or 7
// us, for every slice that a SIMD takes) against 32 KiB of traffic.
template <int NW>
__device__ __forceinline__ void update_quad_rows(double *X, int64_t ldx, int64_t r0, int64_t r1,
                                                 const int *qd, const StepArgs &a, double *vs,
                                                 int *next) {
    constexpr int BW = 64, W = 32, KS = 16;
    const int2 pa = a.prev_pairs[qd[0]], pb = a.prev_pairs[qd[1]];
    const int2 nx = a.prev2_pairs[qd[2]], ny = a.prev2_pairs[qd[3]];
    const int a0 = qd[4], b0 = qd[5];
    const int a1 = a0 == pa.x ? pa.y : pa.x, b1 = b0 == pb.x ? pb.y : pb.x;
    const int off[4] = {a0 == pa.x ? 0 : W, b0 == pb.x ? 0 : W, nx.x == a0 ? 0 : W,
                        ny.x == a1 ? 0 : W};
    const int rot[4] = {a.prev_pair_rot[qd[0]], a.prev_pair_rot[qd[1]], a.prev2_pair_rot[qd[2]],
                        a.prev2_pair_rot[qd[3]]};
    if ((rot[0] | rot[1] | rot[2] | rot[3]) == 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i16 = lane & 15, grp = lane >> 4;
    const int64_t n = a.n;
    const bool whole = (int64_t)(max(max(pa.x, pa.y), max(pb.x, pb.y)) + 1) * W <= n;
    const uint32_t lofs = (uint32_t)((grp * ldx + i16) * 8);  // the host: ldx <= 2^26
    auto at = [&](int64_t e) {  // element e of X for lane 0, this lane's of its slice
        return reinterpret_cast<double *>(reinterpret_cast<char *>(X + e) + lofs);
    };
    auto load = [&](int64_t base, double (&x)[2 * KS]) __attribute__((always_inline)) {
        // the column bases are formed per slice on the scalar unit
        int64_t ld = ldx;
        asm volatile("" : "+s"(ld));
        auto col = [&](int k) {
            const int b = k < 8 ? pa.x : k < 16 ? pa.y : k < 24 ? pb.x : pb.y;
            return (int64_t)b * W + 4 * (k & 7);
        };
        if (whole && base + 16 <= r1) {
#pragma unroll
            for (int k = 0; k < 2 * KS; ++k) x[k] = __builtin_nontemporal_load(at(col(k) * ld + base));
        } else {
            const bool rv = base + i16 < r1;
#pragma unroll
            for (int k = 0; k < 2 * KS; ++k) {
                x[k] = 0.0;
                if (rv && col(k) + grp < n) x[k] = *at(col(k) * ld + base);
            }
        }
    };
    auto store = [&](int b, int t, int64_t base, d4 d) __attribute__((always_inline)) {
        int64_t ld = ldx;
        asm volatile("" : "+s"(ld));
        const int64_t col = (int64_t)b * W + 16 * t;
        if (whole && base + 16 <= r1) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                __builtin_nontemporal_store(d[v], at((col + 4 * v) * ld + base));
        } else {
            const bool rv = base + i16 < r1;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (rv && col + 4 * v + grp < n) *at((col + 4 * v) * ld + base) = d[v];
        }
    };
    // tile j of the product with matrix mat (a tile at a time: 128 registers
    // hold the operands and one result)
    auto tile = [&](int mat, int j, auto operand) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");  // V' is read for each tile
        d4 d = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int i = 4 * k + grp;
            d = mfma16(vs[mat * BW * BW + i * BW + 16 * j + (i16 ^ (i & 15))], operand(k), d);
        }
        return d;
    };

    // V', all of a thread's elements in flight together (those of a pair that
    // did not rotate are old ones, not used)
    constexpr int U = BW * BW / (64 * NW);
    double vv[4][U];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const double *src = (m < 2 ? a.prev_vprime : a.prev2_vprime) + (size_t)qd[m] * BW * BW;
#pragma unroll
        for (int u = 0; u < U; ++u) vv[m][u] = src[threadIdx.x + 64 * NW * u];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = threadIdx.x + 64 * NW * u, i = e % BW, j = e / BW;
            const int i1 = m < 2 ? i : (i - off[m]) & (BW - 1), j1 = (j - off[m]) & (BW - 1);
            vs[m * BW * BW + i1 * BW + (j1 ^ (i1 & 15))] = rot[m] ? vv[m][u] : (i == j ? 1.0 : 0.0);
        }
    if (threadIdx.x == 0) *next = NW;
    __syncthreads();
    // the next slice goes to the wave that is done first
    for (int sl = wave; r0 + 16 * sl < r1;) {
        const int64_t base = r0 + 16 * sl;
        double x[2 * KS];
        load(base, x);
        d4 da[4], db[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) da[j] = tile(0, j, [&](int k) { return x[k]; });
#pragma unroll
        for (int j = 0; j < 4; ++j) db[j] = tile(1, j, [&](int k) { return x[KS + k]; });
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                store(j < 2 ? (m ? a1 : a0) : (m ? b1 : b0), j % 2, base,
                      tile(2 + m, j, [&](int k) {
                          return k < 8 ? da[2 * m + k / 4][k % 4] : db[2 * m + (k - 8) / 4][k % 4];
                      }));
        int got = 0;
        if (lane == 0) got = atomicAdd(next, 1);
        sl = __builtin_amdgcn_readfirstlane(got);
    }
}

}  // namespace

}  // namespace jsvd
