// p-step kernel 2 of 3: sum of the partial Gram matrices and the inner
// pointwise Jacobi of the pivot block-pair with V'_pq accumulated (Section
// 4.3), all in LDS, one workgroup per pivot block-pair: jacobi_kernel rotates
// H_pq itself; inner_kernel works on a triangular factor R, H_pq = R^T R
// (Section 4.1), for the scaled mode and the QR shortening.  Further
// workgroups of the same launch apply the previous p-step's V'_pq
// to V (eq. (2.9)): V lies off the path from one p-step's Gram matrices to
// the next, and these workgroups stream it through HBM on the CUs that the
// pivot pairs leave idle.
#include <type_traits>

#include "jsvd_qrpair.h"
#include "jsvd_rows.h"

namespace jsvd {

namespace {

// ------------------------------------------------- inner, on a factor R
// For what does not run on the Gram matrix: the scaled mode, whose exponents
// go with R's columns, and the QR shortening, which forms R without H.
//
// One workgroup of 16 * BW threads per pivot block-pair (BW = 2w).  R and V'
// live in LDS, column-major with a padded leading dimension.
//
// Cholesky (Section 4.1) by block rows of 16: wave 0 factors a block row
// with lane j holding column j, pivots and multipliers broadcast by
// readlane; then the block row's contribution is subtracted from the
// trailing part of H on FP64 MFMA, one wave per 16 x 16 tile.
//
// Inner Jacobi (Section 4.3): a p-step of the inner strategy has BW/2 pivot
// pairs.  Threads [0, 4 BW) handle R: every pair is one DPP half row of 8
// lanes, lane x owning rows x, x + 8, ... of the pair's two columns; the
// three dot products (subphase 1) are half-row sums, each half row decides
// and computes its rotation (subphases 2-5), applies it to its columns of R
// (subphase 6) and publishes it.  Threads [4 BW, 8 BW) apply the previous
// p-step's rotations to V' at the same time, so V' never lies on the path of
// the rotations; the remaining waves only keep the barriers.  One barrier
// per p-step.  The rotation formulas are computed once per pair and wave
// lane group, so fewer lanes per pair (more rows per lane) means fewer
// waves repeating them: with 8 lanes the R side is one wave per SIMD.
template <int BW>
struct InnerCfg {
    static constexpr int kThreads = BW * 16;
    static constexpr int kLanes = 8;             // lanes per pivot pair
    static constexpr int kRows = BW / kLanes;    // rows per lane and column
    static constexpr int kPairs = BW / 2;        // pivot pairs per p-step
    static constexpr int kHalf = kPairs * kLanes;  // threads on R (and on V')
    static constexpr int kSteps = BW - 1;        // p-steps per inner sweep
    static constexpr int kLD = BW + 1;
};

// HYP: the problem has columns of both signs (J != I); without it every
// pair is trigonometric and the hyperbolic branches are compiled out.
// SC: scaled mode (badly scaled input).  The partial sums are of
// H~ = D^-1 H D^-1, D = diag(2^e_c); R~ = R D^-1 is kept with the column
// exponents e_c in LDS.  A pair's dot products on R~ are those of R times
// 2^-(e_p+e_q) after the factors 2^(e_p-e_q), 2^(e_q-e_p) on h_pp, h_qq, so
// the orthogonality test (scale free) and the rotation formulas see the same
// values as on R up to one exact power of two; the rotation is applied to R~
// with tan phi scaled by 2^(e_q-e_p) (into column p) and 2^(e_p-e_q) (into
// column q), to V' unscaled, and a swap also swaps the two exponents.  At
// the end the exponents of the transformed columns go back to global memory.
// Without SC: the QR shortening only.
template <int BW, bool HYP, bool SC>
__global__ __launch_bounds__(InnerCfg<BW>::kThreads) void inner_kernel(StepArgs a) {
    using Cfg = InnerCfg<BW>;
    constexpr int NT = Cfg::kThreads;
    constexpr int HALF = Cfg::kHalf;
    constexpr int NWAVES = NT / 64;
    constexpr int LD = Cfg::kLD;
    constexpr int ROWS = Cfg::kRows;
    constexpr int NP = Cfg::kPairs;
    constexpr int NS = Cfg::kSteps;
    constexpr int EPT = BW * BW / NT;   // Gram entries summed per thread
    __shared__ double R[BW * LD];
    __shared__ double Vp[BW * LD];
    __shared__ unsigned char tb[NS * BW];   // inner strategy, (p, q) per pair and step
    __shared__ unsigned char sfl[NS * NP];  // pair flags per step, see below
    __shared__ d4 prm[2][NP];               // published rotations: mtn, tn, cs, flags
    __shared__ int flags[2];                // [0] NaN met, [1] zero pivots
    __shared__ int cnt[NWAVES][4];
    __shared__ int ex[BW];                  // scaled mode: column exponents

    const bool qrf = !SC || a.qrf;
    if (blockIdx.x >= a.npairs) {
        // V <- V V'_pq of the previous p-step on one chunk of rows; these
        // workgroups come after the pivot pairs' in the grid, so the pairs
        // are dispatched first
        // start about 7 us late (2 x 127 x 64 cycles): the pair workgroups'
        // partial Gram loads then do not queue behind this V stream
        __builtin_amdgcn_s_sleep(127);
        __builtin_amdgcn_s_sleep(127);
        const int idx = blockIdx.x - a.npairs;
        const int vpair = idx / a.prev_chunks, chunk = idx % a.prev_chunks;
        if (a.prev_pair_rot[vpair] == 0) return;
        const int64_t r0 = (int64_t)chunk * a.prev_rows;
        const int64_t r1 = min(a.n, r0 + (int64_t)a.prev_rows);
        update_rows<BW, NWAVES, 1, true>(a.V, a.ldv, r0, r1, a.prev_pairs[vpair], a.w, a.n,
                                a.prev_vprime + (size_t)vpair * BW * BW, R);
        return;
    }
    const int pair = blockIdx.x;
    const int2 pq = a.pairs[pair];
    const int tid = threadIdx.x;
    if ((int64_t)pq.x * a.w >= a.n) {
        if (tid == 0) a.pair_rot[pair] = 0;
        return;
    }
    const int lane = tid & 63, wave = tid >> 6;

    // ---- H_pq: the partial Gram matrices summed in split order (upper
    // triangle, all loads of a batch of 8 splits issued together); padding
    // columns become unit vectors orthogonal to everything.  The strategy
    // table's loads go first, then the first batch, so that the table setup
    // below waits for its own loads only.
    constexpr int TE = (NS * NP + NT - 1) / NT;   // table entries per thread
    unsigned short tpq[TE];
#pragma unroll
    for (int u = 0; u < TE; ++u) {
        const int e = tid + u * NT;
        tpq[u] = e < NS * NP ? reinterpret_cast<const unsigned short *>(a.inner_tbl)[e] : 0;
    }
    const double *hp = a.hpart + (size_t)pair * a.splits * BW * BW;
    double hv[8][EPT];
    auto load_batch = [&](int s0) {
#pragma unroll
        for (int sp = 0; sp < 8; ++sp)
#pragma unroll
            for (int u = 0; u < EPT; ++u) {
                const int e = tid + u * NT;
                hv[sp][u] = (s0 + sp < a.splits && e / BW <= e % BW)
                                ? hp[(size_t)(s0 + sp) * BW * BW + e] : 0.0;
            }
    };
    if (!qrf) load_batch(0);

    // ---- strategy table and pair flags: 1 hyperbolic (kp < n+ <= kq),
    // 2 a padding column, 4 both columns in the + part, 8 both in the - part
#pragma unroll
    for (int u = 0; u < TE; ++u) {
        const int e = tid + u * NT;
        if (e < NS * NP) {
            const int p = tpq[u] & 0xff, q = tpq[u] >> 8;
            tb[2 * e] = (unsigned char)p;
            tb[2 * e + 1] = (unsigned char)q;
            const int64_t kp = pair_col(p, a.w, pq), kq = pair_col(q, a.w, pq);
            int f = (kp < a.n_plus && kq >= a.n_plus) ? 1 : 0;
            f |= (kq >= a.n || kp >= a.n) ? 2 : 0;
            f |= (kq < a.n_plus) ? 4 : ((kp >= a.n_plus) ? 8 : 0);
            sfl[e] = (unsigned char)f;
        }
    }

    if (qrf) {
        // QR shortening (Section 4.2): the splits' triangular factors folded
        // into R by the peel-off procedure, V' (still free) holding the next
        // factor; then V' = I
        auto load_factor = [&](double *X, int sp) {
            for (int e = tid; e < BW * BW; e += NT) {
                const int i = e / BW, j = e % BW;
                X[j * LD + i] = i <= j ? hp[(size_t)sp * BW * BW + e] : 0.0;
            }
        };
        load_factor(R, 0);
        for (int sp = 1; sp < a.splits; ++sp) {
            load_factor(Vp, sp);
            __syncthreads();
            peel_off<BW, NT>(R, Vp, LD);
        }
        for (int e = tid; e < BW * BW; e += NT) {
            const int i = e % BW, j = e / BW;
            Vp[j * LD + i] = (i == j) ? 1.0 : 0.0;
        }
    } else {
        double s[EPT];
#pragma unroll
        for (int u = 0; u < EPT; ++u) s[u] = 0.0;
        for (int s0 = 0; s0 < a.splits; s0 += 8) {
            if (s0) load_batch(s0);
#pragma unroll
            for (int sp = 0; sp < 8; ++sp)
#pragma unroll
                for (int u = 0; u < EPT; ++u)
                    if (s0 + sp < a.splits) s[u] += hv[sp][u];
        }
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const int e = tid + u * NT, i = e / BW, j = e % BW;
            double h = (i <= j) ? s[u] : 0.0;
            if (i <= j && (pair_col(i, a.w, pq) >= a.n || pair_col(j, a.w, pq) >= a.n))
                h = (i == j) ? 1.0 : 0.0;
            R[j * LD + i] = h;
            Vp[j * LD + i] = (i == j) ? 1.0 : 0.0;
        }
    }
    if (tid < 2) flags[tid] = 0;
    if constexpr (SC) {
        for (int c = tid; c < BW; c += NT) {
            const int64_t gc = pair_col(c, a.w, pq);
            ex[c] = gc < a.n ? a.colexp[gc] : 0;
        }
    }
    __syncthreads();


    // ---- QR shortening: R is there; a NaN or infinity on its diagonal
    // stops the pair as a non-finite Cholesky pivot does
    if (qrf) {
        for (int c = tid; c < BW; c += NT)
            if (!(fabs(R[c * LD + c]) <= 0x1.fffffffffffffp+1023)) flags[0] = 1;
        __syncthreads();
    }

    // ---- nothing to do: when every pair (i, j) of the block pair already
    // passes the relative orthogonality test on H itself, no rotation can
    // happen in the inner sweep (no column of R would change, so its dot
    // products stay those of H up to the rounding of the Cholesky factor),
    // and the pair is left alone as if the sweep had rotated nothing.
    if (!qrf) {
        const double tol = kEps * sqrt((double)BW);
        bool need = false;
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const int e = tid + u * NT, i = e / BW, j = e % BW;
            if (i < j) {
                const double hij = R[j * LD + i], hii = R[i * LD + i], hjj = R[j * LD + j];
                need = need || (hij != 0.0 && !(fabs(hij) <= tol * sqrt(hii) * sqrt(hjj)));
            }
        }
        if (!__syncthreads_or(need ? 1 : 0)) {
            if (tid == 0) a.pair_rot[pair] = 0;
            return;
        }
    }

    // ---- Cholesky H = R^T R (Section 4.1).  A pivot that is not positive
    // (H only semidefinite: dependent columns) makes its row of R zero; a
    // pivot that is NaN or infinite stops the pair.  The panel has no branch,
    // so the updates of one pivot overlap the square root of the next; row k
    // of R is H's row k times 1/sqrt(h_kk).
    if (!qrf) {
#pragma unroll
    for (int kb = 0; kb < BW / 16; ++kb) {
        if (wave == 0) {
            const int j = lane;
            double hb[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) hb[i] = (j < BW) ? R[j * LD + 16 * kb + i] : 0.0;
            int zero_pivots = 0, nan_met = 0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int kk = 16 * kb + k;
                const double hkk = lane_value(hb[k], kk);
                const bool bad = !(fabs(hkk) <= 0x1.fffffffffffffp+1023);  // NaN or infinite
                const bool pos = !bad && hkk > 0.0;
                nan_met |= bad ? 1 : 0;
                zero_pivots += (!bad && !pos) ? 1 : 0;
                double rs, d;
                rsqrt_sqrt(pos ? hkk : 1.0, rs, d);
                double r = (j == kk) ? d : hb[k] * rs;
                r = (pos && j >= kk) ? r : 0.0;
                hb[k] = r;
#pragma unroll
                for (int i = k + 1; i < 16; ++i) hb[i] = fma(-lane_value(r, 16 * kb + i), r, hb[i]);
            }
            if (j < BW) {
#pragma unroll
                for (int i = 0; i < 16; ++i) R[j * LD + 16 * kb + i] = (j >= 16 * kb + i) ? hb[i] : 0.0;
            }
            if (lane == 0) {
                flags[0] |= nan_met;
                flags[1] += zero_pivots;
            }
        }
        __syncthreads();
        if (kb + 1 < BW / 16) {
            // H(i, j) -= sum_k R(16 kb + k, i) R(16 kb + k, j) on the 16 x 16
            // tiles (ti, tj), kb < ti <= tj, one wave and 4 FP64 MFMAs per tile
            constexpr int TB = BW / 16;
            int idx = wave, ti = -1, tj = -1;
#pragma unroll
            for (int t0 = kb + 1; t0 < TB; ++t0) {
                if (ti < 0 && idx < TB - t0) {
                    ti = t0;
                    tj = t0 + idx;
                } else if (ti < 0) {
                    idx -= TB - t0;
                }
            }
            if (ti >= 0) {
                const int l16 = lane & 15, l4 = lane >> 4;
                d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int k = 16 * kb + 4 * c + l4;
                    acc = mfma16(R[(16 * ti + l16) * LD + k], R[(16 * tj + l16) * LD + k], acc);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + l4 + 4 * v, j = 16 * tj + l16;
                    if (i <= j) R[j * LD + i] -= acc[v];
                }
            }
            __syncthreads();
        }
    }
    }  // !qrf
    if (flags[0]) {
        if (tid == 0) {
            a.pair_rot[pair] = 0;
            atomicAdd(&a.counters[C_NONFINITE], 1ull);
        }
        return;
    }
    if (tid == 0 && flags[1]) atomicAdd(&a.counters[C_BREAKDOWN], (unsigned long long)flags[1]);

    // ---- inner Jacobi (Section 4.3)
    constexpr int LN = Cfg::kLanes;
    const bool on_r = tid < HALF;
    const bool on_v = !on_r && tid < 2 * HALF;
    const int gt = on_r ? tid : (on_v ? tid - HALF : 0);
    const int x = gt % LN;      // first row owned by this lane
    const int slot = gt / LN;   // pivot pair of this lane group
    const double tol = kEps * sqrt((double)BW);  // c(eps) = eps sqrt(nhat), nhat = 2w
    const double tol2 = kEps * kEps * BW;        // tol^2, exact
    int rot_total = 0, proper_total = 0, clamp_total = 0, sweeps = 0;

    for (int sw = 0; sw < a.max_inner_sweeps; ++sw) {
        int rot_sweep = 0;
        int p = tb[2 * slot], q = tb[2 * slot + 1], f = sfl[slot];
        for (int st = 0; st < NS + 1; ++st) {
            if (on_r) {
                if (st < NS) {
                    double rp[ROWS], rq[ROWS];
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        rp[r] = R[p * LD + x + LN * r];
                        rq[r] = R[q * LD + x + LN * r];
                    }
                    double hpp = 0.0, hqq = 0.0, hpq = 0.0;
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        hpp = fma(rp[r], rp[r], hpp);
                        hqq = fma(rq[r], rq[r], hqq);
                        hpq = fma(rp[r], rq[r], hpq);
                    }
                    hpp = group_sum<LN>(hpp);
                    hqq = group_sum<LN>(hqq);
                    hpq = group_sum<LN>(hpq);
                    // subphase 2: relative orthogonality (reading: <= skips),
                    // on squares where they cannot leave the normal range.
                    // h_pq != 0 implies h_pp, h_qq > 0.
                    const bool mid = in_trig_range(hpp, hqq);
                    bool rotate;
                    if (mid)
                        rotate = !(hpq * hpq <= tol2 * hpp * hqq);
                    else
                        rotate = hpq != 0.0 && !(fabs(hpq) <= tol * sqrt(hpp) * sqrt(hqq));
                    // subphase 4: hyperbolic iff kp < n+ <= kq
                    const int t = (HYP && (f & 1)) ? -1 : 1;
                    // scaled mode: the pair's h in one common scale
                    int dl = 0, ep = 0, eq = 0;
                    double sp = hpp, sq = hqq;
                    if constexpr (SC) {
                        ep = ex[p];
                        eq = ex[q];
                        dl = eq - ep;
                        sp = ldexp(hpp, -dl);
                        sq = ldexp(hqq, dl);
                    }
                    double tn = 0.0, cs = 1.0;
                    bool clamped = false;
                    if (rotate) {
                        if ((!SC && mid) ||
                            (in_fast_range(sp) && in_fast_range(sq) && in_fast_range(fabs(hpq))))
                            rotation_fast(sp, sq, hpq, t, tn, cs, clamped);
                        else
                            rotation(sp, sq, hpq, t, tn, cs, clamped);
                    }
                    // subphase 5: keep j*sigma^2 non-increasing for trigonometric
                    // pairs (h_pp' = h_pp - tn h_pq, h_qq' = h_qq + tn h_pq)
                    bool swap = false;
                    if (!(f & 3)) {
                        const double npp = fma(-tn, hpq, sp);
                        const double nqq = fma(tn, hpq, sq);
                        swap = (!HYP || (f & 4)) ? (npp < nqq) : ((f & 8) ? (npp > nqq) : false);
                    }
                    // subphase 6, (4.1) / (4.2).  cs == 1 multiplies exactly.
                    const double mtn = (t > 0) ? -tn : tn;
                    if (rotate || swap) {
                        const int cp = swap ? q : p, cq = swap ? p : q;
                        const double mtr = SC ? ldexp(mtn, dl) : mtn;
                        const double tr = SC ? ldexp(tn, -dl) : tn;
#pragma unroll
                        for (int r = 0; r < ROWS; ++r) {
                            const double np = cs * fma(mtr, rq[r], rp[r]);
                            const double nq = cs * fma(tr, rp[r], rq[r]);
                            R[cp * LD + x + LN * r] = np;
                            R[cq * LD + x + LN * r] = nq;
                        }
                        if (SC && swap && x == 0) {
                            ex[p] = eq;
                            ex[q] = ep;
                        }
                    }
                    if (x == 0) {
                        prm[st & 1][slot] = d4{mtn, tn, cs, (double)((rotate || swap ? 1 : 0) | (swap ? 2 : 0))};
                        rot_sweep += rotate ? 1 : 0;
                        proper_total += (rotate && cs != 1.0) ? 1 : 0;
                        clamp_total += clamped ? 1 : 0;
                    }
                    if (st + 1 < NS) {
                        p = tb[(st + 1) * BW + 2 * slot];
                        q = tb[(st + 1) * BW + 2 * slot + 1];
                        f = sfl[(st + 1) * NP + slot];
                    }
                }
            } else if (on_v && st >= 1) {
                // V' <- V' (rotation of p-step st - 1)
                const int s1 = st - 1;
                const d4 pr = prm[s1 & 1][slot];
                const int fl = (int)pr[3];
                if (fl & 1) {
                    const int vp = tb[s1 * BW + 2 * slot], vq = tb[s1 * BW + 2 * slot + 1];
                    const int cp = (fl & 2) ? vq : vp, cq = (fl & 2) ? vp : vq;
                    const double mtn = pr[0], tn = pr[1], cs = pr[2];
                    double xp[ROWS], xq[ROWS];
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        xp[r] = Vp[vp * LD + x + LN * r];
                        xq[r] = Vp[vq * LD + x + LN * r];
                    }
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        Vp[cp * LD + x + LN * r] = cs * fma(mtn, xq[r], xp[r]);
                        Vp[cq * LD + x + LN * r] = cs * fma(tn, xp[r], xq[r]);
                    }
                }
            }
            __syncthreads();
        }
        ++sweeps;
        rot_total += rot_sweep;
        int rs = rot_sweep;
        for (int off = 32; off >= 1; off >>= 1) rs += __shfl_xor(rs, off);
        if (lane == 0) cnt[wave][0] = rs;
        __syncthreads();
        int all = 0;
#pragma unroll
        for (int wv = 0; wv < NWAVES; ++wv) all += cnt[wv][0];
        __syncthreads();
        if (all == 0) break;  // no rotation in the inner sweep
    }

    // ---- write V'_pq and the counts
    for (int off = 32; off >= 1; off >>= 1) {
        rot_total += __shfl_xor(rot_total, off);
        proper_total += __shfl_xor(proper_total, off);
        clamp_total += __shfl_xor(clamp_total, off);
    }
    double *vout = a.vprime + (size_t)pair * BW * BW;
    for (int e = tid; e < BW * BW; e += NT) {
        const int i = e % BW, j = e / BW;
        vout[j * BW + i] = Vp[j * LD + i];
    }
    if (lane == 0) {
        cnt[wave][0] = rot_total;
        cnt[wave][1] = proper_total;
        cnt[wave][2] = clamp_total;
    }
    __syncthreads();
    if (tid == 0) {
        long long r = 0, pr = 0, cl = 0;
        for (int wv = 0; wv < NWAVES; ++wv) {
            r += cnt[wv][0];
            pr += cnt[wv][1];
            cl += cnt[wv][2];
        }
        a.pair_rot[pair] = (int)r;
        atomicAdd(&a.counters[C_ROT], (unsigned long long)r);
        atomicAdd(&a.counters[C_PROPER], (unsigned long long)pr);
        atomicAdd(&a.counters[C_CLAMP], (unsigned long long)cl);
        atomicAdd(&a.counters[C_INNER_SW], (unsigned long long)sweeps);
        if (r) atomicAdd(&a.counters[C_UPDATES], 1ull);
    }
    if constexpr (SC) {
        // exponents of the transformed columns (||g_c|| = ||r_c|| after the
        // update), written only when the update will run (some rotation)
        int all = 0;
#pragma unroll
        for (int wv = 0; wv < NWAVES; ++wv) all += cnt[wv][0];
        if (all != 0) {
            for (int c = tid; c < BW; c += NT) {
                const int64_t gc = pair_col(c, a.w, pq);
                double s2 = 0.0;
                for (int i = 0; i < BW; ++i) s2 = fma(R[c * LD + i], R[c * LD + i], s2);
                const double nrm = sqrt(s2);
                if (gc < a.n) a.colexp[gc] = ex[c] + (nrm > 0.0 && nrm <= 0x1p1000 ? ilogb(nrm) : 0);
            }
        }
    }
}

// ------------------------------------------------- inner, on the Gram matrix
// The inner Jacobi of a pivot block-pair carried out on H_pq itself: each
// rotation is applied to H from both sides, H <- J^T H J, instead of to the
// columns of its Cholesky factor R.  In exact arithmetic H = R^T R at every
// step, so the rotations are the ones of Section 4.3; in floating point the
// errors of both are relative to sqrt(h_ii h_jj) entry by entry (Demmel and
// Veselic, "Jacobi's method is more accurate than QR", SIAM J. Matrix Anal.
// Appl. 13, 1992), and G and V only ever see the product V' of the rotations.
// It takes no Cholesky factorization and no dot products: a pair's h_pp, h_qq
// and h_pq are entries of H.  Launch without a V stream, n = 4096, 2w = 64:
// 44.8 us (on R: 82); n = 1024, 2w = 32: 17.6 us (33.5).  It is bound by
// the chain of BW - 1 dependent steps, about 1050 cycles each at 2w = 32, of
// which some 560 for the LDS reads and the rotation's some 48 dependent FP64
// operations (10 cycles each), 300 to publish it and 150 at the barrier (where
// the pair's entry lies in H is in the table: with the swaps followed by address
// arithmetic in the chain, 18.3 us); at 2w = 64 about 1480, where three SIMDs issue
// some 300 vector instructions per step for the H and V waves and the LDS is busy
// for half of it.  What is on that chain is one wave's work:
//
//   wave 0      (rotations) one lane per pivot pair.  While the other waves
//               apply step s, it forms the entry h_pq of its pair of step
//               s + 1 from the 2 x 2 block of H before step s and the two
//               rotations of step s, decides and computes the rotation of
//               step s + 1 and publishes it;
//   H waves     one lane per 2 x 2 block (I, J), I < J, of pairs (two at
//               BW = 64): block read, rotated from both sides, written to
//               where step s + 1 has its columns;
//   V waves     V' <- V' J, four slots (pairs) per wave, a lane holding two
//               rows (four at BW = 64: two slots of two rows took 48.5 us) of its
//               slot's columns in registers.  From step to step a
//               slot keeps one column and passes the other one on through LDS
//               (position_tables).
//
// H lies in LDS by position, not by column: pair k of the coming step has
// its p at position k and its q at position BW/2 + k, upper triangle by
// position (min, max), leading dimension BW + 1, two buffers by step parity.
// Every lane then reads the same addresses in every step, free of bank
// conflicts; only the writes follow the strategy (positions in the next step
// come from the table, exchanged when the rotation swaps its columns).  The
// diagonal is kept apart (wave 0 only).
template <int BW>
struct JacCfg {
    static constexpr int kThreads = BW * 16;
    static constexpr int kPairs = BW / 2;
    static constexpr int kSteps = BW - 1;
    static constexpr int kLD = BW + 1;
    static constexpr int kBlocks = BW / 32;       // 2 x 2 blocks per lane of an H wave
    static constexpr int kVRows = BW / 32;        // pairs of rows per lane of a V wave
    // roles by wave.  Waves go to the four SIMDs round robin; wave 0's SIMD
    // gets little other work.
    static constexpr int kHFirst = 1, kHCount = BW == 64 ? 4 : 2, kVCount = BW / 8;
    __device__ static constexpr int v_wave(int wave) {  // index among the V waves, or -1
        if (BW == 64) {
            constexpr int at[16] = {-1, -1, -1, -1, -1, 0, 1, 2, -1, 3, 4, 5, -1, 6, 7, -1};
            return at[wave];
        }
        constexpr int at[8] = {-1, -1, -1, 0, -1, 1, 2, 3};
        return at[wave % 8];
    }
};

// The Gram matrix of a pivot pair of 32 columns from G itself, by all eight
// waves: entry (i, j), i <= j, of thread-indexed sums s[].  part: 3072 doubles
// of LDS; ends with a barrier, after which they are free.
template <int EPT>
__device__ __forceinline__ void pair_gram32(const StepArgs &a, int2 pq, double *part,
                                            double (&s)[EPT]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, grp = lane >> 4;
    const int64_t cp = (int64_t)pq.x * a.w + i16, cq = (int64_t)pq.y * a.w + i16;
    d4 g[3] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
    for (int64_t r = 16 * wave + 4 * grp; r - 4 * grp < a.m; r += 128) {
        double x[4], y[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            x[v] = (r + v < a.m && cp < a.n) ? a.G[r + v + cp * a.ldg] : 0.0;
            y[v] = (r + v < a.m && cq < a.n) ? a.G[r + v + cq * a.ldg] : 0.0;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            g[0] = mfma16(x[v], x[v], g[0]);
            g[1] = mfma16(x[v], y[v], g[1]);
            g[2] = mfma16(y[v], y[v], g[2]);
        }
    }
    // waves 4 to 7 add to 0 to 3, whose four sums are added entry by entry
    double *mine = part + (wave & 3) * 768 + lane;
    if (wave >= 4)
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[(4 * t + v) * 64] = g[t][v];
    __syncthreads();
    if (wave < 4)
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) mine[(4 * t + v) * 64] += g[t][v];
    __syncthreads();
    const int j = threadIdx.x % 32;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int i = threadIdx.x / 32 + u * (32 / EPT);
        s[u] = 0.0;
        if (i <= j) {
            const int t = i / 16 + j / 16, v = (i & 15) >> 2, l = (i & 3) * 16 + (j & 15);
            const double *e = part + (4 * t + v) * 64 + l;
            s[u] = (e[0] + e[768]) + (e[2 * 768] + e[3 * 768]);
        }
    }
    __syncthreads();
}

// SOLVE: one workgroup does the whole solve of a single pivot pair (n <= 32,
// w = 16), G and V in global memory (cache): per sweep the Gram matrix, this
// kernel's inner sweeps and the updates of G and V, then the singular values,
// U and the order.  Bound by the chain of the inner sweep (16 us of about 20
// per sweep); four launches, a copy and a wait per sweep take 58 us.
template <int BW, bool HYP, bool SOLVE = false>
__global__ __launch_bounds__(JacCfg<BW>::kThreads) void jacobi_kernel(StepArgs a) {
    using Cfg = JacCfg<BW>;
    constexpr int NT = Cfg::kThreads, NWAVES = NT / 64;
    constexpr int NP = Cfg::kPairs, NS = Cfg::kSteps, LD = Cfg::kLD;
    constexpr int EPT = BW * BW / NT;   // Gram entries summed per thread
    constexpr int HB = BW * LD * 8;     // bytes of one buffer of H
    // H, columns of V' on their way (xch, by slot), position_tables' entry of
    // every step and pair and where wave 0 finds the pair's entry of H (tbl), and
    // of them what the V waves take (vctl); or the four V' of two p-steps' V
    // updates at once
    constexpr int kH = 2 * BW * LD, kXch = 2 * NP * BW, kTbl = NS * NP;
    constexpr int kArena = kH + kXch + 2 * kTbl + (kTbl + 1) / 2;
    __shared__ __align__(16) double arena[BW == 64 && kArena < 4 * BW * BW ? 4 * BW * BW : kArena];
    double(*const H)[BW * LD] = reinterpret_cast<double(*)[BW * LD]>(arena);
    double(*const xch)[NP * BW] = reinterpret_cast<double(*)[NP * BW]>(arena + kH);
    uint4 *const tbl = reinterpret_cast<uint4 *>(arena + kH + kXch);
    unsigned *const vctl = reinterpret_cast<unsigned *>(arena + kH + kXch + 2 * kTbl);
    __shared__ double diag[BW];              // h_cc by position
    __shared__ double2 prm[2][NP];           // published rotations: tan, cos (swapped: -cos)
    __shared__ double mtn[2][HYP ? NP : 1];  // -t tan (hyperbolic pairs: + tan)
    __shared__ unsigned dst[2][NP];          // next positions (times 8) of new p | q << 16
    __shared__ int flags;                    // 1: not orthogonal, 2: a NaN or infinity in H
    __shared__ int rots;                     // rotations of the inner sweep
    __shared__ int total[2];                 // SOLVE: rotations, proper ones of the sweep

    if (!SOLVE && blockIdx.x >= a.npairs) {
        // V <- V V'_pq of an earlier p-step, as in inner_kernel
        const int idx = blockIdx.x - a.npairs;
        const int vpair = idx / a.prev_chunks, chunk = idx % a.prev_chunks;
        if constexpr (BW == 64) {
            if (a.vquads) {
                const int64_t q0 = a.prev_row0 + (int64_t)chunk * a.prev_rows;
                update_quad_rows<NWAVES>(a.V, a.ldv, q0,
                                         min(a.prev_row1, q0 + (int64_t)a.prev_rows),
                                         a.vquads + 8 * vpair, a, arena, &flags);
                return;
            }
        }
        __builtin_amdgcn_s_sleep(127);
        __builtin_amdgcn_s_sleep(127);
        if (a.prev_pair_rot[vpair] == 0) return;
        const int64_t r0 = (int64_t)chunk * a.prev_rows;
        const int64_t r1 = min(a.n, r0 + (int64_t)a.prev_rows);
        update_rows<BW, NWAVES, 1, true>(a.V, a.ldv, r0, r1, a.prev_pairs[vpair], a.w, a.n,
                                a.prev_vprime + (size_t)vpair * BW * BW, arena);
        return;
    }
    const int pair = blockIdx.x;
    const int2 pq = a.pairs[pair];
    const int tid = threadIdx.x;
    if ((int64_t)pq.x * a.w >= a.n) {
        if (tid == 0) a.pair_rot[pair] = 0;
        return;
    }
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- the table and the first partial sums: all loads in flight together
    static_assert(NS * NP <= 2 * NT, "two table entries per thread");
    const unsigned char *gt = a.inner_tbl + 2 * NS * NP;  // after the plain pairs
    const int te = min(2 * tid, NS * NP - 2);
    const uint4 tv = *reinterpret_cast<const uint4 *>(gt + 8 * te);
    const int ej = tid % BW, ei = tid / BW;  // entries (ei + u NT / BW, ej)
    const unsigned char *pos0 = gt + 8 * NS * NP;
    const int pj = pos0[ej];
    int pi[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) pi[u] = pos0[ei + u * (NT / BW)];
    unsigned long long sum[C_COUNT] = {};  // SOLVE: the counters, in wave 0
    if constexpr (SOLVE) {
        if (a.solve_check) {
            // entries so large or columns so small that the norms could leave
            // the range of the unscaled method: the host decides
            bool odd = false;
            for (int64_t c = wave; c < a.n; c += NWAVES) {
                double mx = 0.0;
                for (int64_t r = lane; r < a.m; r += 64) {
                    const double x = fabs(a.G[r + c * a.ldg]);
                    odd = odd || !(x <= 0x1p400);
                    mx = x > mx ? x : mx;
                }
                odd = odd || (__builtin_amdgcn_ballot_w64(mx > 0.0) != 0 &&
                              __builtin_amdgcn_ballot_w64(mx >= 0x1p-400) == 0);
            }
            if (__syncthreads_or(odd)) {
                if (tid == 0) a.counters[C_SOLVE] = kSolveLeft;
                return;
            }
        }
        if (a.V)
            for (int64_t e = tid; e < a.n * a.n; e += NT)
                a.V[e % a.n + e / a.n * a.ldv] = e % a.n == e / a.n ? 1.0 : 0.0;
    }
    bool table_due = true;
    for (int block_sweep = 0; block_sweep < (SOLVE ? a.solve_sweeps : 1); ++block_sweep) {
    const double *hp = a.hpart + (size_t)pair * a.splits * BW * BW;
    double s[EPT];
    if constexpr (SOLVE) {
        pair_gram32<EPT>(a, pq, arena, s);
    } else {
#pragma unroll
    for (int u = 0; u < EPT; ++u) s[u] = 0.0;
    for (int s0 = 0; s0 < a.splits; s0 += 8) {
        // a batch of 8 splits' loads in flight together, summed in split order
        double hv[8][EPT];
#pragma unroll
        for (int sp = 0; sp < 8; ++sp)
#pragma unroll
            for (int u = 0; u < EPT; ++u)
                hv[sp][u] = (s0 + sp < a.splits && ei + u * (NT / BW) <= ej)
                                ? hp[(size_t)(s0 + sp) * BW * BW + tid + u * NT] : 0.0;
#pragma unroll
        for (int sp = 0; sp < 8; ++sp)
#pragma unroll
            for (int u = 0; u < EPT; ++u)
                if (s0 + sp < a.splits) s[u] += hv[sp][u];
    }
    }
    if (table_due && 2 * tid < NS * NP) {
        auto put = [&](int e, unsigned lo, unsigned hi) {
            // where the sent column goes (bytes in xch); bit 31: the kept
            // column is y; bit 30: it is kept again
            vctl[e] = (hi >> 24) * (BW * 8) | (hi & 0x20000u) << 14 | (hi & 0x40000u) << 12;
            // Before the step, the two columns were rotated in pairs I and J of
            // the step before.  Offsets in H of that block's entries (0, 0),
            // (0, 1) and (1, 0); (1, 1) is (0, 0) moved by NP both ways.  I, J,
            // and in bits 31 and 30 whether x (y) was the second of its pair.
            const unsigned I = (lo & 0xff) % NP, J = ((lo >> 8) & 0xff) % NP;
            tbl[e] = make_uint4(
                lo, hi, (min(I, J) * LD + max(I, J)) * 8 | (I * LD + J + NP) * 8 << 16,
                (J * LD + I + NP) * 8 | I << 16 | J << 21 |
                    ((lo & 0xff) >= NP ? 0x80000000u : 0) | (((lo >> 8) & 0xff) >= NP ? 0x40000000u : 0));
        };
        put(2 * tid, tv.x, tv.y);
        put(2 * tid + 1, tv.z, tv.w);
    }
    table_due = false;
    if (tid == 0) flags = 0;

    // ---- H_pq; padding columns become unit vectors orthogonal to everything
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
        const int i = ei + u * (NT / BW);
        if (pair_col(i, a.w, pq) >= a.n || pair_col(ej, a.w, pq) >= a.n)
            s[u] = (i == ej) ? 1.0 : 0.0;
        if (i < ej) H[0][min(pi[u], pj) * LD + max(pi[u], pj)] = s[u];
        if (i == ej) diag[pj] = s[u];
    }
    __syncthreads();

    // ---- nothing to do when every pair (i, j) of the block pair already
    // passes the relative orthogonality test: the pair is left alone.
    const double tol = kEps * sqrt((double)BW);  // c(eps) = eps sqrt(nhat), nhat = 2w
    const double tol2 = kEps * kEps * BW;        // tol^2, exact
    {
        bool need = false, bad = false, wide = false;
        const double hjj = diag[pj];
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const double hii = diag[pi[u]], hij = s[u];
            const bool up = ei + u * (NT / BW) < ej;
            bad = bad || !(fabs(hij) <= 0x1.fffffffffffffp+1023);
            need = need || (up && !(hij * hij <= tol2 * hii * hjj));
            wide = wide || (up && !in_trig_range_bits(hii, hjj));
        }
        if (__builtin_amdgcn_ballot_w64(wide)) {  // the squares are not to be trusted
            need = false;
#pragma unroll
            for (int u = 0; u < EPT; ++u) {
                const double hii = diag[pi[u]], hij = s[u];
                need = need || (ei + u * (NT / BW) < ej && hij != 0.0 &&
                                !(fabs(hij) <= tol * sqrt(hii) * sqrt(hjj)));
            }
        }
        const bool any_need = __builtin_amdgcn_ballot_w64(need) != 0;
        const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0;
        if (lane == 0 && any_need) atomicOr(&flags, 1);
        if (lane == 0 && any_bad) atomicOr(&flags, 2);
    }
    __syncthreads();
    if (flags != 1) {  // nothing to do, or a NaN or infinity in H
        if constexpr (SOLVE) {
            const bool nonfinite = flags == 3;
            sum[C_NONFINITE] += nonfinite;
            sum[C_SOLVE] += 1 + (nonfinite ? 0 : kSolveConverged);
            break;
        }
        if (tid == 0) {
            a.pair_rot[pair] = 0;
            if (flags == 3) atomicAdd(&a.counters[C_NONFINITE], 1ull);
        }
        return;
    }

    // ---- inner Jacobi (Section 4.3)
    const bool on_rot = wave == 0;
    const bool on_h = wave >= Cfg::kHFirst && wave < Cfg::kHFirst + Cfg::kHCount;
    const int vw = __builtin_amdgcn_readfirstlane(Cfg::v_wave(wave));
    // waves without a role end here: barriers wait for the others only
    if (!SOLVE && !on_rot && !on_h && vw < 0) return;
    constexpr int LIVE = 64 * (1 + Cfg::kHCount + Cfg::kVCount);
    const int ltid = lane + 64 * (on_rot ? 0 : on_h ? wave : 1 + Cfg::kHCount + vw);
    char *const hb = reinterpret_cast<char *>(&H[0][0]);
    auto at = [](unsigned x8, unsigned y8) {  // byte offset of (x, y), positions times 8
        return min(x8, y8) * LD + max(x8, y8);
    };

    // H waves: the lane's 2 x 2 blocks (I, J).  Group g of NP lanes takes the
    // NP - 1 - g blocks of row g, then the g + 1 of row NP - 2 - g.
    // (Of the last group's lanes half repeat the other half's blocks: the same
    // values to the same places.)
    int bI[Cfg::kBlocks], bJ[Cfg::kBlocks];
#pragma unroll
    for (int b = 0; b < Cfg::kBlocks; ++b) {
        const int ht = (tid + 64 * (Cfg::kHCount * (b + 1) - Cfg::kHFirst)) % (NP * NP / 2);
        const int g = ht / NP, l = ht % NP;
        const bool first = l < NP - 1 - g;
        bI[b] = first ? g : NP - 2 - g;
        bJ[b] = first ? g + 1 + l : l;
    }
    // wave 0: pair k; columns from cmax on are padding (always the last ones)
    const int k = lane % NP;
    const int64_t nq = a.n - (int64_t)pq.y * a.w;
    const int cmax = (int)(nq > 0 ? a.w + min((int64_t)a.w, nq)
                                  : min((int64_t)a.w, a.n - (int64_t)pq.x * a.w));
    constexpr unsigned long long lanes = (1ull << NP) - 1;
    int rot_total = 0, proper_total = 0, clamp_total = 0, sweeps = 0, rot_sweep = 0;
    double off = 0.0;           // h_pq after the pair's rotation,
    unsigned off_at = 0;        // and where it goes
    uint4 tn = tbl[k];          // the table entry of the coming step
    // V waves: slots 4 vw .. 4 vw + 3, 16 lanes per slot, the rows 2 l, 2 l + 1 (and
    // 32 further) in lane l.  vk: the column of V' kept from the step before; vr:
    // the other one.
    constexpr int VR = Cfg::kVRows;
    const int vs = 4 * (vw < 0 ? 0 : vw) + lane / 16, vrow = 2 * (lane % 16);
    double2 vk[VR], vr[VR];
    unsigned ctl = 0;

    // decide and compute the rotation of pair k in the step of table entry t
    // (h_pp, h_qq, h_pq given), publish it and the new diagonal
    auto rotate_pair = [&](uint4 t, int slot, double hpp, double hqq,
                           double hpq) __attribute__((always_inline)) {
        const int cp = t.y & 0xff, cq = (t.y >> 8) & 0xff;
        bool hyp = false;
        if (HYP) hyp = (pair_col(cp, a.w, pq) < a.n_plus) != (pair_col(cq, a.w, pq) < a.n_plus);
        // subphase 5: keep j sigma^2 non-increasing for trigonometric pairs.
        // |tan| <= 1 leaves the larger diagonal entry the larger one, so the
        // entries before the rotation decide.
        // flip: p is the later column of the two.
        unsigned flip = (t.y & 0x10000u) << 15;
        if (HYP && pair_col(min(cp, cq), a.w, pq) >= a.n_plus) flip ^= 0x80000000u;
        const double up = __builtin_bit_cast(
            double, __builtin_bit_cast(unsigned long long, hqq - hpp) ^ ((unsigned long long)flip << 32));
        const bool swap = (up > 0.0) & (max(cp, cq) < cmax) & !(HYP && hyp);
        const unsigned dp8 = ((t.x >> 16) & 0xff) * 8, dq8 = (t.x >> 24) * 8;
        const unsigned np8 = swap ? dq8 : dp8, nq8 = swap ? dp8 : dq8;

        bool rotate = !(hpq * hpq <= tol2 * hpp * hqq);
        double tn, cs;
        bool clamped;
        rotation_h(hpp, hqq, hpq, hyp, tn, cs, clamped);
        if (!in_trig_range_bits(hpp, hqq)) {
            // outside the range of the squares: IEEE operations.  A diagonal
            // entry that is not positive (H semidefinite to rounding) lands
            // here and rotates unless h_pq is zero.
            rotate = hpq != 0.0 && !(fabs(hpq) <= tol * sqrt(hpp) * sqrt(hqq));
            rotation(hpp, hqq, hpq, hyp ? -1 : 1, tn, cs, clamped);
        }
        tn = rotate ? tn : 0.0;
        cs = rotate ? cs : 1.0;
        const double mt = (HYP && hyp) ? tn : -tn;
        double npp = fma(mt, hpq, hpp), nqq = fma(tn, hpq, hqq);
        off = rotate ? 0.0 : hpq;
        if (HYP && rotate && clamped) {  // not the angle that zeroes h_pq
            npp = cs * cs * fma(tn, fma(tn, hqq, 2.0 * hpq), hpp);
            nqq = cs * cs * fma(tn, fma(tn, hpp, 2.0 * hpq), hqq);
            off = cs * cs * fma(tn, hpp + hqq, fma(tn * tn, hpq, hpq));
        }
        rot_sweep += __builtin_popcountll(__builtin_amdgcn_ballot_w64(rotate) & lanes);
        proper_total += __builtin_popcountll(__builtin_amdgcn_ballot_w64(rotate && cs != 1.0) & lanes);
        if (HYP)
            clamp_total += __builtin_popcountll(__builtin_amdgcn_ballot_w64(rotate && clamped) & lanes);
        // the lanes past NP repeat pairs 0 .. NP - 1: the same values to the
        // same places
        prm[slot][k] = make_double2(tn, swap ? -cs : cs);
        if (HYP) mtn[slot][k] = mt;
        dst[slot][k] = np8 | nq8 << 16;
        *reinterpret_cast<double *>(reinterpret_cast<char *>(diag) + np8) = npp;
        *reinterpret_cast<double *>(reinterpret_cast<char *>(diag) + nq8) = nqq;
        off_at = at(dp8, dq8);
    };

    // one step; PAR: its parity
    auto phase = [&](auto par, int st) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        char *const hc = hb + PAR * HB, *const hn = hb + (1 - PAR) * HB;
        auto ld = [&](unsigned o) { return *reinterpret_cast<const double *>(hc + o); };
        auto put = [&](unsigned o, double v) { *reinterpret_cast<double *>(hn + o) = v; };
        if (on_rot) {
            if (st + 1 < NS) {
                // the new pair's entry is that of two rotated columns of the
                // pairs I and J: c_I c_J u^T X w with X the block before the
                // rotations and u, w = (1, -tan) for a pair's first column,
                // (tan, 1) for its second (the other one if it was swapped)
                const uint4 t = tn;
                const unsigned I = (t.w >> 16) & 31, J = (t.w >> 21) & 31;
                const unsigned s00 = t.z & 0xffff;
                const double2 ra = prm[PAR][I], rb = prm[PAR][J];
                const double x00 = ld(s00), x01 = ld(t.z >> 16), x10 = ld(t.w & 0xffff),
                             x11 = ld(s00 + (NP * LD + NP) * 8);
                const double hpp = diag[k], hqq = diag[k + NP];
                const double ma = HYP ? mtn[PAR][HYP ? I : 0] : -ra.x;
                const double mb = HYP ? mtn[PAR][HYP ? J : 0] : -rb.x;
                put(off_at, off);
                tn = tbl[min(st + 2, NS - 1) * NP + k];
                auto high = [](double v) { return (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32); };
                const bool fa = (int)(high(ra.y) ^ t.w) < 0, fb = (int)(high(rb.y) ^ t.w << 1) < 0;
                const double u0 = fa ? ra.x : 1.0, u1 = fa ? 1.0 : ma;
                const double w0 = fb ? rb.x : 1.0, w1 = fb ? 1.0 : mb;
                const double x0 = fma(w1, x01, w0 * x00), x1 = fma(w1, x11, w0 * x10);
                rotate_pair(t, 1 - PAR, hpp, hqq, fabs(ra.y * rb.y) * fma(u1, x1, u0 * x0));
            } else {
                put(off_at, off);
            }
        } else if (on_h) {
            double x[Cfg::kBlocks][4];
            double2 ri[Cfg::kBlocks], rj[Cfg::kBlocks];
            double mi[Cfg::kBlocks], mj[Cfg::kBlocks];
            unsigned di[Cfg::kBlocks], dj[Cfg::kBlocks];
#pragma unroll
            for (int b = 0; b < Cfg::kBlocks; ++b) {
                const int I = bI[b], J = bJ[b];
                ri[b] = prm[PAR][I];
                rj[b] = prm[PAR][J];
                mi[b] = HYP ? mtn[PAR][I] : -ri[b].x;
                mj[b] = HYP ? mtn[PAR][J] : -rj[b].x;
                di[b] = dst[PAR][I];
                dj[b] = dst[PAR][J];
                x[b][0] = ld((I * LD + J) * 8);
                x[b][1] = ld((I * LD + J + NP) * 8);
                x[b][2] = ld((J * LD + I + NP) * 8);
                x[b][3] = ld(((I + NP) * LD + J + NP) * 8);
            }
#pragma unroll
            for (int b = 0; b < Cfg::kBlocks; ++b) {
                const double cc = fabs(ri[b].y * rj[b].y);
                const double x0 = fma(mj[b], x[b][1], x[b][0]), y0 = fma(rj[b].x, x[b][0], x[b][1]);
                const double x1 = fma(mj[b], x[b][3], x[b][2]), y1 = fma(rj[b].x, x[b][2], x[b][3]);
                const unsigned A0 = di[b] & 0xffff, A1 = di[b] >> 16;
                const unsigned B0 = dj[b] & 0xffff, B1 = dj[b] >> 16;
                put(at(A0, B0), cc * fma(mi[b], x1, x0));
                put(at(A1, B0), cc * fma(ri[b].x, x0, x1));
                put(at(A0, B1), cc * fma(mi[b], y1, y0));
                put(at(A1, B1), cc * fma(ri[b].x, y0, y1));
            }
        } else if (vw >= 0) {
            if (st > 0)
#pragma unroll
                for (int u = 0; u < VR; ++u)
                    vr[u] = *reinterpret_cast<const double2 *>(&xch[1 - PAR][vs * BW + vrow + 32 * u]);
            const double2 r = prm[PAR][vs];
            const double m = HYP ? mtn[PAR][HYP ? vs : 0] : 0.0;
            // tan as seen from the kept column
            const unsigned long long mask = (unsigned long long)(ctl & 0x80000000u) << 32;
            double tk = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, r.x) ^ mask);
            double mk = -tk;
            if (HYP) {
                tk = mask ? m : r.x;
                mk = mask ? r.x : m;
            }
            const double c = fabs(r.y);
            // swapped columns are each other's
            const bool same = ((ctl & 0x40000000u) != 0) != (r.y < 0.0);
#pragma unroll
            for (int u = 0; u < VR; ++u) {
                const double2 k1 = make_double2(c * fma(mk, vr[u].x, vk[u].x), c * fma(mk, vr[u].y, vk[u].y));
                const double2 r1 = make_double2(c * fma(tk, vk[u].x, vr[u].x), c * fma(tk, vk[u].y, vr[u].y));
                vk[u] = make_double2(same ? k1.x : r1.x, same ? k1.y : r1.y);
                vr[u] = make_double2(same ? r1.x : k1.x, same ? r1.y : k1.y);
            }
            if (st + 1 < NS) {
#pragma unroll
                for (int u = 0; u < VR; ++u)
                    *reinterpret_cast<double2 *>(reinterpret_cast<char *>(&xch[PAR][vrow + 32 * u]) +
                                                 (ctl & 0xffff)) = vr[u];
                ctl = vctl[(st + 1) * NP + vs];
            }
        }
        __syncthreads();
    };

    // the kept and the other column of a table entry
    auto kept_col = [&](int e, int &ck, int &cr) {
        const unsigned t = tbl[e].y;
        const bool ky = (t & 0x20000u) != 0;
        ck = (ky ? t >> 8 : t) & 0xff;
        cr = (ky ? t : t >> 8) & 0xff;
    };
    // the V waves' columns after the last step, to a column-major BW x BW matrix
    auto put_v = [&](double *out) __attribute__((always_inline)) {
        int ck, cr;
        kept_col((NS - 1) * NP + vs, ck, cr);
#pragma unroll
        for (int u = 0; u < VR; ++u) {
            *reinterpret_cast<double2 *>(out + ck * BW + vrow + 32 * u) = vk[u];
            *reinterpret_cast<double2 *>(out + cr * BW + vrow + 32 * u) = vr[u];
        }
    };

    if (on_rot) __builtin_amdgcn_s_setprio(3);
    if (vw >= 0) {  // V' = I
        int ck, cr;
        kept_col(vs, ck, cr);
#pragma unroll
        for (int u = 0; u < VR; ++u) {
            const int i = vrow + 32 * u;
            vk[u] = make_double2(i == ck ? 1.0 : 0.0, i + 1 == ck ? 1.0 : 0.0);
            vr[u] = make_double2(i == cr ? 1.0 : 0.0, i + 1 == cr ? 1.0 : 0.0);
        }
    }
    for (int sw = 0; sw < a.max_inner_sweeps; ++sw) {
        rot_sweep = 0;
        if (vw >= 0) ctl = vctl[vs];
        if (on_rot) {
            const uint4 t = tbl[k];
            tn = tbl[NP + k];
            rotate_pair(t, 0, diag[k], diag[k + NP], H[0][k * LD + k + NP]);
        }
        __syncthreads();
        for (int st = 0; st + 1 < NS; st += 2) {
            phase(std::integral_constant<int, 0>{}, st);
            phase(std::integral_constant<int, 1>{}, st + 1);
        }
        phase(std::integral_constant<int, 0>{}, NS - 1);
        ++sweeps;
        rot_total += rot_sweep;
        if (tid == 0) rots = rot_sweep;
        __syncthreads();
        if (rots == 0) break;  // no rotation in the inner sweep
        if (sw + 1 < a.max_inner_sweeps) {
            // the number of steps is odd: H ended in the other buffer.  V' goes
            // back to the slots of step 0.
            for (int e = ltid; e < BW * LD; e += LIVE) H[0][e] = H[1][e];
            double *const all = &xch[0][0];  // both halves: V', column-major
            if (vw >= 0) put_v(all);
            __syncthreads();
            if (vw >= 0) {
                int ck, cr;
                kept_col(vs, ck, cr);
#pragma unroll
                for (int u = 0; u < VR; ++u) {
                    vk[u] = *reinterpret_cast<const double2 *>(all + ck * BW + vrow + 32 * u);
                    vr[u] = *reinterpret_cast<const double2 *>(all + cr * BW + vrow + 32 * u);
                }
            }
            __syncthreads();
        }
    }

    if constexpr (SOLVE) {
        double *const vp = &xch[0][0];  // both halves: V', column-major
        if (vw >= 0) put_v(vp);
        if (on_rot) {
            const int brk = __builtin_popcountll(__builtin_amdgcn_ballot_w64(!(diag[k] > 0.0)) & lanes) +
                            __builtin_popcountll(__builtin_amdgcn_ballot_w64(!(diag[k + NP] > 0.0)) & lanes);
            sum[C_ROT] += rot_total;
            sum[C_PROPER] += proper_total;
            sum[C_CLAMP] += clamp_total;
            sum[C_INNER_SW] += sweeps;
            sum[C_BREAKDOWN] += brk;
            sum[C_UPDATES] += rot_total != 0;
            if (lane == 0) {
                total[0] = rot_total;
                total[1] = proper_total;
            }
        }
        __syncthreads();
        const bool converged = total[1] == 0;
        if (total[0]) {
            update_rows<BW, NWAVES, 1>(a.G, a.ldg, 0, a.m, pq, a.w, a.n, vp, arena);
            __syncthreads();
            if (a.V) update_rows<BW, NWAVES, 1>(a.V, a.ldv, 0, a.n, pq, a.w, a.n, vp, arena);
            __syncthreads();
        }
        sum[C_SOLVE] += 1 + (converged ? kSolveConverged : 0);
        if (converged) break;
    } else {
    // ---- write V'_pq and the counts
    if (vw >= 0) put_v(a.vprime + (size_t)pair * BW * BW);
    if (on_rot) {
        // diagonal entries that are not positive: H was only semidefinite
        // (the padding columns' are 1)
        const int brk = __builtin_popcountll(__builtin_amdgcn_ballot_w64(!(diag[k] > 0.0)) & lanes) +
                        __builtin_popcountll(__builtin_amdgcn_ballot_w64(!(diag[k + NP] > 0.0)) & lanes);
        if (lane == 0) {
            a.pair_rot[pair] = rot_total;
            atomicAdd(&a.counters[C_ROT], (unsigned long long)rot_total);
            atomicAdd(&a.counters[C_PROPER], (unsigned long long)proper_total);
            if (clamp_total) atomicAdd(&a.counters[C_CLAMP], (unsigned long long)clamp_total);
            atomicAdd(&a.counters[C_INNER_SW], (unsigned long long)sweeps);
            if (brk) atomicAdd(&a.counters[C_BREAKDOWN], (unsigned long long)brk);
            if (rot_total) atomicAdd(&a.counters[C_UPDATES], 1ull);
        }
    }
    }
    }

    if constexpr (SOLVE) {
        // ---- sigma_j = ||g_j||, the output order, U = G / sigma and V in it
        __syncthreads();
        double *const nrm = arena;
        int *const perm = reinterpret_cast<int *>(arena + 32);
        for (int64_t c = wave; c < a.n; c += NWAVES) {
            double q = 0.0;
            for (int64_t r = lane; r < a.m; r += 64) q = fma(a.G[r + c * a.ldg], a.G[r + c * a.ldg], q);
#pragma unroll
            for (int d = 32; d > 0; d /= 2) q += __shfl_xor(q, d, 64);
            if (lane == 0) nrm[c] = sqrt(q);
        }
        __syncthreads();
        if (tid < a.n) {
            int rank = tid;
            if (a.solve_sort) {
                // as rank_kernel: +1 columns by non-increasing sigma, then -1
                // columns by non-decreasing sigma, NaN as -infinity
                const bool pos = tid < a.n_plus;
                const int lo = pos ? 0 : a.n_plus, hi = pos ? a.n_plus : (int)a.n;
                auto key = [&](int i) { return nrm[i] != nrm[i] ? -INFINITY : nrm[i]; };
                const double kj = key(tid);
                rank = lo;
                for (int i = lo; i < hi; ++i) {
                    const double ki = key(i);
                    if ((pos ? ki > kj : ki < kj) || (ki == kj && i < tid)) ++rank;
                }
            }
            perm[rank] = tid;
        }
        __syncthreads();
        if (tid < a.n) a.S[tid] = nrm[perm[tid]];
        auto reorder = [&](double *X, int64_t ldx, int64_t rows, bool scale) {
            for (int64_t r = tid; r < rows; r += NT) {
                double x[BW];
#pragma unroll
                for (int c = 0; c < BW; ++c) x[c] = c < a.n ? X[r + perm[c] * ldx] : 0.0;
#pragma unroll
                for (int c = 0; c < BW; ++c)
                    if (c < a.n) {
                        const double sc = scale ? nrm[perm[c]] : 1.0;
                        X[r + c * ldx] = scale ? (sc > 0.0 ? x[c] / sc : 0.0) : x[c];
                    }
            }
        };
        reorder(a.G, a.ldg, a.m, true);
        if (a.V && a.solve_sort) reorder(a.V, a.ldv, a.n, false);
        if (tid == 0)
            for (int c = 0; c < C_COUNT; ++c) a.counters[c] = sum[c];
    }
}

// ----------------------------------------------------------- inner, 2w = 128
// The third blocking level.  R and V' of a 128-column pivot pair (128 KiB
// each) do not both fit in LDS, so, as Section 2 does one level up, the
// inner problem is itself solved by the block method: the Cholesky factor
// R of H_pq is written to a global scratch (L2-resident) and a block Jacobi
// with 16-column sub-blocks runs on it (sub-block Gram matrices, their
// Cholesky factors, one pointwise sweep each and the sub-updates on FP64
// MFMA, as the batched path's blocked method: blocked_sweeps), accumulating
// V' directly in the pair's slot of the V' buffer.  max_inner_sweeps bounds
// the block sweeps of that inner method (1: block-oriented).  Ordinary SVD,
// unscaled; the sub-level strategy is the reverse row-cyclic one.
// 512 threads (kBlkThreads).  Extra workgroups after the pairs' apply the
// previous p-step's V' to V, as in inner_kernel.
constexpr int kW128Threads = kBlkThreads;

__global__ __launch_bounds__(kW128Threads) void inner128_kernel(StepArgs a) {
    constexpr int BW = 128, LD = BW + 1, NT = kW128Threads, NWAVES = NT / 64;
    constexpr int EPT = BW * BW / NT;  // Gram entries summed per thread
    __shared__ __align__(16) double L[BW * LD];  // H, then R; then the block method's R'' and V''
    __shared__ int sflag[2];           // [0] NaN or infinite pivot, [1] zero pivots
    __shared__ int stats[3];           // rotations, proper rotations, sub-pair updates
    static_assert(kBlkLdsDoubles <= BW * LD, "the block method's LDS fits in L");
    static_assert(BW * BW <= BW * LD, "V' of the V workgroups fits in L");

    if (blockIdx.x >= a.npairs) {
        __builtin_amdgcn_s_sleep(127);
        __builtin_amdgcn_s_sleep(127);
        const int idx = blockIdx.x - a.npairs;
        const int vpair = idx / a.prev_chunks, chunk = idx % a.prev_chunks;
        if (a.prev_pair_rot[vpair] == 0) return;
        const int64_t r0 = (int64_t)chunk * a.prev_rows;
        const int64_t r1 = min(a.n, r0 + (int64_t)a.prev_rows);
        update_rows<BW, NWAVES, 1, true>(a.V, a.ldv, r0, r1, a.prev_pairs[vpair], a.w, a.n,
                                         a.prev_vprime + (size_t)vpair * BW * BW, L);
        return;
    }
    const int pair = blockIdx.x;
    const int2 pq = a.pairs[pair];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if ((int64_t)pq.x * a.w >= a.n) {
        if (tid == 0) a.pair_rot[pair] = 0;
        return;
    }

    // ---- H_pq: the partial Gram matrices summed in split order (upper
    // triangle); padding columns become unit vectors
    {
        const double *hp = a.hpart + (size_t)pair * a.splits * BW * BW;
        double sacc[EPT];
#pragma unroll
        for (int u = 0; u < EPT; ++u) sacc[u] = 0.0;
        for (int sp = 0; sp < a.splits; ++sp)
#pragma unroll
            for (int u = 0; u < EPT; ++u) {
                const int e = tid + u * NT;
                if (e / BW <= e % BW) sacc[u] += hp[(size_t)sp * BW * BW + e];
            }
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const int e = tid + u * NT, i = e / BW, j = e % BW;
            double h = (i <= j) ? sacc[u] : 0.0;
            if (i <= j && (pair_col(i, a.w, pq) >= a.n || pair_col(j, a.w, pq) >= a.n))
                h = (i == j) ? 1.0 : 0.0;
            L[j * LD + i] = h;
        }
    }
    if (tid < 2) sflag[tid] = 0;
    if (tid < 3) stats[tid] = 0;
    __syncthreads();

    // ---- nothing to do when every (i, j) passes the orthogonality test of
    // the sub-level (c(eps) = eps sqrt(32), the smaller of the two levels')
    {
        const double tol = kEps * sqrt((double)kBlkBW);
        bool need = false;
#pragma unroll
        for (int u = 0; u < EPT; ++u) {
            const int e = tid + u * NT, i = e / BW, j = e % BW;
            if (i < j) {
                const double hij = L[j * LD + i], hii = L[i * LD + i], hjj = L[j * LD + j];
                need = need || (hij != 0.0 && !(fabs(hij) <= tol * sqrt(hii) * sqrt(hjj)));
            }
        }
        if (!__syncthreads_or(need ? 1 : 0)) {
            if (tid == 0) a.pair_rot[pair] = 0;
            return;
        }
    }

    // ---- Cholesky H = R^T R (Section 4.1) by block rows of 16: wave 0 factors
    // a block row, lane j holding columns j and j + 64 (readlane broadcasts the
    // pivots and multipliers), then the block row's contribution leaves the
    // trailing part of H on FP64 MFMA, 16 x 16 tiles spread over the waves.
    // Non-positive pivots make their row zero; NaN or infinite ones stop the
    // pair (as in inner_kernel).
#pragma unroll 1
    for (int kb = 0; kb < BW / 16; ++kb) {
        if (wave == 0) {
            double hb[2][16];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                for (int i = 0; i < 16; ++i) hb[hh][i] = L[(lane + 64 * hh) * LD + 16 * kb + i];
            int zero_pivots = 0, nan_met = 0;
            const int ph = kb >= 4 ? 1 : 0;  // half holding the panel's own columns
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int kk = 16 * kb + k;
                const double hkk = lane_value(ph ? hb[1][k] : hb[0][k], kk - 64 * ph);
                const bool bad = !(fabs(hkk) <= 0x1.fffffffffffffp+1023);
                const bool pos = !bad && hkk > 0.0;
                nan_met |= bad ? 1 : 0;
                zero_pivots += (!bad && !pos) ? 1 : 0;
                double rs, d;
                rsqrt_sqrt(pos ? hkk : 1.0, rs, d);
                double rr[2];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int j = lane + 64 * hh;
                    double r = (j == kk) ? d : hb[hh][k] * rs;
                    rr[hh] = (pos && j >= kk) ? r : 0.0;
                    hb[hh][k] = rr[hh];
                }
#pragma unroll
                for (int i = k + 1; i < 16; ++i) {
                    const double ri = lane_value(ph ? rr[1] : rr[0], 16 * kb + i - 64 * ph);
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) hb[hh][i] = fma(-ri, rr[hh], hb[hh][i]);
                }
            }
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int j = lane + 64 * hh;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    L[j * LD + 16 * kb + i] = (j >= 16 * kb + i) ? hb[hh][i] : 0.0;
            }
            if (lane == 0) {
                sflag[0] |= nan_met;
                sflag[1] += zero_pivots;
            }
        }
        __syncthreads();
        if (kb + 1 < BW / 16) {
            // H(i, j) -= sum_k R(16 kb + k, i) R(16 kb + k, j), tiles kb < ti <= tj
            constexpr int TB = BW / 16;
            const int rest = TB - 1 - kb, ntiles = rest * (rest + 1) / 2;
            for (int idx = wave; idx < ntiles; idx += NWAVES) {
                int ti = kb + 1, rem = idx;
                while (rem >= TB - ti) {
                    rem -= TB - ti;
                    ++ti;
                }
                const int tj = ti + rem;
                const int l16 = lane & 15, l4 = lane >> 4;
                d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int k = 16 * kb + 4 * c + l4;
                    acc = mfma16(L[(16 * ti + l16) * LD + k], L[(16 * tj + l16) * LD + k], acc);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * ti + l4 + 4 * v, j = 16 * tj + l16;
                    if (i <= j) L[j * LD + i] -= acc[v];
                }
            }
            __syncthreads();
        }
    }
    if (sflag[0]) {
        if (tid == 0) {
            a.pair_rot[pair] = 0;
            atomicAdd(&a.counters[C_NONFINITE], 1ull);
        }
        return;
    }
    if (tid == 0 && sflag[1]) atomicAdd(&a.counters[C_BREAKDOWN], (unsigned long long)sflag[1]);

    // ---- R to the pair's scratch (upper triangle, zeros below), V' := I in
    // the pair's V' slot, then the block method on R
    double *Rg = a.rscratch + (size_t)pair * BW * BW;
    double *Vg = a.vprime + (size_t)pair * BW * BW;
    for (int e = tid; e < BW * BW; e += NT) {
        const int i = e % BW, j = e / BW;
        Rg[e] = (i <= j) ? L[j * LD + i] : 0.0;
        Vg[e] = (i == j) ? 1.0 : 0.0;
    }
    __syncthreads();
    // the pair's padding columns are its last ones
    const int64_t nq = a.n - (int64_t)pq.y * a.w;
    const int n_real = (int)(nq > 0 ? a.w + min((int64_t)a.w, nq)
                                    : min((int64_t)a.w, a.n - (int64_t)pq.x * a.w));
    const int r = blocked_sweeps(Rg, Vg, BW, BW, n_real, max(1, min(a.max_inner_sweeps, 0xffff)),
                                 a.btbl_order, a.btbl_off, a.btbls, a.bjac, L, stats);
    __syncthreads();
    if (tid == 0) {
        if (r & kBlkNonfinite) {
            a.pair_rot[pair] = 0;
            atomicAdd(&a.counters[C_NONFINITE], 1ull);
        } else {
            const int rot = stats[0];
            a.pair_rot[pair] = rot;
            atomicAdd(&a.counters[C_ROT], (unsigned long long)rot);
            atomicAdd(&a.counters[C_PROPER], (unsigned long long)stats[1]);
            atomicAdd(&a.counters[C_INNER_SW], (unsigned long long)(r & 0xffff));
            if (rot) atomicAdd(&a.counters[C_UPDATES], 1ull);
        }
    }
}

}  // namespace

hipError_t launch_solve(const StepArgs &a, hipStream_t s) {
    const dim3 nt(JacCfg<32>::kThreads);
    if (a.n_plus < a.n)
        hipLaunchKernelGGL((jacobi_kernel<32, true, true>), dim3(1), nt, 0, s, a);
    else
        hipLaunchKernelGGL((jacobi_kernel<32, false, true>), dim3(1), nt, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_inner(int bw, const StepArgs &a, hipStream_t s) {
    if (bw == 128) {
        hipLaunchKernelGGL(inner128_kernel, dim3(a.npairs + a.prev_n * a.prev_chunks),
                           dim3(kW128Threads), 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid(a.npairs + a.prev_n * a.prev_chunks);
    const bool hyp = a.n_plus < a.n;
    if (!a.colexp && !a.qrf) {
        // unscaled, by the Gram matrix: two-sided rotations, 1.7 to 1.8 times
        // as fast as on R
        const dim3 nt(JacCfg<32>::kThreads), nt64(JacCfg<64>::kThreads);
        if (bw == 32) {
            if (hyp)
                hipLaunchKernelGGL((jacobi_kernel<32, true>), grid, nt, 0, s, a);
            else
                hipLaunchKernelGGL((jacobi_kernel<32, false>), grid, nt, 0, s, a);
        } else {
            if (hyp)
                hipLaunchKernelGGL((jacobi_kernel<64, true>), grid, nt64, 0, s, a);
            else
                hipLaunchKernelGGL((jacobi_kernel<64, false>), grid, nt64, 0, s, a);
        }
        return hipGetLastError();
    }
    const dim3 blk(InnerCfg<32>::kThreads), blk64(InnerCfg<64>::kThreads);
    if (a.colexp) {
        if (bw == 32) {
            if (hyp)
                hipLaunchKernelGGL((inner_kernel<32, true, true>), grid, blk, 0, s, a);
            else
                hipLaunchKernelGGL((inner_kernel<32, false, true>), grid, blk, 0, s, a);
        } else {
            if (hyp)
                hipLaunchKernelGGL((inner_kernel<64, true, true>), grid, blk64, 0, s, a);
            else
                hipLaunchKernelGGL((inner_kernel<64, false, true>), grid, blk64, 0, s, a);
        }
    } else {
        if (bw == 32) {
            if (hyp)
                hipLaunchKernelGGL((inner_kernel<32, true, false>), grid, blk, 0, s, a);
            else
                hipLaunchKernelGGL((inner_kernel<32, false, false>), grid, blk, 0, s, a);
        } else {
            if (hyp)
                hipLaunchKernelGGL((inner_kernel<64, true, false>), grid, blk64, 0, s, a);
            else
                hipLaunchKernelGGL((inner_kernel<64, false, false>), grid, blk64, 0, s, a);
        }
    }
    return hipGetLastError();
}

}  // namespace jsvd
