// FP64 MFMA matrix products for the QR preprocessing and the SVD adjoint.
//
// gemm_f64_kernel is the general batched product.  Two shapes of the
// blocked Householder QR (eq. (2.1); a panel of 32 reflectors V with its
// 32 x 32 factor T) get kernels of their own, as the general tiling leaves
// them far below the HBM roofline:
//   * Y = V^T C over all rows (split over row slices): 32 output rows, a
//     contraction over thousands of rows -- laid out as the Gram kernel
//     is, each lane reading consecutive rows of one column of both
//     operands, so that the contraction runs along the rows;
//   * C <- alpha V Y + beta C with 32 reflectors: a rank-32 update of a
//     tall C, computed as (V Y)^T = Y^T V^T so that each lane's results are
//     consecutive rows of one column of C (coalesced reads and writes),
//     the 16 x 32 slice of V of a wave held in registers and the block's
//     slice of Y in LDS across the column tiles.
#include "jsvd_device.h"

namespace jsvd {

namespace {

// two doubles loaded as one 16-byte access (8-byte alignment suffices)
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// C = alpha op(A) op(B) + beta C [+ E diag(d)] for a batch of column-major
// matrices, or (split-K) one product whose K range is cut into slices, slice
// b summed into the b-th C of the batch.
// op(A) is M x K, op(B) is K x N.  Workgroup tile 32 WT x 32 WT (4 WT waves
// of WT x 1 MFMA tiles of 16 x 16: two waves per SIMD at WT = 2 cover each
// other's LDS reads), K steps of 32 through two LDS buffers.  Loads are issued
// two steps ahead, into registers, and stored to the buffer one step later (a
// step is 2048 cycles of MFMA at WT = 2, less than a load's latency).  MFMA lane layout: lane l
// supplies A[l%16][l/16] and B[l/16][l%16], element v of the result is
// D[l/16 + 4v][l%16]; op(B)^T takes the A operand's place, so that the lanes
// of a result are consecutive rows of C.  Bound by the MFMAs and the wait for
// the slowest wave at each step's barrier: 1024^3 takes 57 us (38 TFLOP/s), with
// 16-column steps that each waited for their loads 240 us.
constexpr int kGemmK = 32;
template <int T>
constexpr int kGemmThreads = T == 64 ? 512 : 256;

// A 32 x T slice of an operand, element (k, i), i < T: at src[k + i ld] (ALONG_K)
// or src[i + k ld]; nk and ni of its rows and columns exist.  Thread t holds
// its elements as pairs of neighbours in memory.
template <int T, bool ALONG_K>
__device__ __forceinline__ void gemm_load(const double *src, int64_t ld, int nk, int ni,
                                          double (&x)[2 * (16 * T / kGemmThreads<T>)]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int u = 0; u < 16 * T / kGemmThreads<T>; ++u) {
        const int e = t + kGemmThreads<T> * u;  // pair index
        const int k = ALONG_K ? 2 * (e % 16) : e / (T / 2);
        const int i = ALONG_K ? e / 16 : 2 * (e % (T / 2));
        const double *p = ALONG_K ? src + k + (int64_t)i * ld : src + i + (int64_t)k * ld;
        const bool in = k < nk && i < ni;
        const bool both = in && (ALONG_K ? k + 1 < nk : i + 1 < ni);
        if (both) {
            const d2u v = *reinterpret_cast<const d2u *>(p);
            x[2 * u] = v.x;
            x[2 * u + 1] = v.y;
        } else {
            x[2 * u] = in ? *p : 0.0;
            x[2 * u + 1] = 0.0;
        }
    }
}

template <int T, bool ALONG_K>
__device__ __forceinline__ void gemm_stage(double *s,
                                           const double (&x)[2 * (16 * T / kGemmThreads<T>)]) {
    constexpr int LD = T + 2;
    const int t = threadIdx.x;
#pragma unroll
    for (int u = 0; u < 16 * T / kGemmThreads<T>; ++u) {
        const int e = t + kGemmThreads<T> * u;
        if (ALONG_K) {
            const int k = 2 * (e % 16), i = e / 16;
            s[k * LD + i] = x[2 * u];
            s[(k + 1) * LD + i] = x[2 * u + 1];
        } else {
            const int k = e / (T / 2), i = 2 * (e % (T / 2));
            *reinterpret_cast<double2 *>(s + k * LD + i) = make_double2(x[2 * u], x[2 * u + 1]);
        }
    }
}

template <int WT, bool TA, bool TB>
__global__ __launch_bounds__(kGemmThreads<32 * WT>) void gemm_f64_kernel(GemmArgs g) {
    constexpr int T = 32 * WT, LD = T + 2, KT = kGemmK;
    __shared__ __align__(16) double As[2][KT * LD];  // As[k][i] = op(A)[i0 + i][k0 + k]
    __shared__ __align__(16) double Bs[2][KT * LD];  // Bs[k][j] = op(B)[k0 + k][j0 + j]
    const int b = blockIdx.z;
    // Workgroups go to the 8 XCDs round robin: where the grid of tiles divides
    // into 4 x 2 blocks, each XCD takes one of them, so that its L2 sees a
    // quarter of A and half of B.
    int bx = blockIdx.x, by = blockIdx.y;
    if (gridDim.x % 4 == 0 && gridDim.y % 2 == 0) {
        const int lin = bx + gridDim.x * by, xcd = lin % 8, i = lin / 8, w = gridDim.x / 4;
        bx = (xcd % 4) * w + i % w;
        by = (xcd / 4) * (gridDim.y / 2) + i / w;
    }
    const int i0 = bx * T, j0 = by * T;
    const double *A = g.A + (g.ksplit ? 0 : (size_t)b * g.sa) + (TA ? (size_t)i0 * g.lda : i0);
    const double *B = g.B + (g.ksplit ? 0 : (size_t)b * g.sb) + (TB ? j0 : (size_t)j0 * g.ldb);
    double *C = g.C + (size_t)b * g.sc;
    // K range of this product (split-K: one slice per batch index)
    const int kbeg = g.ksplit ? (int)min((int64_t)g.K, (int64_t)b * g.ksplit) : 0;
    const int kend = g.ksplit ? (int)min((int64_t)g.K, (int64_t)(b + 1) * g.ksplit) : g.K;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wi = (wave & 1) * 16 * WT, wj = (wave >> 1) * 16;
    const int l16 = lane & 15, lg = lane >> 4;
    const int ni = g.M - i0, nj = g.N - j0;
    d4 acc[WT];
#pragma unroll
    for (int x = 0; x < WT; ++x) acc[x] = d4{0.0, 0.0, 0.0, 0.0};

    constexpr int NX = 2 * (16 * T / kGemmThreads<T>);
    auto load = [&](int k0, double (&xa)[NX], double (&xb)[NX]) __attribute__((always_inline)) {
        gemm_load<T, TA>(A + (TA ? k0 : (size_t)k0 * g.lda), g.lda, kend - k0, ni, xa);
        gemm_load<T, !TB>(B + (TB ? (size_t)k0 * g.ldb : k0), g.ldb, kend - k0, nj, xb);
    };
    auto stage = [&](int buf, const double (&xa)[NX], const double (&xb)[NX]) __attribute__((always_inline)) {
        gemm_stage<T, TA>(As[buf], xa);
        gemm_stage<T, !TB>(Bs[buf], xb);
    };
    // one K step: (xa, xb) hold the next step's tiles and go to the other
    // buffer, (ya, yb) receive the one after's
    auto step = [&](int k0, int buf, const double (&xa)[NX], const double (&xb)[NX], double (&ya)[NX],
                    double (&yb)[NX]) __attribute__((always_inline)) {
        if (k0 + 2 * KT < kend) load(k0 + 2 * KT, ya, yb);
#pragma unroll
        for (int kk = 0; kk < KT; kk += 4) {
            double av[WT];
#pragma unroll
            for (int x = 0; x < WT; ++x) av[x] = As[buf][(kk + lg) * LD + wi + 16 * x + l16];
            const double bv = Bs[buf][(kk + lg) * LD + wj + l16];
#pragma unroll
            for (int x = 0; x < WT; ++x) acc[x] = mfma16(bv, av[x], acc[x]);
        }
        if (k0 + KT < kend) stage(buf ^ 1, xa, xb);
        __syncthreads();
    };
    double xa[NX] = {}, xb[NX] = {}, ya[NX] = {}, yb[NX] = {};
    if (kbeg < kend) {
        load(kbeg, xa, xb);
        stage(0, xa, xb);
        if (kbeg + KT < kend) load(kbeg + KT, xa, xb);
    }
    __syncthreads();
    for (int k0 = kbeg; k0 < kend; k0 += 2 * KT) {
        step(k0, 0, xa, xb, ya, yb);
        if (k0 + KT < kend) step(k0 + KT, 1, ya, yb, xa, xb);
    }
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int gi = i0 + wi + 16 * x + l16;
            const int gj = j0 + wj + lg + 4 * v;
            if (gi < g.M && gj < g.N) {
                double r = g.alpha == 1.0 ? acc[x][v] : g.alpha * acc[x][v];
                if (g.beta != 0.0) r = fma(g.beta, C[gi + (size_t)gj * g.ldc], r);
                if (g.E) r += g.E[(size_t)b * g.se + gi + (size_t)gj * g.lde] * g.d[(size_t)b * g.sd + gj];
                C[gi + (size_t)gj * g.ldc] = r;
            }
        }
}

template <int WT>
void gemm_f64(const GemmArgs &g, hipStream_t s) {
    constexpr int T = 32 * WT;
    const dim3 grid((unsigned)((g.M + T - 1) / T), (unsigned)((g.N + T - 1) / T), (unsigned)g.batch);
    const dim3 blk(kGemmThreads<T>);
    if (g.ta && g.tb)
        hipLaunchKernelGGL((gemm_f64_kernel<WT, true, true>), grid, blk, 0, s, g);
    else if (g.ta)
        hipLaunchKernelGGL((gemm_f64_kernel<WT, true, false>), grid, blk, 0, s, g);
    else if (g.tb)
        hipLaunchKernelGGL((gemm_f64_kernel<WT, false, true>), grid, blk, 0, s, g);
    else
        hipLaunchKernelGGL((gemm_f64_kernel<WT, false, false>), grid, blk, 0, s, g);
}

// out_b (M x N, ld M) = A[rows of slice b]^T B[rows of slice b], slices of
// ksplit rows; M <= 16 MT.  Grid (column blocks of 64, slices), 256
// threads: the four waves take 8-row steps of the slice (each lane 2
// consecutive rows of one column of A and of B: the same rows are the
// contraction index of both MFMA operands), and their accumulators are
// summed in a fixed order at the end.
template <int MT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void gemm_tn_rows_kernel(const double *A, int64_t lda,
                                                           const double *B, int64_t ldb, int M,
                                                           int N, int64_t K, int64_t ksplit,
                                                           double *out, int64_t so) {
    constexpr int NTL = 4;  // column tiles of 16 of B per workgroup
    constexpr int S = 2;    // consecutive rows per lane
    __shared__ d4 red[MT * NTL * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, grp = lane >> 4;
    const int b = blockIdx.y;
    const int j0 = blockIdx.x * 64;
    const int64_t r0 = (int64_t)b * ksplit, r1 = min(K, r0 + ksplit);
    const double *ca[MT];
    const double *cb[NTL];
    bool va[MT], vb[NTL];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int c = 16 * t + i16;
        va[t] = c < M;
        ca[t] = A + (va[t] ? c : 0) * lda;
    }
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
        const int c = j0 + 16 * t + i16;
        vb[t] = c < N;
        cb[t] = B + (vb[t] ? c : 0) * ldb;
    }
    d4 acc[MT][NTL];
#pragma unroll
    for (int x = 0; x < MT; ++x)
#pragma unroll
        for (int y = 0; y < NTL; ++y) acc[x][y] = d4{0.0, 0.0, 0.0, 0.0};
    // every column of both operands present: the S = 2 consecutive rows of a
    // lane as one 16-byte load, without selects
    const bool allv = M == 16 * MT && j0 + 64 <= N;
    for (int64_t base = r0 + wave * 4 * S; base < r1; base += 16 * S) {
        const int64_t rb = base + grp * S;
        double xa[MT][S], xb[NTL][S];
        if (allv && rb + S <= r1) {
            static_assert(S == 2, "one 16-byte load per lane and column");
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                const d2u v = *reinterpret_cast<const d2u *>(ca[t] + rb);
                xa[t][0] = v.x;
                xa[t][1] = v.y;
            }
#pragma unroll
            for (int t = 0; t < NTL; ++t) {
                const d2u v = *reinterpret_cast<const d2u *>(cb[t] + rb);
                xb[t][0] = v.x;
                xb[t][1] = v.y;
            }
        } else {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int s = 0; s < S; ++s) xa[t][s] = (va[t] && rb + s < r1) ? ca[t][rb + s] : 0.0;
#pragma unroll
            for (int t = 0; t < NTL; ++t)
#pragma unroll
                for (int s = 0; s < S; ++s) xb[t][s] = (vb[t] && rb + s < r1) ? cb[t][rb + s] : 0.0;
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int x = 0; x < MT; ++x)
#pragma unroll
                for (int y = 0; y < NTL; ++y) acc[x][y] = mfma16(xa[x][s], xb[y][s], acc[x][y]);
    }
    // fixed-order sum over the four waves: ((w0 + w1) + w2) + w3
    for (int wv = 0; wv < 4; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int x = 0; x < MT; ++x)
#pragma unroll
                for (int y = 0; y < NTL; ++y) {
                    d4 &r = red[(x * NTL + y) * 64 + lane];
                    r = wv == 0 ? acc[x][y] : r + acc[x][y];
                }
        }
        __syncthreads();
    }
    double *o = out + (int64_t)b * so;
    for (int e = threadIdx.x; e < MT * NTL * 256; e += 256) {
        const int k = e >> 8, rem = e & 255, v = rem >> 6, l = rem & 63;
        const int x = k / NTL, y = k % NTL;
        const int row = 16 * x + (l >> 4) + 4 * v, col = j0 + 16 * y + (l & 15);
        if (row < M && col < N) o[row + (int64_t)col * M] = red[k * 64 + l][v];
    }
}

// C (rows x N, ld ldc) = alpha A Y + beta C with A rows x K (ld lda), Y K x N
// (ld ldy), K <= 32.  Grid (row blocks of 64, column blocks of 64), 256
// threads: the block's K x 64 slice of Y is staged in LDS once (each lane
// of a tile would otherwise fetch 16 strided columns of Y per MFMA step);
// wave w owns rows [16 w, 16 w + 16) of the block, keeps its 16 x K slice of
// A in registers (lane l: row l % 16, columns l / 16 + 4 k) and walks the
// column tiles of 16: per tile C's 16 x 16 tile is read first (beta != 0),
// then the K / 4 MFMAs of Y^T A^T, and the tile is written back as 16
// consecutive rows per column.
__global__ __launch_bounds__(256) void gemm_rank_kernel(const double *A, int64_t lda,
                                                        const double *Y, int64_t ldy,
                                                        double *C, int64_t ldc, int rows, int N,
                                                        int K, double alpha, double beta) {
    constexpr int KS = 8;       // MFMA steps of 4 along K (K <= 32)
    constexpr int CB = 64;      // columns per workgroup
    constexpr int YLD = 36;     // LDS leading dimension of the Y slice (two lanes per bank pair)
    __shared__ double ys[CB * YLD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i16 = lane & 15, grp = lane >> 4;
    const int jbeg = blockIdx.y * CB, jend = min(N, jbeg + CB);
    for (int e = threadIdx.x; e < CB * 32; e += 256) {
        const int c = e / 32, k = e % 32;
        ys[c * YLD + k] = (jbeg + c < N && k < K) ? Y[k + (int64_t)(jbeg + c) * ldy] : 0.0;
    }
    const int64_t row = (int64_t)blockIdx.x * 64 + wave * 16 + i16;
    const bool rv = row < rows;
    double av[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        const int kk = 4 * k + grp;
        av[k] = (rv && kk < K) ? A[row + (int64_t)kk * lda] : 0.0;
    }
    __syncthreads();
    for (int j0 = jbeg; j0 < jend; j0 += 16) {
        double cv[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int col = j0 + grp + 4 * v;
            cv[v] = (beta != 0.0 && rv && col < N) ? C[row + (int64_t)col * ldc] : 0.0;
        }
        const double *yc = ys + (j0 - jbeg + i16) * YLD;  // the column of Y this lane supplies
        d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < KS; ++k) acc = mfma16(yc[4 * k + grp], av[k], acc);
        // acc[v] = (Y^T A^T)(j0 + grp + 4 v, row) = (A Y)(row, j0 + grp + 4 v)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int col = j0 + grp + 4 * v;
            if (rv && col < N) {
                double r = alpha == 1.0 ? acc[v] : alpha * acc[v];
                if (beta != 0.0) r = fma(beta, cv[v], r);
                C[row + (int64_t)col * ldc] = r;
            }
        }
    }
}

}  // namespace

hipError_t launch_gemm(const GemmArgs &g, hipStream_t s) {
    if (g.ta && !g.tb && g.ksplit > 0 && g.M <= 32 && g.alpha == 1.0 && g.beta == 0.0 && !g.E) {
        dim3 grid((unsigned)((g.N + 63) / 64), (unsigned)g.batch);
        if (g.M <= 16)
            hipLaunchKernelGGL(gemm_tn_rows_kernel<1>, grid, dim3(256), 0, s, g.A, g.lda, g.B,
                               g.ldb, g.M, g.N, (int64_t)g.K, g.ksplit, g.C, g.sc);
        else
            hipLaunchKernelGGL(gemm_tn_rows_kernel<2>, grid, dim3(256), 0, s, g.A, g.lda, g.B,
                               g.ldb, g.M, g.N, (int64_t)g.K, g.ksplit, g.C, g.sc);
        return hipGetLastError();
    }
    if (!g.ta && !g.tb && g.batch == 1 && !g.ksplit && g.K <= 32 && !g.E) {
        dim3 grid((unsigned)((g.M + 63) / 64), (unsigned)((g.N + 63) / 64));
        hipLaunchKernelGGL(gemm_rank_kernel, grid, dim3(256), 0, s, g.A, g.lda, g.B, g.ldb, g.C,
                           g.ldc, g.M, g.N, g.K, g.alpha, g.beta);
        return hipGetLastError();
    }
    // 64 x 64 tiles where they give a workgroup per CU (256), 32 x 32 below
    // (more of the chip, each operand read twice as often).  The adjoint's five
    // products at 1024 x 1024 (256 tiles of 64): 0.27 ms with 64 x 64, 0.31 ms
    // with 32 x 32; at 700 x 500 (88 tiles) 0.11 ms with 32 x 32.  Products of
    // at most 32 rows or columns would fill half of a 64 x 64 tile: the adjoint of
    // 2000 problems of 20 x 12 takes 53 us with 32 x 32, 95 with 64 x 64, of 400 of
    // 64 x 32 46 and 54.
    const int64_t tiles = (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.batch;
    if (tiles >= 256 && g.M > 32 && g.N > 32)
        gemm_f64<2>(g, s);
    else
        gemm_f64<1>(g, s);
    return hipGetLastError();
}

}  // namespace jsvd
