// fp64 dense linear algebra for the reconstruction solves of Sec. 4 (the
// closed-form U and V updates of Algorithm "MPIFA", Part 1).  These run once
// per layer on n x n and r x r systems; the hot part of the reconstruction is
// the accumulation of the calibration sums, which runs on the MFMA GEMM.
//
//   gemm64        C = alpha op(A) op(B) + beta C with arbitrary element strides
//                 (transposes are strides, no copies) on fp64 MFMA tiles;
//                 optional lower-triangle tiles only, for symmetric results;
//                 optionally a batch of equal products.
//   Cholesky      A = L L^T, right-looking in blocks of 256 columns, each
//                 factored 64 columns at a time: diagonal block in one
//                 workgroup's registers (which also gives its inverse), panel
//                 as a product with that inverse, the update of the block's
//                 own columns, and one 256-deep update of the rest.
//   spd solve     L L^T X = B for many right-hand sides: blocked forward and
//                 backward substitution; each 256-wide diagonal block is
//                 applied as its explicit inverse (put together from the
//                 64-wide ones), so every step is a gemm64 at least 256 deep.
// Updates 64 columns deep moved the trailing matrix for every 64 columns
// and took half of the solve's time.
#pragma once

#include "common.hpp"

namespace pifa {

constexpr int kG64 = 64;    // columns factored at a time
constexpr int kB64 = 256;   // block size of the trailing updates and solves

typedef double f64x4 __attribute__((ext_vector_type(4)));

// C[i*sc0 + j*sc1] = alpha * sum_k A[i*sa0 + k*sa1] * B[k*sb0 + j*sb1] + beta * C[...]
// for i < Mr, j < Nc, on v_mfma_f64_16x16x4_f64.  LOWER: only tiles whose
// first row >= first column (tiles on the diagonal are computed whole).
// beta == 0 ignores C's old value.
// Tile BT x BT, K step BK, 16 waves in a 4 x 4 grid (1024 threads), each a
// (BT/4) x (BT/4) block of 16 x 16 MFMA outputs.  Both operands are staged
// k-major in LDS ([k][i] and [k][j]), so any stride pattern loads with the
// unit-stride axis across consecutive threads and every fragment read is
// unit-stride.  MFMA lane layout: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; element v of the result is D[4 v + l / 16][l % 16].
// Each output is one fp64 FMA chain over k in ascending order.
// C may be A where every workgroup writes only the rows it reads (Nc <= BT).
// Grid: (ceil(Nc / BT), ceil(Mr / BT), batch).
struct Batch64 {
    // product z is at element offsets (z / per) * hi + (z % per) * lo
    int n = 1, per = 1;
    int64_t a_hi = 0, a_lo = 0, b_hi = 0, b_lo = 0, c_hi = 0, c_lo = 0;
};

template <int BT, int BK>
__global__ __launch_bounds__(1024) void gemm64(int64_t Mr, int64_t Nc, int64_t K, double alpha, const double* A,
                                               int64_t sa0, int64_t sa1, const double* __restrict__ B, int64_t sb0,
                                               int64_t sb1, double beta, double* C, int64_t sc0, int64_t sc1,
                                               int lower, Batch64 bt) {
    constexpr int NT = 1024, LD = BT + 1, PT = BT * BK / NT;
    constexpr int WT = BT / 4, TT = WT / 16;
    static_assert(PT >= 1 && BT * BK % NT == 0 && WT % 16 == 0 && BK % 4 == 0, "bad fp64 tile");
    const int64_t i0 = (int64_t)blockIdx.y * BT, j0 = (int64_t)blockIdx.x * BT;
    if (lower && j0 > i0) return;
    {
        const int64_t hi = blockIdx.z / bt.per, lo = blockIdx.z % bt.per;
        A += hi * bt.a_hi + lo * bt.a_lo;
        B += hi * bt.b_hi + lo * bt.b_lo;
        C += hi * bt.c_hi + lo * bt.c_lo;
    }
    __shared__ double As[2][BK * LD];
    __shared__ double Bs[2][BK * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3;
    const bool a_k1 = sa1 == 1, b_j1 = sb1 == 1;
    // element e of a staged tile: (row ii, depth kk) of A, (depth kb, column jj) of B
    auto a_at = [&](int e, int& ii, int& kk) {
        ii = a_k1 ? e / BK : e % BT;
        kk = a_k1 ? e % BK : e / BT;
    };
    auto b_at = [&](int e, int& kb, int& jj) {
        jj = b_j1 ? e % BT : e / BK;
        kb = b_j1 ? e / BT : e % BK;
    };
    // this thread's elements: source pointers (a valid one where the row or
    // column is out of range) that step with K, LDS offsets
    const double *pa[PT], *pb[PT];
    int la[PT], lb[PT], ka[PT], kb_[PT];
    bool oka[PT], okb[PT];
#pragma unroll
    for (int q = 0; q < PT; ++q) {
        int ii, kk, kb, jj;
        a_at(tid + NT * q, ii, kk);
        b_at(tid + NT * q, kb, jj);
        oka[q] = i0 + ii < Mr;
        okb[q] = j0 + jj < Nc;
        pa[q] = A + (oka[q] ? i0 + ii : 0) * sa0 + kk * sa1;
        pb[q] = B + kb * sb0 + (okb[q] ? j0 + jj : 0) * sb1;
        ka[q] = kk;
        kb_[q] = kb;
        la[q] = kk * LD + ii;
        lb[q] = kb * LD + jj;
    }
    double ra[PT], rb[PT];
    auto gload = [&](int64_t k0) {
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            ra[q] = (oka[q] && k0 + ka[q] < K) ? *pa[q] : 0.0;
            rb[q] = (okb[q] && k0 + kb_[q] < K) ? *pb[q] : 0.0;
            pa[q] += BK * sa1;
            pb[q] += BK * sb0;
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            As[buf][la[q]] = ra[q];
            Bs[buf][lb[q]] = rb[q];
        }
    };
    f64x4 acc[TT][TT];
#pragma unroll
    for (int a = 0; a < TT; ++a)
#pragma unroll
        for (int b = 0; b < TT; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int64_t nk = (K + BK - 1) / BK;
    gload(0);
    sstore(0);
    __syncthreads();
    const int fr = lane & 15, fk = lane >> 4;
    for (int64_t kt = 0; kt < nk; ++kt) {
        const int cur = (int)(kt & 1);
        if (kt + 1 < nk) gload((kt + 1) * BK);  // in flight during this tile's MFMAs
#pragma unroll
        for (int s = 0; s < BK / 4; ++s) {
            double fa[TT], fb[TT];
#pragma unroll
            for (int a = 0; a < TT; ++a) fa[a] = As[cur][(s * 4 + fk) * LD + wm * WT + a * 16 + fr];
#pragma unroll
            for (int b = 0; b < TT; ++b) fb[b] = Bs[cur][(s * 4 + fk) * LD + wn * WT + b * 16 + fr];
#pragma unroll
            for (int a = 0; a < TT; ++a)
#pragma unroll
                for (int b = 0; b < TT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
        // the other buffer was last read before the previous barrier
        if (kt + 1 < nk) sstore(cur ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < TT; ++a)
#pragma unroll
        for (int b = 0; b < TT; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t i = i0 + wm * WT + a * 16 + 4 * v + fk, j = j0 + wn * WT + b * 16 + fr;
                if (i < Mr && j < Nc) {
                    double* c = C + i * sc0 + j * sc1;
                    *c = beta == 0.0 ? alpha * acc[a][b][v] : fma(alpha, acc[a][b][v], beta * *c);
                }
            }
}

// *out = 1e-13 * max_i A[i][i] (n x n, row stride ld): the smallest pivot a
// factorisation accepts, i.e. a bound of about 1e13 on the condition number.
// One workgroup of 256 threads.
constexpr double kPivotTol = 1e-13;

__global__ __launch_bounds__(256) void pivot_floor64(const double* __restrict__ A, int64_t n, int64_t ld,
                                                     double* __restrict__ out) {
    __shared__ double red[256];
    double mx = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) mx = fmax(mx, A[i * ld + i]);
    red[threadIdx.x] = mx;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = kPivotTol * red[0];
}

// Cholesky of the nb x nb (nb <= 64) block at A (row stride ld), in place
// (lower triangle; the upper part is neither read nor written), and the
// inverse of the factor into Linv (row stride ldi, 64 x 64, zero above the
// diagonal, identity past nb).
// One workgroup of 256 threads; thread (ty, tx) of a 16 x 16 grid holds rows
// ty + 16a and columns tx + 16b (a, b < 4) of the block and of an identity
// matrix in registers.  Step j eliminates column j below the diagonal from
// both, without square roots (A = L D L^T first): the owners of column j and
// of the identity's row j publish them in LDS (alternating buffers), one
// barrier, and every thread reads the pivot and its rows' and columns' values
// and updates its 32 elements.  The identity becomes the unit factor's
// inverse; square roots of the pivots scale both at the end.  Bound: the
// latency of 64 dependent steps (LDS, barrier, division); the two-barrier
// form with the block in LDS and a square root per step took 46 us (this 30),
// and the inverses 23 us in a kernel of their own.
// *info is set to 1 on a pivot that is not finite or not above *floor (the
// matrix is not numerically positive definite).
__global__ __launch_bounds__(256) void chol_diag(double* __restrict__ A, int64_t ld, int nb,
                                                 const double* __restrict__ floor, int* __restrict__ info,
                                                 double* __restrict__ Linv, int64_t ldi) {
    __shared__ double col[2][kG64], row[2][kG64], piv[kG64];
    const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
    double a[4][4], e[4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = ty + 16 * p, c = tx + 16 * q;
            const bool in = c <= i && i < nb;
            const double v = A[in ? (int64_t)i * ld + c : 0];  // in bounds, no branch
            e[p][q] = i == c ? 1.0 : 0.0;
            a[p][q] = in ? v : e[p][q];
        }
    const double fl = *floor;
    bool bad = false;
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
#pragma unroll 1
        for (int jj = 0; jj < 16; ++jj) {
            const int j = 16 * jb + jj, buf = j & 1;
            if (tx == jj)
#pragma unroll
                for (int p = 0; p < 4; ++p) col[buf][ty + 16 * p] = a[p][jb];
            if (ty == jj)
#pragma unroll
                for (int q = 0; q < 4; ++q) row[buf][tx + 16 * q] = e[jb][q];
            __syncthreads();
            const double d = col[buf][j];
            const bool ok = j >= nb || (d > fl && d > 0.0 && __builtin_isfinite(d));
            bad |= !ok;
            const double dd = ok ? d : 1.0;
            if (tid == 0) piv[j] = dd;
            const double inv = 1.0 / dd;
            double f[4], lc[4], er[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int i = ty + 16 * p, c = tx + 16 * p;
                f[p] = i > j ? col[buf][i] * inv : 0.0;
                lc[p] = c > j ? col[buf][c] : 0.0;
                er[p] = row[buf][c];
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q <= p) a[p][q] -= f[p] * lc[q];
                    if (q <= p) e[p][q] -= f[p] * er[q];
                }
        }
    }
    __syncthreads();
    if (bad && tid == 0) *info = 1;
    if (tid < kG64) piv[tid] = sqrt(piv[tid]);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = ty + 16 * p, c = tx + 16 * q;
            if (c <= i && i < nb) A[(int64_t)i * ld + c] = i == c ? piv[i] : a[p][q] / piv[c];
            Linv[i * ldi + c] = c <= i ? e[p][q] / piv[i] : 0.0;
        }
}

// out = a * X + b * Y + d * I (m x n row-major; Y may be null, then b is
// ignored; out may be X or Y)
__global__ void axpby_diag64(int64_t m, int64_t n, double a, const double* X, double b, const double* Y, double d,
                             double* out) {
    const int64_t total = m * n;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        double v = a * X[e];
        if (Y) v += b * Y[e];
        if (d != 0.0 && e / n == e % n) v += d;
        out[e] = v;
    }
}

// out (cols x rows) = in^T (rows x cols), fp64, 32 x 32 LDS tiles.
__global__ __launch_bounds__(256) void transpose64(const double* __restrict__ in, int64_t rows, int64_t cols,
                                                   double* __restrict__ out) {
    __shared__ double t[32][33];
    const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int k = ty; k < 32; k += 8) {
        const int64_t r = r0 + k, c = c0 + tx;
        t[k][tx] = (r < rows && c < cols) ? in[r * cols + c] : 0.0;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {
        const int64_t c = c0 + k, r = r0 + tx;
        if (c < cols && r < rows) out[c * rows + r] = t[tx][k];
    }
}

// Epilogue for the MFMA GEMM: out[m * ld + n] += acc (the running fp64 sums
// of the calibration statistics; fp32 products are accumulated in fp64).
// With lower_tiles, output tiles entirely above the diagonal are skipped (a
// symmetric sum; complete_lower64 fills them afterwards).
// out holds at least kAccF64MinElems values, a run of any tile.
constexpr int64_t kAccF64MinElems = 32;

struct AccF64Epi {
    double* out;
    int64_t ld, N, M;
    bool lower_tiles;
    __device__ __forceinline__ bool skip_tile(int64_t m0, int64_t n0, int BM, int BN) const {
        (void)BN;
        return lower_tiles && n0 >= m0 + BM;
    }
    struct Col {
        int64_t n;
        bool ok;
    };
    __device__ __forceinline__ Col col(int64_t n) const { return Col{n, n < N}; }
    __device__ __forceinline__ void store(int64_t m, const Col& c, float v) const {
        if (m < M && c.ok) out[m * ld + c.n] += (double)v;
    }
    // A run's old values are loaded ahead of the run before it (Old): added in
    // place run by run, every run waited a memory round trip for its own (a
    // 4096 x 4096 x 2048 product 113 us, 106 so; the lower tiles 95, 90).
    // 16-byte accesses, which global memory takes at 8-byte alignment, so rows
    // of any length take them.
    typedef double f64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
    template <int W>
    struct Old {
        double v[W];
    };
    template <int W>
    __device__ __forceinline__ Old<W> old(int64_t m, int64_t n) const {
        static_assert(W <= kAccF64MinElems, "run past the smallest sums");
        Old<W> o;
        // unconditional, from a valid address, where the run is not whole (the
        // sums' allocation holds a run; a branch here took 3% of a batch)
        const bool whole = m < M && n + W <= N;
        const f64x2_a8* src = reinterpret_cast<const f64x2_a8*>(out + (whole ? m * ld + n : 0));
#pragma unroll
        for (int x = 0; x < W / 2; ++x) {
            const f64x2_a8 s = src[x];
            o.v[2 * x] = s[0];
            o.v[2 * x + 1] = s[1];
        }
        return o;
    }
    template <int W>
    __device__ __forceinline__ void run(int64_t m, int64_t n, const float (&v)[W], const Old<W>& o) const {
        if (m >= M || n >= N) return;
        double* dst = out + m * ld + n;
        if (n + W <= N) {
#pragma unroll
            for (int x = 0; x < W / 2; ++x)
                reinterpret_cast<f64x2_a8*>(dst)[x] =
                    f64x2_a8{o.v[2 * x] + (double)v[2 * x], o.v[2 * x + 1] + (double)v[2 * x + 1]};
        } else {
#pragma unroll
            for (int x = 0; x < W; ++x)
                if (n + x < N) dst[x] += (double)v[x];
        }
    }
};

// out = the symmetric matrix of which S (n x n row-major) holds the lower
// triangle (and whole diagonal tiles): completes a sum accumulated in its
// lower tiles only.  out may be S.  One workgroup per 32 x 32 tile of the
// lower triangle, transposed through LDS so that both halves are read and
// written along rows (element by element across the rows it took 65 us for n
// = 4096, and the copy to the caller's buffer 55 more).
__global__ __launch_bounds__(256) void complete_lower64(const double* S, int64_t n, double* out) {
    __shared__ double t[32][33];
    if (blockIdx.x > blockIdx.y) return;
    const int64_t i0 = (int64_t)blockIdx.y * 32, j0 = (int64_t)blockIdx.x * 32;
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int k = ty; k < 32; k += 8) {
        const int64_t i = i0 + k, j = j0 + tx;
        const double v = i < n && j < n ? S[i * n + j] : 0.0;
        t[k][tx] = v;
        if (out != S && i < n && j <= i) out[i * n + j] = v;
    }
    __syncthreads();
    for (int k = ty; k < 32; k += 8) {  // row j0 + k of the upper triangle
        const int64_t j = j0 + k, i = i0 + tx;
        if (i < n && j < i) out[j * n + i] = t[tx][k];
    }
}

}  // namespace pifa
