// PIFA build on the GPU (Algorithm "Pivoting Factorization", Sec. 3.2), fp64.
//
// QR with column pivoting (Businger & Golub) on A = W'^T: column j of A is
// row j of W', so A is held as d_out contiguous columns of length d_in -- the
// bytes of W' in row-major order.  Step k picks the column of largest
// residual norm (ties to the lowest original row index), swaps it into
// position k and turns A[k:, k] into a Householder reflector H = I - tau v v^T
// (v[0] = 1 implicit, v[1:] stored below the diagonal, R[k][k] on it); the
// steps run in panels whose trailing update is one GEMM (qr_panel_* below).
// After r steps R11 (r x r, upper triangular) and R12 (r x (d_out - r)) sit in
// the first r entries of the columns.  The coefficient matrix solves
// W_p^T C^T = W_np^T in the least-squares sense through those factors:
// C R11^T = R12^T (row by row a back substitution), done by
// coeff_solve in blocks of 64 unknowns, each workgroup owning 64 rows of C.
#pragma once

#include "common.hpp"

namespace pifa {

constexpr int kPivotThreads = 512;  // per workgroup of a pivot step
constexpr int kPivotBlocks = 16;    // workgroups of a pivot step, at most

// Cross-lane moves on the VALU (DPP) instead of the LDS crossbar that
// __shfl_xor uses.  dpp<CTRL, ROWS>(x, old): lane l gets x from the lane CTRL
// names; lanes of rows outside the ROWS mask get old.  Controls used:
// quad_perm [1,0,3,2] (0xB1) and [2,3,0,1] (0x4E), row_ror:4 (0x124) and
// :8 (0x128), row_bcast:15 (0x142) and :31 (0x143).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp32(uint32_t x, uint32_t old) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ double dpp64(double x, double old) {
    const uint2 u = __builtin_bit_cast(uint2, x), o = __builtin_bit_cast(uint2, old);
    const uint2 r = {dpp32<CTRL, ROWS>(u.x, o.x), dpp32<CTRL, ROWS>(u.y, o.y)};
    return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ double lane63(double x) {
    const uint2 u = __builtin_bit_cast(uint2, x);
    const uint2 r = {(uint32_t)__builtin_amdgcn_readlane((int)u.x, 63), (uint32_t)__builtin_amdgcn_readlane((int)u.y, 63)};
    return __builtin_bit_cast(double, r);
}

// The sum of x over the wave's 64 lanes (every lane active), returned to
// every lane: a butterfly within each quad and each row of 16 lanes, then the
// rows folded into lane 63.  A fixed order, so the result is deterministic,
// and equal inputs give equal sums.  (About 4x faster than the same
// reduction through __shfl_xor, which moves doubles through the LDS
// crossbar: the 17 sums of a pivot step took 22 K of its 49 K cycles.)
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp64<0xB1>(x, 0.0);
    x += dpp64<0x4E>(x, 0.0);
    x += dpp64<0x124>(x, 0.0);
    x += dpp64<0x128>(x, 0.0);
    x += dpp64<0x142, 0xA>(x, 0.0);  // rows 1 and 3 add rows 0 and 2
    x += dpp64<0x143, 0xC>(x, 0.0);  // rows 2 and 3 add rows 0 + 1
    return lane63(x);
}

// A (d_out columns of length d_in) = W' rows; norm2[j] = ||A_j||^2; perm[j] = j.
__global__ __launch_bounds__(256) void qr_init(const double* __restrict__ W, double* __restrict__ A,
                                               double* __restrict__ norm2, int32_t* __restrict__ perm,
                                               int64_t d_out, int64_t d_in) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t j = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (j >= d_out) return;
    const double* w = W + j * d_in;
    double* a = A + j * d_in;
    double s = 0.0;
    for (int64_t i = lane; i < d_in; i += kWave) {
        const double x = w[i];
        a[i] = x;
        s += x * x;
    }
    s = wave_sum(s);
    if (lane == 0) {
        norm2[j] = s;
        perm[j] = (int32_t)j;
    }
}

// The pivoting runs in panels of at most kPanel steps (the blocked form of
// LAPACK's xGEQP3 / xLAQPS): inside a panel the trailing columns are not
// updated; each step k = k0 + j instead adds a column to
//   F (d_out x kPanel, row c at F + c * kPanel):  F[c, j] = tau_k a_c^(k)T v_k,
// where a_c^(k) = a_c - V[:, 0:j] F[c, 0:j]^T is column c after the panel's
// earlier reflections and V holds their Householder vectors (stored in
// A's columns k0 .. k-1 below the diagonal, with an implicit 1 on it).  Row k
// of every trailing column is brought up to date at its step (it becomes
// row k of R), and the residual norms are downdated by that row's squares.
// At the end of a panel one GEMM, A[rows >= k0+nb, cols >= k0+nb] -= V F^T,
// applies the panel's reflections to the rest of the trailing matrix, and
// the residual norms of the trailing columns are recomputed exactly, so every
// panel starts from exact norms.  The trailing matrix is read once per step
// and written once per panel, instead of read twice and written once per
// step.
constexpr int kPanel = 16;

// One step of a wave argmax over (value v, key k, index i): take the partner
// lane's triple (dpp64 / dpp32 with control CTRL, rows ROWS; lanes outside
// ROWS see their own) if its value is larger, or equal with a smaller key.
template <int CTRL, int ROWS>
__device__ __forceinline__ void argmax_step(double& v, int32_t& k, int32_t& i) {
    const double ov = dpp64<CTRL, ROWS>(v, v);
    const int32_t ok = (int32_t)dpp32<CTRL, ROWS>((uint32_t)k, (uint32_t)k);
    const int32_t oi = (int32_t)dpp32<CTRL, ROWS>((uint32_t)i, (uint32_t)i);
    if (ov > v || (ov == v && ok < k)) {
        v = ov;
        k = ok;
        i = oi;
    }
}

// The pivot of step k, for a workgroup of kPivotThreads threads (all of them
// call it): the column c in [k, d_out) of largest norm2[c], ties to the
// lowest original index perm[c]; k where no norm compares (all NaN).  The
// comparison is a total order, so every workgroup finds the same column.
// Eight candidates are loaded at a time (clamped, so no branch per load), and
// every wave folds the waves' results itself: one barrier.
__device__ __forceinline__ int64_t block_pivot(const double* __restrict__ norm2, const int32_t* __restrict__ perm,
                                               int64_t k, int64_t d_out, double* s_val, int32_t* s_idx,
                                               int32_t* s_key) {
    static_assert(kPivotThreads / kWave <= 16, "the waves' results are folded within a row of 16 lanes");
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    double bv = -1.0;
    int32_t bi = -1, bk = INT32_MAX;
    for (int64_t c0 = k + tid; c0 < d_out; c0 += 8 * kPivotThreads) {
        double v[8];
        int32_t key[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t c = min(c0 + u * kPivotThreads, d_out - 1);  // the last column again: no effect
            v[u] = norm2[c];
            key[u] = perm[c];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v[u] > bv || (v[u] == bv && key[u] < bk)) {
                bv = v[u];
                bi = (int32_t)min(c0 + u * kPivotThreads, d_out - 1);
                bk = key[u];
            }
    }
    argmax_step<0xB1, 0xF>(bv, bk, bi);
    argmax_step<0x4E, 0xF>(bv, bk, bi);
    argmax_step<0x124, 0xF>(bv, bk, bi);
    argmax_step<0x128, 0xF>(bv, bk, bi);
    argmax_step<0x142, 0xA>(bv, bk, bi);
    argmax_step<0x143, 0xC>(bv, bk, bi);
    if (lane == kWave - 1) {
        s_val[wave] = bv;
        s_idx[wave] = bi;
        s_key[wave] = bk;
    }
    __syncthreads();
    const int w = lane & (kPivotThreads / kWave - 1);
    bv = s_val[w];
    bi = s_idx[w];
    bk = s_key[w];
    argmax_step<0xB1, 0xF>(bv, bk, bi);
    argmax_step<0x4E, 0xF>(bv, bk, bi);
    argmax_step<0x124, 0xF>(bv, bk, bi);
    argmax_step<0x128, 0xF>(bv, bk, bi);
    const int64_t p = __builtin_amdgcn_readlane(bi, 63);
    return p < k ? k : p;
}

// The sum over each row of 16 lanes, returned to all of them.
__device__ __forceinline__ double row_sum(double x) {
    x += dpp64<0xB1>(x, 0.0);
    x += dpp64<0x4E>(x, 0.0);
    x += dpp64<0x124>(x, 0.0);
    x += dpp64<0x128>(x, 0.0);
    return x;
}

// The reflector of a column x with squared norm s and leading entry alpha:
// R's diagonal entry beta, tau, and inv with v = x * inv below the leading 1.
// A zero column keeps its entries (tau = 0).
struct Reflector {
    double beta, tau, inv;
};
__device__ __forceinline__ Reflector reflector(double s, double alpha) {
    const double xnorm = sqrt(s);
    if (xnorm == 0.0) return {alpha, 0.0, 1.0};
    const double beta = -copysign(xnorm, alpha);
    return {beta, (beta - alpha) / beta, 1.0 / (alpha - beta)};
}

// What the workgroups of qr_panel_pivot leave for the step's GEMV and for the
// next step: row t < kPanel holds the workgroups' shares of sum_{i > k} V[i, t] x[i],
// row kPanel those of ||x||^2; then alpha = x[k].  Two of them, by the
// step's parity: a step writes its own while it reads the one before.
struct PivotSums {
    double share[kPanel + 1][kPivotBlocks];
    double alpha;
};

// Step k = k0 + j, part 1 (n_wg <= kPivotBlocks workgroups, rows interleaved
// between them; each finds the pivot for itself):
//   * pivot: the column p of largest (downdated) residual norm, ties to the
//     lowest original index.  Column k moves to p; F row, norm and original
//     index follow in part 2, because other workgroups still compare them here;
//   * column k = the pivot column after the panel's earlier reflections,
//     x = a_p - V[:, 0:j] F[p, 0:j]^T on rows [k, d_in), not yet scaled;
//   * the sums the reflector needs (PivotSums);
//   * the reflector of step k - 1 of the same panel is scaled where its rows
//     are read anyway (v = x inv, R's diagonal entry above it).
// Latency-bound: rows of V and of column k are loaded before the pivot is
// known.  One workgroup of 1024 threads for all rows took 15.1 us per step at
// 4096 x 4096, bound by one CU's loads of V and its 17 sums; spread out, the
// whole build of r = 2048 went from 72.5 to 60.1 ms.
// status[0] is set to 1 if a pivot column is zero.
__global__ __launch_bounds__(kPivotThreads) void qr_panel_pivot(double* __restrict__ A,
                                                                const double* __restrict__ norm2,
                                                                const int32_t* __restrict__ perm,
                                                                const double* __restrict__ F,
                                                                PivotSums* __restrict__ sums,
                                                                int64_t* __restrict__ pivot, int* __restrict__ status,
                                                                int64_t k, int64_t k0, int64_t d_out, int64_t d_in,
                                                                int n_wg) {
    constexpr int kWaves = kPivotThreads / kWave;
    __shared__ double s_val[kWaves];
    __shared__ int32_t s_idx[kWaves], s_key[kWaves];
    __shared__ double s_sum[kWaves][kPanel + 1];
    __shared__ double fk[kPanel];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int j = (int)(k - k0);
    double* x = A + k * d_in;
    const int64_t stride = (int64_t)n_wg * kPivotThreads;
    int64_t i = (int64_t)blockIdx.x * kPivotThreads + tid;

    double vrow[kPanel], xk = 0.0;
    auto load = [&](int64_t row) {
        const bool ok = row < d_in;
        xk = ok ? x[row] : 0.0;
#pragma unroll
        for (int t = 0; t < kPanel; ++t) vrow[t] = (ok && row >= k && t < j) ? A[(k0 + t) * d_in + row] : 0.0;
    };
    load(i);
    Reflector prev = {0.0, 0.0, 1.0};
    if (j > 0) {
        const PivotSums& ps = sums[(k - 1) & 1];
        const int g = lane & (kPivotBlocks - 1);
        const double s = row_sum(g < n_wg ? ps.share[kPanel][g] : 0.0);
        prev = reflector(s, ps.alpha);
        if (s == 0.0 && blockIdx.x == 0 && tid == 0) status[0] = 1;
    }

    const int64_t p = block_pivot(norm2, perm, k, d_out, s_val, s_idx, s_key);
    if (tid < kPanel) fk[tid] = tid < j ? F[p * kPanel + tid] : 0.0;
    if (blockIdx.x == 0 && tid == 0) *pivot = p;
    double* ap = A + p * d_in;
    __syncthreads();  // fk

    PivotSums& out = sums[k & 1];
    double s = 0.0, dot[kPanel];
#pragma unroll
    for (int t = 0; t < kPanel; ++t) dot[t] = 0.0;
    for (; i < d_in; i += stride) {
        double v = p != k ? ap[i] : xk;
        if (p != k) ap[i] = xk;
        if (i >= k) {
#pragma unroll
            for (int t = 0; t < kPanel; ++t) {
                if (t == j - 1) {
                    vrow[t] *= prev.inv;
                    A[(k0 + t) * d_in + i] = vrow[t];
                }
                v -= vrow[t] * fk[t];  // zero past j
            }
            s += v * v;
            if (i == k) out.alpha = v;
            else {
#pragma unroll
                for (int t = 0; t < kPanel; ++t) dot[t] += vrow[t] * v;
            }
        } else if (j > 0 && i == k - 1) {
            A[(k - 1) * d_in + i] = prev.beta;
        }
        if (i >= k || p != k) x[i] = v;
        if (i + stride < d_in) load(i + stride);
    }
    s = wave_sum(s);
    if (lane == 0) s_sum[wave][kPanel] = s;
#pragma unroll
    for (int t = 0; t < kPanel; ++t)
        if (t < j) {
            const double d = wave_sum(dot[t]);
            if (lane == 0) s_sum[wave][t] = d;
        }
    __syncthreads();
    if (tid < j || tid == kPanel) {
        double d = 0.0;
        for (int w = 0; w < kWaves; ++w) d += s_sum[w][tid];
        out.share[tid][blockIdx.x] = d;
    }
}

// The scaling of a panel's last reflector, k (no next step reads its rows).
__global__ __launch_bounds__(256) void qr_panel_finish(double* __restrict__ A, const PivotSums* __restrict__ sums,
                                                       int* __restrict__ status, int64_t k, int64_t d_in, int n_wg) {
    const PivotSums& ps = sums[k & 1];
    const int g = threadIdx.x & (kPivotBlocks - 1);
    const double s = row_sum(g < n_wg ? ps.share[kPanel][g] : 0.0);
    const Reflector h = reflector(s, ps.alpha);
    double* x = A + k * d_in;
    const int64_t i = k + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < d_in) x[i] = i == k ? h.beta : x[i] * h.inv;
    if (i == k && s == 0.0) status[0] = 1;
}

// Step k = k0 + j, part 2: one wave per trailing column c > k, read only
// except for three values per column:
//   F[c, j]  = tau_k a_c^T v_k + F[c, 0:j] aux[0:j]  (a_c as of the panel start),
//              aux[t] = -tau_k V[k:, t]^T v_k
//   R[k][c]  = a_c[k] - V[k, 0:j] F[c, 0:j]^T - F[c, j]   (written to a_c[k])
//   norm2[c] -= R[k][c]^2
// with v_k = x inv below its leading 1 (x is not scaled yet: column k).  Each
// wave folds the pivot workgroups' sums itself, behind its column's loads.
// The wave of column p, where column k went, takes k's F row, norm and
// original index over.
__global__ __launch_bounds__(256) void qr_panel_gemv(double* __restrict__ A, double* __restrict__ norm2,
                                                     int32_t* __restrict__ perm, double* __restrict__ F,
                                                     const PivotSums* __restrict__ sums,
                                                     const int64_t* __restrict__ pivot, int64_t k, int64_t k0,
                                                     int64_t d_out, int64_t d_in, int n_wg) {
    static_assert(kPanel == 16 && kPivotBlocks == 16, "lane l folds share l % 16 of rows l / 16 + 4 q");
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t c = k + 1 + (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (c >= d_out) return;
    const int j = (int)(k - k0);
    const double* v = A + k * d_in;  // x
    double* a = A + c * d_in;
    const PivotSums& ps = sums[k & 1];
    const bool moved = *pivot == c;  // column k came here
    const int64_t src = moved ? k : c;
    const int g = lane & 15;
    double share[4], f[4], vk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int t = 4 * q + lane / 16;
        share[q] = (t < j && g < n_wg) ? ps.share[t][g] : 0.0;
        f[q] = (t < j && g == 0) ? F[src * kPanel + t] : 0.0;
        vk[q] = (t < j && g == 0) ? A[(k0 + t) * d_in + k] : 0.0;
    }
    const double nshare = g < n_wg ? ps.share[kPanel][g] : 0.0;
    const double alpha = ps.alpha, akc = a[k], n2c = norm2[src];
    double d;
    if ((d_in & 1) == 0) {
        // 16-byte loads of rows [s2, d_in), s2 = k + 1 rounded up to even,
        // four pairs in flight per lane (clamped indices, masked products: no
        // branch per load); row k + 1 on its own when it is odd.  The order
        // depends only on k, so equal columns give equal sums.
        const int64_t s = k + 1, s2 = s + (s & 1), n2 = d_in / 2;
        const double2* v2 = reinterpret_cast<const double2*>(v);
        const double2* a2 = reinterpret_cast<const double2*>(a);
        double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int64_t q = s2 / 2 + lane; q < n2; q += 4 * kWave) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t qu = q + u * kWave;
                const bool ok = qu < n2;
                const int64_t qc = ok ? qu : n2 - 1;
                const double2 vv = v2[qc], aa = a2[qc];
                acc[2 * u] += ok ? vv.x * aa.x : 0.0;
                acc[2 * u + 1] += ok ? vv.y * aa.y : 0.0;
            }
        }
        d = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
        if (lane == 0 && (s & 1) && s < d_in) d += v[s] * a[s];
    } else {
        double d1 = 0.0, d2 = 0.0;
        int64_t i = k + 1 + lane;
        for (; i + kWave < d_in; i += 2 * kWave) {
            d1 += v[i] * a[i];
            d2 += v[i + kWave] * a[i + kWave];
        }
        if (i < d_in) d1 += v[i] * a[i];
        d = d1 + d2;
    }
    d = wave_sum(d);
    const Reflector h = reflector(row_sum(nshare), alpha);
    // lane 16 w holds rows 4 q + w of F[c, :], V[k, :] and the sums V^T x
    double corr = 0.0, row = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        corr += f[q] * row_sum(share[q]);
        row += f[q] * vk[q];
    }
    corr = wave_sum(corr);
    row = wave_sum(row);
    double* Fc = F + c * kPanel;
    if (moved && g == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int t = 4 * q + lane / 16;
            if (t < j) Fc[t] = f[q];
        }
    }
    if (lane == 0) {
        const double fj = h.tau * (akc + h.inv * d) - h.tau * (row + h.inv * corr);
        Fc[j] = fj;
        const double rkc = akc - row - fj;
        a[k] = rkc;
        norm2[c] = fmax(n2c - rkc * rkc, 0.0);
        if (moved) {
            const int32_t t = perm[k];
            perm[k] = perm[c];
            perm[c] = t;
        }
    }
}

// Exact residual norms ||A_c[k:]||^2 of columns c >= k (one wave per column).
__global__ __launch_bounds__(256) void qr_norms(const double* __restrict__ A, double* __restrict__ norm2, int64_t k,
                                                int64_t d_out, int64_t d_in) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t c = k + (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (c >= d_out) return;
    const double* a = A + c * d_in;
    double s = 0.0;
    for (int64_t i = k + lane; i < d_in; i += kWave) s += a[i] * a[i];
    s = wave_sum(s);
    if (lane == 0) norm2[c] = s;
}

// diag[k] = R[k][k] = A_k[k] for k < r.
__global__ void extract_diag(const double* __restrict__ A, double* __restrict__ diag, int64_t r, int64_t d_in) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < r; k += (int64_t)gridDim.x * blockDim.x)
        diag[k] = A[k * d_in + k];
}

// R11 in row-major form: RT[s][t] = A_t[s] for s <= t < r, 0 below.
__global__ void extract_r11(const double* __restrict__ A, double* __restrict__ RT, int64_t r, int64_t d_in) {
    const int64_t total = r * r;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s = e / r, t = e % r;
        RT[e] = t >= s ? A[t * d_in + s] : 0.0;
    }
}

// C (n_np x r) with C R11^T = R12^T, i.e. for each row q of C:
//   sum_{t >= s} R11[s][t] c[t] = b[s],  b[s] = A_{r+q}[s]   (s < r),
// solved from the last unknown up in blocks of kSolveBlock unknowns,
// right-looking: X = the right-hand sides (coeff_rhs); for each block, from
// the last, coeff_block_solve finds the block's unknowns of every row by
// substitution against R11's diagonal block, and one fp64 MFMA GEMM (gemm64)
// subtracts their contribution from the right-hand sides of all earlier
// unknowns.  The GEMMs carry the n_np r^2 FLOPs over the whole chip, where a
// left-looking solve with one workgroup per 64 rows of C kept n_np / 64
// workgroups busy (32 at 4096 x 4096, r = 2048).
constexpr int kSolveBlock = 64;

__global__ void coeff_rhs(const double* __restrict__ A, double* __restrict__ X, int64_t r, int64_t n_np,
                          int64_t d_in) {
    const int64_t total = n_np * r;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t q = e / r, s = e % r;
        X[e] = A[(r + q) * d_in + s];
    }
}

// Unknowns [s0, s0 + nb) of rows [64 b, 64 b + 64) of X, in place: thread t
// substitutes row 64 b + t against the diagonal block of R11 (upper
// triangular, row-major in RT with row stride r).
__global__ __launch_bounds__(kSolveBlock) void coeff_block_solve(const double* __restrict__ RT, double* __restrict__ X,
                                                                  int64_t r, int64_t n_np, int64_t s0, int nb) {
    __shared__ double sD[kSolveBlock][kSolveBlock + 1];
    __shared__ double sB[kSolveBlock][kSolveBlock + 1];
    const int tid = threadIdx.x;
    const int64_t q0 = (int64_t)blockIdx.x * kSolveBlock;
    for (int e = tid; e < kSolveBlock * kSolveBlock; e += kSolveBlock) {
        const int a = e / kSolveBlock, b = e % kSolveBlock;
        sD[a][b] = (a < nb && b < nb) ? RT[(s0 + a) * r + s0 + b] : 0.0;
        const int64_t q = q0 + a;
        sB[a][b] = (q < n_np && b < nb) ? X[q * r + s0 + b] : 0.0;
    }
    __syncthreads();
    for (int a = nb - 1; a >= 0; --a) {
        double v = sB[tid][a];
        for (int b = a + 1; b < nb; ++b) v -= sD[a][b] * sB[tid][b];
        sB[tid][a] = v / sD[a][a];
    }
    __syncthreads();
    for (int e = tid; e < kSolveBlock * kSolveBlock; e += kSolveBlock) {
        const int row = e / kSolveBlock, col = e % kSolveBlock;
        const int64_t q = q0 + row;
        if (q < n_np && col < nb) X[q * r + s0 + col] = sB[row][col];
    }
}

// Outputs in sorted order: W_p[i] = W'[pivot_idx[i]], and
// C_out[q][i] = C_sel[row_src[q]][col_src[i]].
__global__ void gather_rows(const double* __restrict__ W, const int32_t* __restrict__ rows, double* __restrict__ out,
                            int64_t n_rows, int64_t n_cols) {
    const int64_t total = n_rows * n_cols;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / n_cols, c = e % n_cols;
        out[e] = W[(int64_t)rows[i] * n_cols + c];
    }
}

__global__ void gather_coeffs(const double* __restrict__ Csel, const int32_t* __restrict__ row_src,
                              const int32_t* __restrict__ col_src, double* __restrict__ out, int64_t n_np,
                              int64_t r) {
    const int64_t total = n_np * r;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t q = e / r, i = e % r;
        out[e] = Csel[(int64_t)row_src[q] * r + col_src[i]];
    }
}

}  // namespace pifa
