// Kernels of the PIFA layer backward pass (bf16 layers).
//
// Forward (Algorithm "PIFA Layer", row-major):  Y_p = X W_p^T,
// Y_np = Y_p C^T, Y[:, I] = Y_p, Y[:, I^c] = Y_np.  With G = dL/dY the chain
// rule gives
//   G_p  = G[:, I] + G[:, I^c] C      (M x r)
//   dX   = G_p W_p                    (M x d_in)
//   dW_p = G_p^T X                    (r x d_in)
//   dC   = G[:, I^c]^T Y_p            (n_np x r)
// All four are products for the prefill GEMM (gemm_dma.hpp, gemm_mfma.hpp).  G_p and dX
// take K-contiguous operands; dW_p and dC reduce over the activation rows
// and read their operands K-major (rows of G_p, X, G[:, I^c], Y[:, I]).  This
// file holds the gathers of G[:, I^c], G[:, I] and Y[:, I] as rows, the
// transposed weight packs and the epilogues of the G_p and dX products (and the
// transpose that calibration batches of unaligned rows take).
//
// Precision: G_p multiplies W_p in dX = G_p W_p with the same cancellation as
// Y_p C^T in the forward (C rebuilds W_np from W_p): a bf16 G_p misses the
// bf16 bar there (about 7e-3 measured on QR-pivoted layers), fp16 meets it
// (about 2e-3).  G_p is therefore kept in fp32 and converted row by row to
// fp16 times 2^s_m, s_m chosen from the row's largest |value|, against an
// fp16 copy of W_p^T scaled by 2^c; the product is multiplied back by
// 2^-(s_m + c), which is exact.  dW_p and dC have no such cancellation and
// use bf16 operands; all products accumulate in fp32.
#pragma once

#include "common.hpp"
#include "epilogue.hpp"
#include "layout.hpp"

namespace pifa {

// Element (n, k) of a lane-ordered matrix with KB 128-column blocks per row group.
__device__ __forceinline__ int64_t lane_order_index(int64_t n, int64_t k, int64_t KB) {
    const int64_t g = n / kPackRows, b = k / kPackCols;
    const int rr = (int)(n % kPackRows), cc = (int)(k % kPackCols);
    const int l = 16 * (cc / 32) + rr, c = (cc % 32) / 8, e = cc % 8;
    return ((g * KB + b) * kPackChunks + c * 64 + l) * 8 + e;
}

template <typename T>
__device__ __forceinline__ float to_f32(T v);
template <>
__device__ __forceinline__ float to_f32<bf16>(bf16 v) {
    return bf16_bits_to_f32(__builtin_bit_cast(uint16_t, v));
}
template <>
__device__ __forceinline__ float to_f32<f16>(f16 v) {
    return (float)v;
}

// dst = lane order of a (rows_log x cols_log) matrix of type TD whose element
// (i, c) is src(c mod period, i) * scale, where src is a lane-ordered matrix
// (src_kb column blocks per row group) of which rows < src_rows and columns
// < src_cols are valid; everything else is zero.  Used for W_p^T in fp16
// times 2^c and for C^T in bf16 (scale undoing C's fp16 scale, exact for
// bf16-representable C); period = cols_log unless a copy repeats along K.
template <typename TS, typename TD>
__global__ void pack_transposed(const TS* __restrict__ src, int64_t src_kb, int64_t src_rows, int64_t src_cols,
                                int64_t period, float scale, TD* __restrict__ dst, int64_t rows_log,
                                int64_t cols_log) {
    const int64_t KB = packed_kblocks(cols_log);
    const int64_t nchunks = packed_groups(rows_log) * KB * kPackChunks;
    for (int64_t ch = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; ch < nchunks;
         ch += (int64_t)gridDim.x * blockDim.x) {
        const int64_t blk = ch / kPackChunks;
        const int pos = (int)(ch % kPackChunks);
        const int c = pos / 64, l = pos % 64;
        const int64_t g = blk / KB, b = blk % KB;
        const int64_t i = g * kPackRows + (l % 16);
        const int64_t k0 = b * kPackCols + 32 * (l / 16) + 8 * c;
        TD* out = dst + ch * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t k = k0 + e;
            const int64_t s = k % period;
            float v = 0.f;
            if (i < rows_log && k < cols_log && s < src_rows && i < src_cols)
                v = to_f32<TS>(src[lane_order_index(s, i, src_kb)]) * scale;
            if constexpr (__is_same(TD, f16)) out[e] = (f16)v;
            else reinterpret_cast<uint16_t*>(out)[e] = f32_to_bf16_bits(v);
        }
    }
}

// One pass over a 64 x 64 tile of in (M x n, row stride n), written
// transposed: out[j * ld + m] for m < ld (zero for m >= M), with 16-byte
// stores (ld a multiple of 8).  Rows of 16-byte units are read 8 columns per
// load, others one.  Grid: (ceil(ld / 64), ceil(n / 64)).
constexpr int kTrTile = 64;

__global__ __launch_bounds__(256) void transpose_tile(const bf16* __restrict__ in, int64_t M, int64_t n,
                                                      bf16* __restrict__ out, int64_t ld) {
    __shared__ uint16_t tile[kTrTile][kTrTile + 2];
    const uint16_t* src = reinterpret_cast<const uint16_t*>(in);
    const int64_t m0 = (int64_t)blockIdx.x * kTrTile, j0 = (int64_t)blockIdx.y * kTrTile;
    const int tid = threadIdx.x;
    if ((n & 7) == 0 && (reinterpret_cast<uintptr_t>(in) & 15) == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ch = tid + 256 * i, mm = ch / 8, j8 = (ch % 8) * 8;
            const int64_t m = m0 + mm, j = j0 + j8;
            uint16_t v[8] = {};
            if (m < M && j < n) {
                const u32x4 w = *reinterpret_cast<const u32x4*>(src + m * n + j);
                __builtin_memcpy(v, &w, 16);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) tile[mm][j8 + e] = v[e];
        }
    } else {
        // every load is unconditional (clamped row, a valid column): under a
        // lane condition each would be a branch whose join waits for it, one
        // memory round trip per element
        const int jj = tid % kTrTile;
        const int64_t j = j0 + jj;
        constexpr int kPer = kTrTile * kTrTile / 256;
        uint16_t v[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int64_t m = m0 + tid / kTrTile + 4 * i;
            v[i] = src[(m < M ? m : M - 1) * n + (j < n ? j : 0)];
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int mm = tid / kTrTile + 4 * i;
            tile[mm][jj] = (m0 + mm < M && j < n) ? v[i] : (uint16_t)0;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int ch = tid + 256 * i;  // 512 chunks of 8 elements per tile
        const int a = ch / 8, b8 = (ch % 8) * 8;
        const int64_t j = j0 + a, m = m0 + b8;  // row j of the transpose, columns m .. m + 7
        if (j < n && m < ld) {
            uint16_t v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = tile[b8 + e][a];
            *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(out) + j * ld + m) = __builtin_bit_cast(u32x4, v);
        }
    }
}

// Rows of in (M x d, row stride d) split by column sets: out_a[m][j] =
// in[m][ia[j]] for j < na (zeros up to lda) and, if out_b, out_b[m][j] =
// in[m][ib[j]] for j < nb (zeros up to ldb); lda and ldb are even and the
// outputs 4-byte aligned.  Both kernels below give a lane two neighbouring
// columns of several rows, so that a wave's stores are 256 contiguous bytes.
struct ColumnSplit {
    const bf16* in;
    int64_t d, M;
    const int32_t* ia;
    int64_t na;
    bf16* out_a;
    int64_t lda;
    const int32_t* ib;
    int64_t nb;
    bf16* out_b;
    int64_t ldb;

    int64_t pairs() const { return (lda + (out_b ? ldb : 0)) / 2; }

    // pair p of the output columns: a's, then b's
    struct Pair {
        int32_t c0, c1;  // source columns, -1 for a zero
        uint16_t* out;
        int64_t ld;
    };
    __device__ __forceinline__ Pair pair(int64_t p) const {
        const bool b = 2 * p >= lda;
        const int32_t* idx = b ? ib : ia;
        const int64_t n = b ? nb : na, j = b ? 2 * p - lda : 2 * p;
        const int32_t c0 = idx[j < n ? j : n - 1], c1 = idx[j + 1 < n ? j + 1 : n - 1];
        return Pair{j < n ? c0 : -1, j + 1 < n ? c1 : -1, reinterpret_cast<uint16_t*>(b ? out_b : out_a) + j,
                    b ? ldb : lda};
    }
};

// A workgroup reads R rows once, whole lines at a time, into LDS and gathers
// from there: with sorted indices the 2-byte LDS reads of a wave span a few
// hundred bytes (8 columns per lane, for 16-byte stores, put 8 lanes on each
// bank).  The rows are one span of memory, read in 16-byte units from the
// boundary below its start, whatever its alignment.  Bound: memory.
// Dynamic LDS: R rows and, unless every row starts on a 16-byte boundary, 16
// bytes more.
constexpr int kSplitRows = 4;  // R, and rows per lane of the direct form

__global__ __launch_bounds__(512) void split_columns(ColumnSplit s, int R) {
    extern __shared__ __attribute__((aligned(16))) uint16_t rows[];
    const int64_t m0 = (int64_t)blockIdx.x * R;
    const int nr = (int)((s.M - m0) < R ? (s.M - m0) : R);
    const uint16_t* src = reinterpret_cast<const uint16_t*>(s.in) + m0 * s.d;
    const int shift = (int)((reinterpret_cast<uintptr_t>(src) & 15) / 2);  // LDS position of the first value
    const int64_t n = nr * s.d, units = ceil_div(shift + n, (int64_t)8);
    if (m0 * s.d >= shift && 8 * units - shift <= (s.M - m0) * s.d) {
        const u32x4* span = reinterpret_cast<const u32x4*>(src - shift);
        for (int64_t q = threadIdx.x; q < units; q += 512) reinterpret_cast<u32x4*>(rows)[q] = span[q];
    } else {  // the matrix starts or ends inside a unit
        for (int64_t e = threadIdx.x; e < n; e += 512) rows[shift + e] = src[e];
    }
    __syncthreads();
    auto gather = [&](const int32_t* __restrict__ idx, int64_t ni, bf16* __restrict__ out, int64_t ld) {
        for (int64_t j = 2 * threadIdx.x; j < ld; j += 2 * 512) {
            const int32_t c0 = idx[j < ni ? j : ni - 1], c1 = idx[j + 1 < ni ? j + 1 : ni - 1];
            for (int r = 0; r < nr; ++r) {
                const uint16_t* row = rows + shift + r * s.d;
                const uint32_t x = j < ni ? row[c0] : 0, y = j + 1 < ni ? row[c1] : 0;
                *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(out) + (m0 + r) * ld + j) = x | (y << 16);
            }
        }
    };
    gather(s.ia, s.na, s.out_a, s.lda);
    if (s.out_b) gather(s.ib, s.nb, s.out_b, s.ldb);
}

// Straight from memory, kSplitRows rows per lane with their loads in flight
// together: no barrier and no pass through LDS, but a line is asked for once
// per 2-byte value.  Grid: (ceil(M / kSplitRows), ceil(pairs / 256)).
__global__ __launch_bounds__(256) void split_columns_direct(ColumnSplit s) {
    const int64_t p = (int64_t)blockIdx.y * 256 + threadIdx.x, m0 = (int64_t)blockIdx.x * kSplitRows;
    if (p >= (s.lda + (s.out_b ? s.ldb : 0)) / 2) return;
    const ColumnSplit::Pair c = s.pair(p);
    const uint16_t* src = reinterpret_cast<const uint16_t*>(s.in);
    uint32_t x[kSplitRows], y[kSplitRows];
#pragma unroll
    for (int r = 0; r < kSplitRows; ++r) {  // unconditional, from valid addresses
        const uint16_t* row = src + (m0 + r < s.M ? m0 + r : s.M - 1) * s.d;
        x[r] = row[c.c0 >= 0 ? c.c0 : 0];
        y[r] = row[c.c1 >= 0 ? c.c1 : 0];
    }
#pragma unroll
    for (int r = 0; r < kSplitRows; ++r)
        if (m0 + r < s.M)
            *reinterpret_cast<uint32_t*>(c.out + (m0 + r) * c.ld) =
                (c.c0 >= 0 ? x[r] : 0u) | (c.c1 >= 0 ? y[r] << 16 : 0u);
}

// Epilogue of G_p = G[:, I^c] C (+ G[:, I]): acc(m, n) for n < r_pad.
//   * adds gpi[m * r_pad + n] = G[m, piv[n]] (zeros at n >= r), the gathered
//     pivot columns: the register-staged tiles and the K-split reduction start
//     from it (init), the direct tiles add it to the finished sums (Old).
//     Loaded ahead of the loop it left the 256 x 256 and 256 x 192 tiles 32 to
//     126 registers short, which they spilled around every K tile: 4096 x 3648
//     x 496 71 us, 4096 x 2880 x 8144 269, so 48 and 214;
//   * writes G_p in fp32 to gp[m * r_pad + n], for the row-wise fp16
//     conversion;
//   * writes bf16(G_p) to gpb[m * r_pad + n]: the K-major A operand of
//     dW_p = G_p^T X.
// The padding columns are not masked here: C^T's padding rows and their
// starting values are zero, and no reader takes more than r columns.  gpi, gp
// and gpb have 16-byte aligned rows (r_pad is a multiple of 64).
struct GradPivotEpi {
    static constexpr bool kRowsPlusStaged = true;
    const bf16* gpi;
    int64_t r_pad;
    float* gp;
    bf16* gpb;
    int64_t M;

    struct Col {
        int64_t n;
        bool ok;
    };
    __device__ __forceinline__ Col col(int64_t n) const { return Col{n, n < r_pad}; }
    // Loads below are unconditional, from clamped (valid) addresses: a load
    // under a lane-dependent condition is compiled as a branch that waits for it.
    __device__ __forceinline__ float init(int64_t m, const Col& c) const {
        const uint16_t* g16 = reinterpret_cast<const uint16_t*>(gpi);
        const float g = bf16_bits_to_f32(g16[(m < M ? m : 0) * r_pad + (c.ok ? c.n : 0)]);
        return (c.ok && m < M) ? g : 0.f;
    }
    // A run of W columns starts at a multiple of 8 and goes in pieces of 8,
    // each wholly inside or wholly past the r_pad columns: where W does not
    // divide r_pad's unit of 64 (24, on the 256 x 192 tile) the last run of a
    // row is cut.
    template <int W>
    struct Old {
        u32x4 g[W / 8];
    };
    template <int W>
    __device__ __forceinline__ Old<W> old(int64_t m, int64_t n) const {
        static_assert(W % 8 == 0, "pieces of 8 columns");
        const bf16* row = gpi + (m < M ? m : 0) * r_pad;
        Old<W> o;
#pragma unroll
        for (int x = 0; x < W / 8; ++x)
            o.g[x] = *reinterpret_cast<const u32x4*>(row + (n + 8 * x < r_pad ? n + 8 * x : 0));
        return o;
    }
    template <int W>
    __device__ __forceinline__ void run(int64_t m, int64_t n, const float (&v)[W], const Old<W>& o) const {
        if (m >= M) return;
        float* d = gp + m * r_pad + n;
        uint16_t* b = reinterpret_cast<uint16_t*>(gpb) + m * r_pad + n;
#pragma unroll
        for (int x = 0; x < W; x += 8) {
            if (n + x >= r_pad) return;
            float s[8];
            uint16_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t u = o.g[x / 8][e / 2];
                s[e] = v[x + e] + bf16_bits_to_f32((uint16_t)(e % 2 ? u >> 16 : u));
                h[e] = f32_to_bf16_bits(s[e]);
            }
            reinterpret_cast<f32x4*>(d + x)[0] = f32x4{s[0], s[1], s[2], s[3]};
            reinterpret_cast<f32x4*>(d + x)[1] = f32x4{s[4], s[5], s[6], s[7]};
            store_run16<8>(b + x, h);
        }
    }
    __device__ __forceinline__ void store(int64_t m, const Col& c, float v) const {
        if (m >= M || !c.ok) return;
        gp[m * r_pad + c.n] = v;
        reinterpret_cast<uint16_t*>(gpb)[m * r_pad + c.n] = f32_to_bf16_bits(v);
    }
    // rows m .. m + 3 (m % 4 == 0) of column c, fp32 rows only
    __device__ __forceinline__ void store4_rows(int64_t m, const Col& c, const float (&v)[4]) const {
        if (!c.ok || m >= M) return;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (m + e < M) gp[(m + e) * r_pad + c.n] = v[e];
    }
    __device__ __forceinline__ StagedEpi<bf16> staged() const {
        return StagedEpi<bf16>{reinterpret_cast<uint16_t*>(gpb), r_pad, r_pad, 1.f, nullptr, M};
    }
};

// Row m of gp (n = r_pad fp32 values, n % 4 == 0, of which r are G_p's and
// the rest count as zero) -> fp16 out[m][:] times 2^s_m with the row's largest
// |value| in [2^14, 2^15) (s_m = 0 for a zero row), and inv[m] = 2^-s_m.
// One workgroup of 256 threads per row.
__global__ __launch_bounds__(256) void rows_to_f16(const float* __restrict__ gp, int64_t r, int64_t n,
                                                   f16* __restrict__ out, float* __restrict__ inv) {
    __shared__ float red[256 / kWave];
    const int64_t m = blockIdx.x;
    const f32x4* row = reinterpret_cast<const f32x4*>(gp + m * n);
    const int64_t nq = n / 4;
    float mx = 0.f;
    for (int64_t q = threadIdx.x; q < nq; q += 256) {
        const f32x4 v = row[q];  // past r: zeros, or NaN, which fmaxf passes over
        mx = fmaxf(mx, fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))));
    }
    for (int off = kWave / 2; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    int s = 0;
    if (mx > 0.f && __builtin_isfinite(mx)) {
        int e = 0;
        (void)frexpf(mx, &e);  // mx = f * 2^e, f in [0.5, 1)
        s = 15 - e;            // mx * 2^s in [2^14, 2^15)
        s = s < -100 ? -100 : (s > 100 ? 100 : s);
    }
    const float sc = ldexpf(1.f, s);
    for (int64_t q = threadIdx.x; q < nq; q += 256) {
        f32x4 v = row[q];
        // a padding column is NaN where the gradient's row holds an infinity
        // (the product's zero weights times it): as a zero it adds nothing to dX
        const int left = (int)(r - 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] : 0.f;
        f16 h[4] = {(f16)(v[0] * sc), (f16)(v[1] * sc), (f16)(v[2] * sc), (f16)(v[3] * sc)};
        *reinterpret_cast<uint64_t*>(out + m * n + 4 * q) = __builtin_bit_cast(uint64_t, h);
    }
    if (threadIdx.x == 0) inv[m] = ldexpf(1.f, -s);
}

// Epilogue writing round(acc(m, n) * row_scale[m] * out_scale) to
// out[m * ldo + n] (bf16) for m < M, n < N.
struct RowScaleEpi {
    bf16* out;
    int64_t ldo, N;
    const float* row_scale;
    float out_scale;
    int64_t M;
    bool vec;  // rows of out are 16-byte aligned
    struct Col {
        int64_t n;
        bool ok;
    };
    __device__ __forceinline__ Col col(int64_t n) const { return Col{n, n < N}; }
    __device__ __forceinline__ void store(int64_t m, const Col& c, float v) const {
        if (m < M && c.ok) Store<bf16>::put(out + m * ldo + c.n, v * row_scale[m] * out_scale);
    }
    template <int W>
    struct Old {
        float scale;
    };
    template <int W>
    __device__ __forceinline__ Old<W> old(int64_t m, int64_t n) const {
        (void)n;
        return Old<W>{row_scale[m < M ? m : 0]};
    }
    template <int W>
    __device__ __forceinline__ void run(int64_t m, int64_t n, const float (&v)[W], const Old<W>& o) const {
        if (m >= M || n >= N) return;
        const float s = o.scale;
        uint16_t h[W];
#pragma unroll
        for (int x = 0; x < W; ++x) h[x] = f32_to_bf16_bits(v[x] * s * out_scale);
        uint16_t* dst = reinterpret_cast<uint16_t*>(out) + m * ldo + n;
        if (n + W <= N && vec) {
            store_run16<W>(dst, h);
        } else {
#pragma unroll
            for (int x = 0; x < W; ++x)
                if (n + x < N) dst[x] = h[x];
        }
    }
    // rows m .. m + 3 (m % 4 == 0) of column c: one 16-byte load of their
    // scales (row_scale holds M rounded up to 4 values)
    __device__ __forceinline__ void store4(int64_t m, const Col& c, const float (&v)[4]) const {
        if (m >= M || !c.ok) return;
        const f32x4 s = *reinterpret_cast<const f32x4*>(row_scale + m);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (m + e < M) Store<bf16>::put(out + (m + e) * ldo + c.n, v[e] * s[e] * out_scale);
    }
};

}  // namespace pifa
