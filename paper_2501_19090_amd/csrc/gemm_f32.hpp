// fp32 products on the fp32 matrix cores: acc(m, n) = sum_k A[m, k] * B[n, k],
// both row-major, with v_mfma_f32_16x16x4_f32 (fp32 products and sums).
//
// A BM x BN tile per workgroup of four waves (WM x 4 / WM), K in tiles of 32:
// the operand tiles go straight into an LDS ring of S stages
// (buffer_load ... lds), tile t + S - 1 being issued when tile t is read.
// LDS rows are 128 bytes, 16-byte chunk c of row n in slot c ^ ((n / 2) % 8),
// which spreads a fragment read over all banks (gemm_dma.hpp).  A lane reads
// four consecutive K values of its row and feeds them to four MFMAs, whose
// lane groups cover the other chunks; A and B use the same K order.
// Bound: the matrix cores (256 FLOP per cycle and CU, 154 TFLOP/s on a large
// library product).  1024 x 2048 x 4096 takes 150 us on 64 x 64 tiles (114
// TFLOP/s; waves of 16 x 64, with waves of 32 x 32 170 us; 128 x 64 tiles 152;
// 32 x 32 MFMAs the same); the vector-ALU kernel before it took 521 (33).
// Any shape and alignment works: rows of whole 16-byte chunks (VEC) are
// loaded 16 bytes per lane, others 4; loads out of range put zeros in LDS.
#pragma once

#include "common.hpp"
#include "epilogue.hpp"
#include "gemm_dma.hpp"

namespace pifa {

__device__ __forceinline__ void dma4(u32x4 rsrc, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds"
                 :
                 : "v"(voff), "s"(rsrc), "s"(lds)
                 : "memory", "m0");
}

// One operand's K tile: ROWS rows of 32 values, in pieces of one load
// instruction (VEC: 8 rows, else 2), dealt to the workgroup's four waves.
template <int ROWS, bool VEC>
struct F32Tile {
    static constexpr int kBytes = ROWS * 128;
    static constexpr int kPer = VEC ? 8 : 2;  // rows per piece
    static constexpr int kPieces = ROWS / kPer / 4;
    static_assert(ROWS % (4 * kPer) == 0, "pieces do not split over the waves");
    u32x4 rs;
    uint32_t off[kPieces];
    int kk[kPieces];  // K offset in the tile of the value(s) this lane loads

    __device__ __forceinline__ void init(const float* p, int64_t ld, int64_t row0, int64_t rows, int64_t K, int wave,
                                         int lane) {
        rs = raw_rsrc31(p + row0 * ld, ((rows - row0 - 1) * ld + K) * 4);
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            const int row = kPer * (wave + 4 * j) + lane / (64 / kPer), sw = (row >> 1) & 7;
            kk[j] = VEC ? 4 * ((lane & 7) ^ sw) : 4 * (((lane & 31) >> 2) ^ sw) + (lane & 3);
            off[j] = (uint32_t)((row * ld + kk[j]) * 4);
        }
    }
    __device__ __forceinline__ void issue(int64_t k0, int64_t K, int wave, uint32_t lds) const {
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            const uint32_t o = k0 + kk[j] < K ? off[j] + (uint32_t)(k0 * 4) : kMaskedOffset;
            if constexpr (VEC) dma16(rs, o, lds + (wave + 4 * j) * 1024);
            else dma4(rs, o, lds + (wave + 4 * j) * 256);
        }
    }
    // K values 16 s + 4 (l / 16) .. + 3 of row w0 + l % 16
    __device__ __forceinline__ static f32x4 frag(const char* st, int w0, int s, int lane) {
        const int n = w0 + (lane & 15);
        return *reinterpret_cast<const f32x4*>(st + n * 128 + (((4 * s + (lane >> 4)) ^ ((n >> 1) & 7)) << 4));
    }
};

template <int BM, int BN, int WM, int S, bool VEC, typename Epi>
__global__ __launch_bounds__(256) void gemm_nt_f32(const float* __restrict__ A, int64_t lda, int64_t M,
                                                   const float* __restrict__ B, int64_t ldb, int64_t N, int64_t K,
                                                   Epi epi) {
    using TA = F32Tile<BM, VEC>;
    using TB = F32Tile<BN, VEC>;
    constexpr int WN = 4 / WM, TM = BM / WM / 16, TN = BN / WN / 16;
    constexpr int STAGE = TA::kBytes + TB::kBytes, DPW = TA::kPieces + TB::kPieces;
    static_assert((S - 1) * DPW < 64, "more loads in flight than the counter holds");
    __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
    int64_t tm, tn;
    tile_coords<BM, BN>(blockIdx.x, ceil_div(M, BM), ceil_div(N, BN), tm, tn);
    const int64_t m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    TA ta;
    TB tb;
    ta.init(A, lda, m0, M, K, wave, lane);
    tb.init(B, ldb, n0, N, K, wave, lane);
    auto issue = [&](int64_t t) {
        const uint32_t lds = lds0 + (uint32_t)(t % S) * STAGE;
        ta.issue(t * 32, K, wave, lds);
        tb.issue(t * 32, K, wave, lds + TA::kBytes);
    };
    // the K tiles' halves are summed apart: chains half as long, less rounding
    f32x4 acc[2][TM][TN];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[s][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int64_t nk = ceil_div(K, 32);
#pragma unroll
    for (int t = 0; t < S - 1; ++t) issue(t);
    for (int64_t t = 0; t < nk; ++t) {
        wait_vm<(S - 2) * DPW>();  // this wave's part of tile t has landed
        slot_barrier();            // everyone's has, and tile t - 1 is read
        issue(t + S - 1);
        const char* st = smem + (t % S) * STAGE;
        f32x4 a[2][TM], b[2][TN];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[s][i] = TA::frag(st, wm + 16 * i, s, lane);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[s][j] = TB::frag(st + TA::kBytes, wn + 16 * j, s, lane);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[s][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][i][e], b[s][j][e], acc[s][i][j], 0, 0, 0);
        wait_lgkm0();
    }
    wait_vm<0>();
    // lane holds column lane % 16, rows 4 (lane / 16) + v
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const auto c = epi.col(n0 + wn + 16 * j + (lane & 15));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) 
                epi.store(m0 + wm + 16 * i + 4 * (lane >> 4) + v, c, acc[0][i][j][v] + acc[1][i][j][v]);
    }
}

}  // namespace pifa
