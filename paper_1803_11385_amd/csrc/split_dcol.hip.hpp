// The gradient of the column matrix, out[i][n] = sum over k of A[i][k] * W[n][k] (A = dY, rows of 32, 64 or 128 channels; W the weights,
// a row for each of the 27 * c_in columns), with fp32 operands on the bf16 matrix instruction: operands cut into three bf16
// pieces as in split_wgrad.hip.hpp, six products per term.
#pragma once
#include "split_conv.hip.hpp"

namespace hch {

// A workgroup of 8 wavefronts takes 128 rows, a wavefront 16 of them, which it cuts once and keeps in registers; then the columns
// of its share pass by, 128 / KS of them at a time: one piece of 8 weights for each thread, cut on its way into LDS, two stages, one barrier.
// Bound by the stores of the matrix with 32 channels, by the matrix instructions and LDS with more.  With the gather behind it, against
// gemm_f32_kernel: 16 -> 32 (channels of X, of dY) at 82 000 voxels 63 -> 50 us, 32 -> 64 at 23 000 50.5 -> 35, at 282 000 564 -> 402, 64 -> 128 at 5400
// 37 -> 32, at 82 000 456 -> 305.
// KS: steps of 32 channels.
template <int KS>
struct DcolLds {
    static constexpr int NT = 8 / KS, BN = 16 * NT, PIECES = KS * 4;
    static constexpr int LKS = BN * 16, PLANE = PIECES * LKS, STAGE = 3 * PLANE, BYTES = 2 * STAGE;
    static_assert(BN * PIECES == 512, "a piece for each thread");
};

template <int KS>
__global__ __launch_bounds__(512, 4) void dcol_split_kernel(
    const float *__restrict__ A, const float *__restrict__ W, float *__restrict__ out, int M, int N, unsigned row_tiles, int chunks)
{
    typedef DcolLds<KS> L;
    constexpr int NT = L::NT, BN = L::BN, K = 32 * KS, SRD3 = 0x00020000;
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::BYTES];
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x / NUM_XCD);
    if (tile >= row_tiles) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int row = ((int)tile * 8 + __builtin_amdgcn_readfirstlane(tid >> 6)) * 16 + li;
    const int c_beg = (int)blockIdx.y * chunks, c_end = min(c_beg + chunks, (N + BN - 1) / BN);
    if (c_beg >= c_end) return;
    const __amdgpu_buffer_rsrc_t rs_a = __builtin_amdgcn_make_buffer_rsrc((void *)A, 0, M * K * 4, SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, N * K * 4, SRD3);

    // weights: piece wp (8 channels) of column wn of a chunk
    const int wn = tid / L::PIECES, wp = tid % L::PIECES;
    u32x4 rw[2];
    auto fetch = [&](int chunk) {                                          // columns past the end: past the buffer, zero
        const int off = ((chunk * BN + wn) * K + wp * 8) * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) rw[h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, off + 16 * h, 0, 0));
    };
    auto cut = [&](const u32x4 *r, u32x4 *p) {
        float f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = __uint_as_float(r[j >> 2][j & 3]);
        split3(f, p[0], p[1], p[2]);
    };
    auto stash = [&](int stage) {
        u32x4 p[3];
        cut(rw, p);
        unsigned char *dst = lds + stage * L::STAGE + wp * L::LKS + (wn ^ unit_swap(wp & 3)) * 16;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4 *>(dst + pl * L::PLANE) = p[pl];
    };
    fetch(c_beg);
    u32x4 x[KS][3];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        u32x4 r[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            r[h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_a, (row * K + s * 32 + lk * 8) * 4 + 16 * h, 0, 0));
        cut(r, x[s]);
    }
    stash(0);
    __syncthreads();
    for (int chunk = c_beg, stage = 0; chunk < c_end; ++chunk, stage ^= 1) {
        fetch(chunk + 1);                                                  // past the last: multiplied by nobody
        f32x4 acc[NT], low[NT];
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            // the operands change places: a lane ends up with 4 neighbouring columns of one row
            constexpr int G = NT < 4 ? NT : 4;
#pragma unroll
            for (int b0 = 0; b0 < NT; b0 += G) {
                u32x4 w[G][3];
#pragma unroll
                for (int b = 0; b < G; ++b)
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
                        w[b][pl] = *reinterpret_cast<const u32x4 *>(lds + stage * L::STAGE + pl * L::PLANE + (s * 4 + lk) * L::LKS + ((b0 + b) * 16 + (li ^ unit_swap(lk))) * 16);
                constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int b = 0; b < G; ++b) acc[b0 + b] = mfma_bf16(w[b][0], x[s][0], acc[b0 + b]);
#pragma unroll
                for (int t = 0; t < 5; ++t)
#pragma unroll
                    for (int b = 0; b < G; ++b) low[b0 + b] = mfma_bf16(w[b][PB[t]], x[s][PA[t]], low[b0 + b]);
            }
        }
        bool bad = false;
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            acc[b] += low[b];
#pragma unroll
            for (int e = 0; e < 4; ++e) bad |= non_finite(acc[b][e]);
            acc[b] *= SPLIT_UNSCALE;
        }
        if (__builtin_expect(__ballot(bad) != 0, 0)) {
            // an infinity or NaN among the operands, or a sum out of range: with the fp32 instruction, from memory
#pragma unroll
            for (int b = 0; b < NT; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int k = lk * 8; k < K; k += 32) {
                float f[8], w[8];
                load8(A + (int64_t)min(row, M - 1) * K + k, 8, f);
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    load8(W + (int64_t)min(chunk * BN + b * 16 + li, N - 1) * K + k, 8, w);
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 8; ++j) t = mfma_f32(w[j], f[j], t);
                    acc[b] += t;
                }
            }
        }
        if (row < M) {
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int col = chunk * BN + b * 16 + lk * 4;
                if (col < N) *reinterpret_cast<f32x4 *>(out + (int64_t)row * N + col) = acc[b];
            }
        }
        if (chunk + 1 < c_end) stash(stage ^ 1);
        __syncthreads();
    }
}

}  // namespace hch
