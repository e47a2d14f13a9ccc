// Gathered product of the 3x3x3 convolution (forward, data gradient) for few voxels, C[i][n] = sum over the taps t and
// channels k of X[nbr[i][t]][k] * W(t, k, n), with fp32 operands on the bf16 matrix instruction: both operands cut into three bf16
// pieces as in split_wgrad.hip.hpp, six products per term.
#pragma once
#include "split_conv.hip.hpp"

namespace hch {

// A workgroup computes 16 rows by 16*NT columns, rows in data order; its WV = 8 wavefronts share out the reduction, not the rows: in units of 8
// channels of one tap that any of the 16 rows has, 4 units (32 terms) to a step, a wavefront takes every WV-th step.  Each reads its rows and weights
// from memory straight into the operands' layout, cuts both and keeps sums of its own, which meet in LDS as they are, leading pieces' and the others'
// apart, and are added in 64 bits and rounded once (with a rounding per wavefront short reductions came out further from the exact sums than
// conv_split_kernel's one chain: 1 -> 4 channels 5.5e-8 for 3.2e-8).  Nothing is shared on the way, so there is no barrier between the index rows and
// the end, and no launch that adds up partial sums.
// Bound by the latency of that chain: index rows, rows and weights, the last sum; conv_split_kernel, whose workgroups walk through all steps one
// after the other, or through a part of them with a launch to add the parts, takes longer wherever all workgroups of this one are resident at once.
// It reads and cuts every weight for 16 rows only, which is what it loses with more rows (figures at conv_small_faster).
// BT: W(t, k, n) = W[26 - t][n][k] (the data gradient's view of the weights), else W[t][k][n].
constexpr int SMALL_WAVES = 8;
template <int NT, bool BT>
__global__ __launch_bounds__(64 * SMALL_WAVES, 2) void conv_small_kernel(
    const float *__restrict__ X, const float *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr, int M, int N, int c, int vec_out)
{
    constexpr int ROWS = 16, BN = 16 * NT, WV = SMALL_WAVES, SRD3 = 0x00020000;
    constexpr uint32_t OUT = 0x80000000u;
    __shared__ __attribute__((aligned(16))) int32_t idx[ROWS * 27];
    __shared__ uint8_t taplist[32];
    __shared__ __attribute__((aligned(16))) f32x4 sums[WV][2][NT][64];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = (int)blockIdx.x * ROWS, n0 = (int)blockIdx.y * BN;
    const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, M * 27 * 4, SRD3);
    for (int e = tid; e < ROWS * 27; e += 64 * WV) {
        const bool ok = row0 + e / 27 < M;
        const int v = (int)__builtin_amdgcn_raw_buffer_load_b32(rs_n, ok ? (row0 * 27 + e) * 4 : (int)OUT, 0, 0);
        idx[e] = ok ? v : -1;
    }
    __syncthreads();
    // taps that the rows have, the list of them (each wavefront writes the same)
    int any = -1;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) any &= idx[r * 27 + min(lane, 26)] >> 31;
    const uint32_t present = (uint32_t)__ballot(lane < 27 && any == 0);
    const int n_present = __popc(present), c8 = (c + 7) >> 3, n_units = n_present * c8, n_steps = (n_units + 3) >> 2;
    if (lane < 32) {
        if (lane >= n_present) taplist[lane] = 0;                          // past the last: tap 0, with no weights
        if (present >> lane & 1u) taplist[__popc(present & ((1u << lane) - 1u))] = (uint8_t)lane;
    }
    __builtin_amdgcn_wave_barrier();

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)((int64_t)M * c * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, 27 * c * N * 4, SRD3);
    const bool whole = (c & 7) == 0;                                       // units have 8 channels each
    // rows and weights of step s: 8 channels of row li, and the same of columns b * 16 + li
    auto fetch = [&](int s, float *x, float (*w)[8]) {
        const int unit = s * 4 + lk, at = unit / c8, u = unit - at * c8;
        const int tap = taplist[min(at, 31)];
        const bool real = at < n_present;
        const int row = __mul24(idx[li * 27 + tap], c * 4), xo = row < 0 || !real ? (int)OUT : row + u * 32;
        // (channels past the row's end, the next row's, meet weights of zero -- and if they are not finite, the plain sums are taken)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, xo + 16 * h, 0, 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) x[4 * h + j] = v[j];
        }
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int col = n0 + b * 16 + li;
            const bool ok = real && col < N;
            if (BT && whole) {
                const int o = ok ? (((26 - tap) * N + col) * c + u * 8) * 4 : (int)OUT;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, o + 16 * h, 0, 0));
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[b][4 * h + j] = v[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = u * 8 + j, o = BT ? ((26 - tap) * N + col) * c + k : (tap * c + k) * N + col;
                    w[b][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, ok && k < c ? o * 4 : (int)OUT, 0, 0));
                }
            }
        }
    };

    f32x4 acc[NT], low[NT];
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const float *x, const float (*w)[8]) {
        u32x4 xp[3], wp[NT][3];
        split3(x, xp[0], xp[1], xp[2]);
#pragma unroll
        for (int b = 0; b < NT; ++b) split3(w[b], wp[b][0], wp[b][1], wp[b][2]);
        constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = mfma_bf16(wp[b][0], xp[0], acc[b]);
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int b = 0; b < NT; ++b) low[b] = mfma_bf16(wp[b][PB[t]], xp[PA[t]], low[b]);
    };
    if (wave < n_steps) {
        float x0[8], x1[8], w0[NT][8], w1[NT][8];
        fetch(wave, x0, w0);
        int s = wave;
        for (; s + WV < n_steps; s += 2 * WV) {
            fetch(s + WV, x1, w1);
            multiply(x0, w0);
            fetch(s + 2 * WV, x0, w0);                                     // past the last step: nothing that counts
            multiply(x1, w1);
        }
        if (s < n_steps) multiply(x0, w0);
    }
    bool bad = false;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= non_finite(acc[b][e] + low[b][e]);
        acc[b] *= SPLIT_UNSCALE;
        low[b] *= SPLIT_UNSCALE;
    }
    if (__builtin_expect(__ballot(bad) != 0, 0)) {
        // an infinity or NaN among the operands, or a sum out of range: this wavefront's sums with the fp32 instruction, one
        // unit at a time, added only where the row has the tap, as in conv_split_kernel
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = wave; s < n_steps; s += WV)
            for (int u = s * 4; u < min(s * 4 + 4, n_units); ++u) {
                const int tap = taplist[u / c8], k0 = u % c8 * 8 + lk * 2, row = idx[li * 27 + tap];
                if (__ballot(row >= 0) == 0) continue;
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    const int col = n0 + b * 16 + li;
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int k = k0 + j;
                        const float xv = row >= 0 && k < c ? X[(int64_t)row * c + k] : 0.f;
                        const float wv = k < c && col < N ? W[BT ? ((int64_t)(26 - tap) * N + col) * c + k : ((int64_t)tap * c + k) * N + col] : 0.f;
                        t = mfma_f32(wv, xv, t);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][e] += row >= 0 ? t[e] : 0.f;
                }
            }
    }
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        sums[wave][0][b][lane] = acc[b];
        sums[wave][1][b][lane] = low[b];
    }
    __syncthreads();
    for (int q = tid; q < NT * 64; q += 64 * WV) {
        const int b = q >> 6, l = q & 63;
        double t[4] = {0., 0., 0., 0.};
#pragma unroll
        for (int w = 0; w < WV; ++w)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 part = sums[w][h][b][l];
#pragma unroll
                for (int e = 0; e < 4; ++e) t[e] += (double)part[e];
            }
        const f32x4 v = {(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
        const int row = row0 + (l & 15), col = n0 + b * 16 + (l >> 4) * 4;
        if (row >= M) continue;
        float *dst = C + (int64_t)row * N + col;
        if (vec_out && col + 4 <= N) *reinterpret_cast<f32x4 *>(dst) = v;
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < N) dst[e] = v[e];
    }
}

}  // namespace hch
