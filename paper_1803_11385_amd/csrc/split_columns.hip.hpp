// The forward product of the columns algorithm, C[i][n] = sum over k of col[i][k] * W[k][n], k = tap * c + channel, together with the column matrix
// itself: operands cut into three bf16 pieces as in split_wgrad.hip.hpp, six products per term.
#pragma once
#include "split_conv.hip.hpp"

namespace hch {

// conv_split_kernel's way through LDS and registers over all 27 taps and the rows in the order of the data; the rows that are gathered for a product
// are also stored as they come, instead of written by hash2col_kernel and read back by gemm_f32_kernel.  One tap after the other without padding; an
// absent row is a row of zeros, in the products as well.  Rows of a multiple of 4 channels.  Bound by the stores of the column matrix with few output
// columns (4 -> 16 at 280 000 rows: 121 MB in 34 us), by the matrix instructions and the cutting, as conv_split_kernel, with more.  The two launches
// -> this one: 4 -> 16 at 280 000 rows 66 -> 34 us, 12 -> 20 199 -> 138, 16 -> 32 237 -> 127, 32 -> 64 503 -> 230; at 82 000 16 -> 32 67 -> 38, 32 ->
// 64 144 -> 85; at 23 000 32 -> 64 49 -> 33, 64 -> 128 115 -> 79; at 800 18 -> 14.5, 128 -> 256 34 -> 26.
// STREAM: stores past the caches, a form of the kernel (as a condition in the loop the compiler makes one store of both).  64-byte pieces only
// (pieces that share a sector with the next step's become two writes: 12 -> 20 at 280 000 258 us), and with matrices beyond the last-level cache: 16
// -> 32 at 159 000 (263 MB) 93 -> 75, 32 -> 64 at 282 000 298 -> 230, 16 -> 16 197 -> 124, at 593 000 32 -> 64 615 -> 583, with the weight gradient
// that reads the matrix 305 -> 278 (16 -> 32), 593 -> 571, 301 -> 277, 1190 -> 1150; below, 32 -> 16 at 82 000 (270 MB) 56 -> 62. FAST: rows of a
// multiple of 32 channels; a step lies within one tap.
template <int NT, int WV, bool FAST, bool STREAM>
__global__ __launch_bounds__(64 * WV) void columns_split_kernel(
    const float *__restrict__ X, const float *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr, float *__restrict__ col,
    int M, int N, int c, unsigned m_tiles, int64_t c_split_stride, int vec_out)
{
    typedef ConvLds<NT, WV> L;
    constexpr int BN = L::BN, ROWS = L::ROWS, GROUP = ROWS * WV / 64;     // 64-row tiles per workgroup
    constexpr uint32_t OUT = 0x80000000u;
    constexpr int SRD3 = 0x00020000;
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::BYTES];

    const unsigned mtile = xcd_tile(blockIdx.x, gridDim.x / NUM_XCD);
    if (mtile >= (m_tiles + GROUP - 1) / GROUP) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (int)blockIdx.y * BN;
    const int row0 = ((int)mtile * WV + wave) * ROWS;                      // this wavefront's first row
    unsigned char *a_lds = lds + wave * L::A;
    int32_t *idx = reinterpret_cast<int32_t *>(lds + L::O_IDX + wave * L::IDX);
    const int K = 27 * c, n_steps = (K + 31) >> 5;
    const int per = (n_steps + (int)gridDim.z - 1) / (int)gridDim.z;
    const int s_beg = min((int)blockIdx.z * per, n_steps), s_end = min(s_beg + per, n_steps);

    // index rows of the wavefront's rows, tap-major in LDS; rows past the end have no neighbours
    {
        const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, M * 27 * 4, SRD3);
        int32_t v[(ROWS * 27 + 63) / 64];
#pragma unroll
        for (int q = 0; q < (ROWS * 27 + 63) / 64; ++q) {
            const int e = q * 64 + lane;
            v[q] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_n, (row0 * 27 + e) * 4, 0, 0);
            if (row0 + e / 27 >= M) v[q] = -1;
        }
#pragma unroll
        for (int q = 0; q < (ROWS * 27 + 63) / 64; ++q) {
            const int e = q * 64 + lane, rr = e / 27, t = e - rr * 27;
            if (rr < ROWS) idx[t * ROWS + rr] = v[q];
        }
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)((int64_t)M * c * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, K * N * 4, SRD3);
    // gathered rows: piece ap (16 bytes) of rows ar and ar + 8; weights: UN consecutive terms of one column per thread
    const int ap = lane & 7, ar = lane >> 3;
    constexpr int AU = ROWS / 8, UN = BN * 32 / (64 * WV);
    static_assert(UN >= 2 && UN <= 8, "whole pairs, within one unit");
    const int bn = tid % BN, kp = tid / BN;
    const int bk = kp * UN / 8, bs = kp * UN % 8;                           // unit, first term within it
    const bool b_col = n0 + bn < N;
    // this thread's first weight of the next step: the reduction advances the per-lane offset, which decides inside or outside (zero weights
    // past term K), and the scalar offset stays within the first rows
    uint32_t w_off = b_col ? ((uint32_t)(s_beg * 32 + kp * UN) * N + n0 + bn) * 4u : OUT;
    // tap and channel of the next step (FAST) or of this lane's piece of it
    int tap = (s_beg * 32 + (FAST ? 0 : ap * 4)) / c, ch = s_beg * 32 + (FAST ? 0 : ap * 4) - tap * c;
    if constexpr (FAST) { tap = __builtin_amdgcn_readfirstlane(tap); ch = __builtin_amdgcn_readfirstlane(ch); }
    const int d_tap = FAST ? 0 : 32 / c, d_ch = 32 - d_tap * c;
    auto fetch = [&](u32x4 *ra, float *rb) {
        const int t = min(tap, 26);                                        // past the end: any tap, with no weights
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            const int off = __mul24(idx[t * ROWS + ar + 8 * q], c * 4);
            if constexpr (FAST) ra[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off + ap * 16, __builtin_amdgcn_readfirstlane(ch * 4), 0));
            else ra[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off < 0 ? off : off + ch * 4, 0, 0));
        }
        tap += d_tap; ch += d_ch;
        if (ch >= c) { ch -= c; ++tap; }
#pragma unroll
        for (int j = 0; j < UN; ++j) rb[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, (int)w_off, j * N * 4, 0));
        w_off += 128u * N;
    };
    int k_col = s_beg * 32 + ap * 4;                                       // place in the column matrix of the piece laid down next
    auto stash_a = [&](const u32x4 *ra) {
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            const int r = ar + 8 * q;
            *reinterpret_cast<u32x4 *>(a_lds + r * 128 + ((ap ^ row_swap(r)) << 4)) = ra[q];
        }
        if (n0 == 0 && k_col < min(s_end * 32, K))
#pragma unroll
            for (int q = 0; q < AU; ++q) {
                if (row0 + ar + 8 * q >= M) continue;
                u32x4 *dst = reinterpret_cast<u32x4 *>(col + (int64_t)(row0 + ar + 8 * q) * K + k_col);
                if constexpr (STREAM) __builtin_nontemporal_store(ra[q], dst); else *dst = ra[q];
            }
        k_col += 32;
    };
    auto stash_b = [&](int stage, const float *rb) {
        unsigned char *dst = lds + L::O_B + stage * L::B + bk * L::LKS + (bn ^ unit_swap(bk)) * 16 + bs * 2;
        uint32_t p[3][UN / 2];
        split3n<UN / 2>(rb, p[0], p[1], p[2]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) __builtin_memcpy(__builtin_assume_aligned(dst + pl * L::PLANE, UN * 2), p[pl], UN * 2);
    };

    f32x4 acc[NT], low[NT];                                                // leading pieces' products and the others, as there
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int stage, u32x4 *ra, float *rb) {
        float f[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4 raw = *reinterpret_cast<const u32x4 *>(a_lds + li * 128 + (((lk * 2 + h) ^ row_swap(li)) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * h + e] = __uint_as_float(raw[e]);
        }
        stash_a(ra);                                                       // step t + 1, after the reads of step t
        stash_b(stage ^ 1, rb);
        fetch(ra, rb);                                                     // step t + 3
        // the operands change places: a lane ends up with 4 neighbouring columns of one row
        u32x4 x[3], w[NT][3];
        split3(f, x[0], x[1], x[2]);
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                w[b][pl] = *reinterpret_cast<const u32x4 *>(lds + L::O_B + stage * L::B + pl * L::PLANE + lk * L::LKS + (b * 16 + (li ^ unit_swap(lk))) * 16);
        constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = mfma_bf16(w[b][0], x[0], acc[b]);
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int b = 0; b < NT; ++b) low[b] = mfma_bf16(w[b][PB[t]], x[PA[t]], low[b]);
        __syncthreads();
    };
    if (s_beg < s_end) {
        u32x4 ra0[AU], ra1[AU];
        float rb0[UN], rb1[UN];
        fetch(ra0, rb0);
        fetch(ra1, rb1);
        stash_a(ra0);
        stash_b(0, rb0);
        fetch(ra0, rb0);
        __syncthreads();
        int t = s_beg;
        for (; t + 1 < s_end; t += 2) {
            step(0, ra1, rb1);
            step(1, ra0, rb0);
        }
        if (t < s_end) step(0, ra1, rb1);
    }

    C += (int64_t)blockIdx.z * c_split_stride;
    bool bad = false;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        acc[b] += low[b];
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= non_finite(acc[b][e]);
        acc[b] *= SPLIT_UNSCALE;
    }
    if (__builtin_expect(__ballot(bad) != 0, 0)) {
        // an infinity or NaN among the operands, or a sum out of range: the sums of this slice with the fp32 instruction, from memory
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int k_end = min(s_end * 32, K);
        for (int k0 = s_beg * 32; k0 < k_end; k0 += 32) {
            float x[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = k0 + lk * 8 + 4 * h, t = min(k / c, 26), row = idx[t * ROWS + li];
                const float *src = X + (int64_t)max(row, 0) * c + k - t * c;
#pragma unroll
                for (int j = 0; j < 4; ++j) x[4 * h + j] = row >= 0 && k < K ? src[j] : 0.f;
            }
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int n = n0 + b * 16 + li;
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int k = k0 + lk * 8 + j;
                    t = mfma_f32(k < K && n < N ? W[(int64_t)k * N + n] : 0.f, x[j], t);
                }
                acc[b] += t;
            }
        }
    }
    if (row0 + li >= M) return;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        const int n = n0 + b * 16 + lk * 4;
        float *dst = C + (int64_t)(row0 + li) * N + n;
        if (vec_out && n + 4 <= N) *reinterpret_cast<f32x4 *>(dst) = acc[b];
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) dst[e] = acc[b][e];
    }
}

}  // namespace hch
