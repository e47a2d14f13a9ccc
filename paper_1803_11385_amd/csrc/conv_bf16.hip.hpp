// Gathered product of the 3x3x3 convolution with bf16 operands (forward, data gradient) over the row order:
// C[i][n] = sum over the taps t and channels k of X[nbr[i][t]][k] * W(t, k, n).
#pragma once
#include "split_conv.hip.hpp"

namespace hch {

// A workgroup of 4 or 8 wavefronts computes 128 or 256 rows of the order `rowmap` by 16*NT columns, a wavefront 32 of them; a
// step is KS channels of one tap that the workgroup's rows have, and a wavefront whose own rows lack the tap sits it
// out.  Rows pass through LDS of the wavefront's own, weights through two shared stages, loads run two steps
// ahead in two sets of registers, as in conv_split_kernel; nothing is cut here.
// BT: W(t, k, n) = W[26 - t][n][k] (the data gradient's view of the weights), else W[t][k][n].
// NT == 2: sums of 128 terms, added up, instead of one chain of them all, in registers that four workgroups to a CU leave free (tiles of 64
// columns have none): 64 -> 32 at 127 000 rows 1.41e-7 -> 0.75e-7 from the exact sums, 31 and 31 us, 32 -> 16 1.0e-7 -> 0.66e-7, 20.3 and 21.0.
// FULL: rows of a multiple of KS channels, 16-byte aligned.
// 128 rows, four workgroups to a CU, against 256: 32 -> 64 at 127 000 rows 32 -> 29 and 34 -> 30 us (data gradient), at 609 000 105 -> 96 and 103 -> 95,
// at 32 000 22 -> 16 and 22 -> 16; 64 -> 64, with 64 channels a step three to a CU, at 127 000 44 -> 46 and 41 -> 41, at 280 000 68 -> 71 and 63 -> 63.
// Bound, with 256 rows, by waits of the two workgroups per CU, 0.45 of a wavefront's life, on LDS first: it is busy 0.57 of the time (data
// gradient 0.55), 0.40 (0.33) of that with bank conflicts; matrix pipes 0.18 (0.19), vector pipes 0.21, 64 -> 64 at 280 000
// rows.
// Against gemm_bf16_kernel, which multiplies every tap of every row and transposes the weights in a launch of its own or on the
// way: 64 -> 64 at 280 000 rows 102 -> 73 us and 97 -> 67 (data gradient), at 609 000 205 -> 145 and 193 -> 133.  The same
// kernel over the rows as they come: 113 and 101, 215 and 192.
template <int NT, int KS, int WAVES>
struct ConvBf16Lds {
    static constexpr int BN = 16 * NT, ROWS = 32, WV = WAVES, PIECES = KS / 8;    // 16-byte pieces of a row of a step
    static constexpr int A = ROWS * KS * 2, LKS = BN * 16, B = PIECES * LKS, IDX = 27 * ROWS * 4;
    static constexpr int O_B = WV * A, O_IDX = O_B + 2 * B, BYTES = O_IDX + WV * IDX;
    // where piece p of row r lies, and column n of piece p of the weights: see row_swap and unit_swap
    static __device__ __forceinline__ int a_at(int r, int p)
    {
        const int q = r >> 2 & 3, swap = KS == 64 ? (r >> 1 & 7) : ((q ^ q >> 1) & 1) * 2 + (q >> 1);
        return (r * PIECES + (p ^ swap)) * 16;
    }
    static __device__ __forceinline__ int b_at(int p, int n) { return p * LKS + (n ^ ((p & 7) * 2)) * 16; }
};

template <int NT, int KS, int WAVES, bool FULL, bool BT>
__device__ __forceinline__ void conv_bf16_rows(
    const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr,
    const int32_t *__restrict__ rowmap, const uint32_t *__restrict__ tilemask, int M, int N, int c, unsigned m_tiles, int vec_out)
{
    typedef ConvBf16Lds<NT, KS, WAVES> L;
    constexpr int BN = L::BN, ROWS = L::ROWS, WV = L::WV, P = L::PIECES, GROUP = ROWS * WV / 64;
    constexpr uint32_t OUT = 0x80000000u;
    constexpr int SRD3 = 0x00020000;
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::BYTES];

    unsigned mtile = xcd_chunk_tile(blockIdx.x, skip_chunk(m_tiles, GROUP));
    const unsigned groups = (m_tiles + GROUP - 1) / GROUP;
    if (mtile >= groups) return;
    mtile = groups - 1 - mtile;                                           // most neighbours first
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = (int)blockIdx.y * BN;
    const int row0 = ((int)mtile * WV + wave) * ROWS;
    unsigned char *a_lds = lds + wave * L::A;
    int32_t *idx = reinterpret_cast<int32_t *>(lds + L::O_IDX + wave * L::IDX);

    uint32_t present = 0;
#pragma unroll
    for (int q = 0; q < GROUP; ++q)
        if (mtile * GROUP + q < m_tiles) present |= tilemask[mtile * GROUP + q];
    present = (uint32_t)__builtin_amdgcn_readfirstlane((int)present);
    const int per_tap = FULL ? c / KS : (c + KS - 1) / KS, n_steps = __popc(present) * per_tap;

    // index rows of the wavefront's rows, tap-major in LDS; the centre tap is the row's own voxel
    uint32_t mine = 0;
    {
        const bool ok = lane < ROWS && row0 + lane < M;
        const int vox = ok ? rowmap[row0 + lane] : -1;
        if (lane < ROWS) idx[13 * ROWS + lane] = vox;
        __builtin_amdgcn_wave_barrier();
        const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, M * 27 * 4, SRD3);
        constexpr int Q = (ROWS * 27 + 63) / 64;
        int32_t v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int e = q * 64 + lane, rr = min(e / 27, ROWS - 1), t = e - (e / 27) * 27;
            const int vx = idx[13 * ROWS + rr];
            v[q] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_n, vx >= 0 ? (vx * 27 + t) * 4 : (int)OUT, 0, 0);
            if (vx < 0 || e >= ROWS * 27) v[q] = -1;
            mine |= v[q] >= 0 ? 1u << t : 0u;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int e = q * 64 + lane, rr = e / 27, t = e - rr * 27;
            if (rr < ROWS && t != 13) idx[t * ROWS + rr] = v[q];
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mine |= (uint32_t)__shfl_xor((int)mine, d);
        mine = (uint32_t)__builtin_amdgcn_readfirstlane((int)mine);
    }
    __builtin_amdgcn_wave_barrier();

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)((int64_t)M * c * 2), SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, 27 * c * N * 2, SRD3);

    // gathered rows: piece ap of rows ar, ar + 64 / P, ...
    const int ap = lane % P, ar = lane / P;
    constexpr int AU = ROWS * P / 64;
    // weights: BT: piece bp of column bn; else 4 channels, from bk, of columns bn and bn + 1
    constexpr int B_TASKS = BT ? BN * P : BN / 2 * (KS / 4);
    constexpr int BQ = (B_TASKS + 64 * WV - 1) / (64 * WV);                // for a thread
    const bool b_mine = B_TASKS >= 64 * WV || tid < B_TASKS;
    static_assert(B_TASKS % (64 * WV) == 0 || BQ == 1, "whole rounds");
    int bn[BQ], bk[BQ], b_off[BQ];
#pragma unroll
    for (int q = 0; q < BQ; ++q) {
        const int e = tid + q * 64 * WV;
        bn[q] = BT ? e / P : e % (BN / 2) * 2;
        bk[q] = BT ? e % P * 8 : e / (BN / 2) * 4;
        b_off[q] = b_mine && n0 + bn[q] < N ? (BT ? ((n0 + bn[q]) * c + bk[q]) * 2 : (bk[q] * N + n0 + bn[q]) * 2) : (int)OUT;
    }
    uint32_t rem = present;
    int cb = 0;
    auto fetch = [&](u32x4 *ra, u32x4 *rb) {
        const int tap = rem ? __builtin_ctz(rem) : 0;                      // past the end: any tap, never multiplied
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            const int off = __mul24(idx[tap * ROWS + ar + 64 / P * q], c * 2) + ap * 16;
            ra[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off, __builtin_amdgcn_readfirstlane(cb * 2), 0));
        }
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            if constexpr (BT) {
                rb[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, b_off[q], __builtin_amdgcn_readfirstlane(((26 - tap) * N * c + cb) * 2), 0));
            } else {
                // (a scalar offset past the end of the weights would let any per-lane offset in, so of a tap's last step in part the rows are
                // counted per lane)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if constexpr (FULL) rb[q][j] = __builtin_amdgcn_raw_buffer_load_b32(rs_w, b_off[q], __builtin_amdgcn_readfirstlane((tap * c + cb + j) * N * 2), 0);
                    else rb[q][j] = __builtin_amdgcn_raw_buffer_load_b32(rs_w, b_off[q] + j * N * 2, __builtin_amdgcn_readfirstlane((tap * c + cb) * N * 2), 0);
                }
            }
        }
        cb += KS;
        if (cb >= c) { cb = 0; rem &= rem - 1u; }
    };
    auto stash_a = [&](const u32x4 *ra) {
#pragma unroll
        for (int q = 0; q < AU; ++q) *reinterpret_cast<u32x4 *>(a_lds + L::a_at(ar + 64 / P * q, ap)) = ra[q];
    };
    auto stash_b = [&](int stage, const u32x4 *r) {
        unsigned char *dst = lds + L::O_B + stage * L::B;
        if (!b_mine) return;
#pragma unroll
        for (int q = 0; q < BQ; ++q) {
            const u32x4 &rb = r[q];
            if constexpr (BT) *reinterpret_cast<u32x4 *>(dst + L::b_at(bk[q] >> 3, bn[q])) = rb;
            else {
                *reinterpret_cast<u32x2 *>(dst + L::b_at(bk[q] >> 3, bn[q]) + (bk[q] & 4) * 2) = u32x2{pack_lo(rb[0], rb[1]), pack_lo(rb[2], rb[3])};
                *reinterpret_cast<u32x2 *>(dst + L::b_at(bk[q] >> 3, bn[q] + 1) + (bk[q] & 4) * 2) = u32x2{pack_hi(rb[0], rb[1]), pack_hi(rb[2], rb[3])};
            }
        }
    };

    // NT == 2: sums of 128 terms at a time, added up
    f32x4 acc[2][NT];
    [[maybe_unused]] f32x4 total[2][NT];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (NT == 2) total[a][b] = acc[a][b];
        }
    auto add_up = [&]() {
        if constexpr (NT == 2)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    total[a][b] += acc[a][b];
                    acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
    };
    uint32_t rem_m = rem;                                                  // the step being multiplied
    int cb_m = 0;
    auto step = [&](int stage, u32x4 *ra, u32x4 *rb) {
        u32x4 x[2][KS / 32];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int k = 0; k < KS / 32; ++k) x[a][k] = *reinterpret_cast<const u32x4 *>(a_lds + L::a_at(a * 16 + li, k * 4 + lk));
        stash_a(ra);                                                       // step t + 1, after the reads of step t
        stash_b(stage ^ 1, rb);
        fetch(ra, rb);                                                     // step t + 3
        const bool run = (mine >> (rem_m ? __builtin_ctz(rem_m) : 0)) & 1u;
        [[maybe_unused]] const int left = (c - cb_m - lk * 8) >> 1;         // pairs of channels that the lane's 8 have
        [[maybe_unused]] const bool whole = cb_m + KS <= c;
        cb_m += KS;
        if (cb_m >= c) { cb_m = 0; rem_m &= rem_m - 1u; }
        if (run) {
            // channels past the end, the next row's or the next tap's numbers, out of both operands (nothing may come of them, were they
            // infinite)
            auto cut = [&](u32x4 &v) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = j < left ? v[j] : 0u;
            };
            if constexpr (!FULL) {
                static_assert(FULL || KS == 32, "one piece per lane");
                if (!whole) { cut(x[0][0]); cut(x[1][0]); }
            }
            // the operands change places: a lane ends up with 4 neighbouring columns of one row
#pragma unroll
            for (int k = 0; k < KS / 32; ++k) {
                u32x4 w[NT];
#pragma unroll
                for (int b = 0; b < NT; ++b) w[b] = *reinterpret_cast<const u32x4 *>(lds + L::O_B + stage * L::B + L::b_at(k * 4 + lk, b * 16 + li));
                if constexpr (!FULL)
                    if (!whole)
#pragma unroll
                        for (int b = 0; b < NT; ++b) cut(w[b]);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < NT; ++b) acc[a][b] = mfma_bf16(w[b], x[a][k], acc[a][b]);
            }
        }
        __syncthreads();
    };
    if (n_steps > 0) {
        u32x4 ra0[AU], ra1[AU], rb0[BQ], rb1[BQ];
        fetch(ra0, rb0);
        fetch(ra1, rb1);
        stash_a(ra0);
        stash_b(0, rb0);
        fetch(ra0, rb0);
        __syncthreads();
        int t = 0;
        for (; t + 1 < n_steps; t += 2) {
            step(0, ra1, rb1);
            step(1, ra0, rb0);
            if (KS == 64 || (t & 2)) add_up();
        }
        if (t < n_steps) step(0, ra1, rb1);
    }
    if constexpr (NT == 2) {
        add_up();
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b) acc[a][b] = total[a][b];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int vox = idx[13 * ROWS + a * 16 + li];
        if (vox < 0) continue;
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int col = n0 + b * 16 + lk * 4;
            float *dst = C + (int64_t)vox * N + col;
            if (vec_out && col + 4 <= N) *reinterpret_cast<f32x4 *>(dst) = acc[a][b];
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < N) dst[e] = acc[a][b][e];
        }
    }
}

template <int NT, int KS, int WAVES, bool BT>
__global__ __launch_bounds__(64 * WAVES, NT == 4 && KS == 64 && WAVES == 4 ? 3 : 4) void conv_bf16_kernel(
    const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr,
    const int32_t *__restrict__ rowmap, const uint32_t *__restrict__ tilemask, int M, int N, int c, unsigned m_tiles, int vec_out)
{
    conv_bf16_rows<NT, KS, WAVES, true, BT>(X, W, C, nbr, rowmap, tilemask, M, N, c, m_tiles, vec_out);
}

// Rows of any even number of channels, 4-byte aligned: steps of 32 channels, the last of a tap in part.  50 -> 50 at 127 000 rows 606 us, with
// the fp32 instruction, -> 51, 12 -> 20 at 280 000 73 -> 37, 24 -> 40 (gemm_bf16_kernel) 59 -> 45.
template <int NT, bool BT>
__global__ __launch_bounds__(256, 4) void conv_ragged_bf16_kernel(
    const uint16_t *__restrict__ X, const uint16_t *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr,
    const int32_t *__restrict__ rowmap, const uint32_t *__restrict__ tilemask, int M, int N, int c, unsigned m_tiles, int vec_out)
{
    conv_bf16_rows<NT, 32, 4, false, BT>(X, W, C, nbr, rowmap, tilemask, M, N, c, m_tiles, vec_out);
}

}  // namespace hch
