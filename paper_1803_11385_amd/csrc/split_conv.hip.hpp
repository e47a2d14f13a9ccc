// Gathered product of the 3x3x3 convolution (forward, data gradient), C[i][n] = sum over the taps t
// and channels k of X[nbr[i][t]][k] * W(t, k, n), with fp32 operands on the bf16 matrix instruction:
// both operands cut into three bf16 pieces as in split_wgrad.hip.hpp, six products per term.
#pragma once
#include "split_wgrad.hip.hpp"

namespace hch {

// the first `have` (none to all) of 8 consecutive numbers, zeros behind them
__device__ __forceinline__ void load8(const float *p, int have, float *v)
{
    if (have >= 8) __builtin_memcpy(v, p, 32);
    else
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = j < have ? p[j] : 0.f;
}

// A workgroup of WV wavefronts (4 or 8) computes 64 or 128 rows of the order `rowmap` by 16*NT columns; a
// wavefront has 16 rows of its own.  The reduction runs over the taps that the workgroup's rows have
// (`tilemask`), in units of 8 channels of one tap, 4 units (32 terms) to a step.
//   * Gathered rows: a wavefront loads its own rows, 8 lanes per 128 bytes of a row, lays them into a
//     stretch of LDS that nobody else reads (no barrier), reads them back as the operand wants them
//     (8 consecutive terms of one row per lane) and cuts them in registers.  Each element is cut
//     once per column tile of the output, which is why a wavefront takes all columns.
//   * Weights: the same share of every step for each thread, cut before it goes to LDS, two stages, one
//     barrier a step.
//   * Loads run two steps ahead in two sets of registers, as in gemm_f32_kernel.
//   * The index rows of a wavefront are read once, whole rows at a time, into LDS.
//   * The last rows of the order have the most neighbours; their workgroups start first, or a launch ends with
//     a few of them running alone (32 -> 64 at 280 000 voxels 141 -> 131 us).
// Bound by no single unit: at four wavefronts per SIMD the vector pipes issue 0.53 of all cycles, the matrix
// pipes are busy 0.32, LDS 0.5, fills of L1 run at 8.6 TB/s (64 -> 64, 280 000 voxels, 64 rows), and they
// stand in each other's way.  Products of a step issued between the splitting of the next one took more registers
// than that gave back (two wavefronts per SIMD: 196 -> 250 us), 32 rows per wavefront the same (203),
// 16 wavefronts share one barrier (202).  Eight wavefronts load and split the weights for twice the rows:
// 198 -> 187 us.  Forward and data gradient at 280 000 voxels, before (four wavefronts, rows in ascending
// order, conflicts on half of the LDS reads, half of the threads without weights where there are 32
// columns) -> now: 32 -> 64 120 and 140 us -> 107 and 117 (bench.py's shapes 137 and 158 -> 116 and 138), 64 -> 64 210 and 207
// -> 185 and 175, 50 -> 50 227 and 261 -> 184 and 183; gemm_f32_kernel over the coarser row order took 196 and 196, 354 and 365, 1112 and 1117.
// FAST: rows of a multiple of 32 channels; a step lies within one tap, offsets that change from step
// to step are scalar, and a wavefront whose own rows lack the tap sits the step out.  Otherwise any
// number of channels: a tap is padded to a multiple of 8, with weights of zero.
// BT: W(t, k, n) = W[26 - t][n][k] (the data gradient's view of the weights), else W[t][k][n].

// Where a 16-byte piece lies in LDS.  ds_read_b128 serves 16 lanes a clock, not 16 neighbours: lanes 0-3, 12-15 and
// 20-27 of each half, then the others.  With these permutations any 16 of them read 16 different
// sixteenths of the 256 bytes that the banks span (4 clocks a read; the plain layouts took 8), and the writes
// of 8 neighbouring lanes stay apart too.  Gathered rows: piece ^ row_swap(row); weights: column ^ unit_swap(unit).
__device__ __forceinline__ int row_swap(int r) { return (r >> 1 & 1) | (r >> 3 & 1) * 6; }
__device__ __forceinline__ int unit_swap(int k) { return (k & 1) * 2 + (k >> 1) * 12; }

template <int NT, int WV>
struct ConvLds {
    static constexpr int BN = 16 * NT, ROWS = 16;
    static constexpr int A = ROWS * 128;                                   // one wavefront's rows of a step
    static constexpr int LKS = BN * 16, PLANE = 4 * LKS, B = 3 * PLANE;   // one stage of weights
    static constexpr int IDX = 27 * ROWS * 4;                              // one wavefront's index rows, tap-major
    static constexpr int O_B = WV * A, O_IDX = O_B + 2 * B, O_TAP = O_IDX + WV * IDX, BYTES = O_TAP + 32;
};

template <int NT, int WV, bool FAST, bool BT>
__global__ __launch_bounds__(64 * WV) void conv_split_kernel(
    const float *__restrict__ X, const float *__restrict__ W, float *__restrict__ C, const int32_t *__restrict__ nbr,
    const int32_t *__restrict__ rowmap, const uint32_t *__restrict__ tilemask,
    int M, int N, int c, unsigned m_tiles, int64_t c_split_stride, int vec_out)
{
    typedef ConvLds<NT, WV> L;
    constexpr int BN = L::BN, ROWS = L::ROWS, GROUP = ROWS * WV / 64;     // 64-row tiles per workgroup
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
    const int row0 = ((int)mtile * WV + wave) * ROWS;                   // this wavefront's first row of the order
    unsigned char *a_lds = lds + wave * L::A;
    int32_t *idx = reinterpret_cast<int32_t *>(lds + L::O_IDX + wave * L::IDX);
    uint8_t *taplist = lds + L::O_TAP;

    // taps of the workgroup's rows, the list of them, and this slice's steps
    uint32_t present = tilemask[mtile * GROUP];
    if (GROUP == 2 && mtile * 2 + 1 < m_tiles) present |= tilemask[mtile * 2 + 1];
    present = (uint32_t)__builtin_amdgcn_readfirstlane((int)present);
    if (tid < 32) {
        if (tid >= __popc(present)) taplist[tid] = 0;                      // past the last: tap 0, with no weights
        if (present >> tid & 1u) taplist[__popc(present & ((1u << tid) - 1u))] = (uint8_t)tid;
    }
    const int c8 = (c + 7) >> 3;
    const int n_units = __popc(present) * c8, n_steps = (n_units + 3) >> 2;
    const int per = (n_steps + (int)gridDim.z - 1) / (int)gridDim.z;
    const int s_beg = min((int)blockIdx.z * per, n_steps), s_end = min(s_beg + per, n_steps);

    // index rows of the wavefront's rows, tap-major in LDS; the centre tap is the row's own voxel
    uint32_t mine = 0;                                                     // taps of this wavefront's rows
    {
        const int r = lane < ROWS ? lane : 0;
        const bool ok = lane < ROWS && row0 + r < M;
        const int vox = ok ? rowmap[row0 + r] : -1;
        if (lane < ROWS) idx[13 * ROWS + lane] = vox;
        __builtin_amdgcn_wave_barrier();
        const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, M * 27 * 4, SRD3);
        int32_t v[(ROWS * 27 + 63) / 64];
#pragma unroll
        for (int q = 0; q < (ROWS * 27 + 63) / 64; ++q) {
            const int e = q * 64 + lane, rr = min(e / 27, ROWS - 1), t = e - (e / 27) * 27;
            const int vx = idx[13 * ROWS + rr];
            v[q] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_n, vx >= 0 ? (vx * 27 + t) * 4 : (int)OUT, 0, 0);
            if (vx < 0 || e >= ROWS * 27) v[q] = -1;
            if (FAST) mine |= v[q] >= 0 ? 1u << t : 0u;
        }
#pragma unroll
        for (int q = 0; q < (ROWS * 27 + 63) / 64; ++q) {
            const int e = q * 64 + lane, rr = e / 27, t = e - rr * 27;
            if (rr < ROWS && t != 13) idx[t * ROWS + rr] = v[q];
        }
        if (FAST) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) mine |= (uint32_t)__shfl_xor((int)mine, d);
            mine = (uint32_t)__builtin_amdgcn_readfirstlane((int)mine);
        }
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)((int64_t)M * c * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, 27 * c * N * 4, SRD3);

    // ---- one step's loads.  Gathered rows: piece ap (16 bytes) of rows ar, ar + 8, ...
    const int ap = lane & 7, ar = lane >> 3;
    constexpr int AU = ROWS / 8;
    // weights: UN consecutive terms of one column per thread
    constexpr int UN = BN * 32 / (64 * WV), KP = 32 / UN;
    static_assert(UN >= 2 && UN <= 8, "whole pairs, within one unit");
    const int bn = BT ? tid / KP : tid % BN, kp = BT ? tid % KP : tid / BN;
    const int bk = kp * UN / 8, bs = kp * UN % 8;                           // unit, first term within it
    const bool b_col = n0 + bn < N;
    // FAST: list position and channel block of the next step (scalar)
    uint32_t rem = present;
    int cb = 0;
    // otherwise: list position and unit within the tap, of this lane's piece and of this thread's weights
    int a_tap = 0, a_u = 0, b_tap = 0, b_u = 0;
    const int d_tap = 4 / c8, d_u = 4 - d_tap * c8;
    if constexpr (FAST) {
        const int per_tap = c >> 5, skip = s_beg / per_tap;
        for (int q = 0; q < skip; ++q) rem &= rem - 1u;
        cb = (s_beg - skip * per_tap) * 32;
    } else {
        const int ua = s_beg * 4 + (ap >> 1), ub = s_beg * 4 + bk;
        a_tap = ua / c8; a_u = ua - a_tap * c8;
        b_tap = ub / c8; b_u = ub - b_tap * c8;
    }
    const int n_present = __popc(present);
    auto fetch = [&](u32x4 *ra, float *rb) {
        if constexpr (FAST) {
            const int tap = rem ? __builtin_ctz(rem) : 0;                  // past the end: any tap, never multiplied
#pragma unroll
            for (int q = 0; q < AU; ++q) {
                const int off = __mul24(idx[tap * ROWS + ar + 8 * q], c * 4) + ap * 16;
                ra[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off, __builtin_amdgcn_readfirstlane(cb * 4), 0));
            }
            if constexpr (BT) {
                const int base = __builtin_amdgcn_readfirstlane(((26 - tap) * N * c + cb) * 4);
                const int off = b_col ? ((n0 + bn) * c + kp * UN) * 4 : (int)OUT;
                if constexpr (UN >= 4) {
#pragma unroll
                    for (int h = 0; h < UN / 4; ++h) {
                        const f32x4 w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, off + 16 * h, base, 0));
#pragma unroll
                        for (int j = 0; j < 4; ++j) rb[4 * h + j] = w[j];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < UN; ++j) rb[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, off + 4 * j, base, 0));
                }
            } else {
                const int off = b_col ? (kp * UN * N + n0 + bn) * 4 : (int)OUT;
#pragma unroll
                for (int j = 0; j < UN; ++j)
                    rb[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, off, __builtin_amdgcn_readfirstlane((tap * c + cb + j) * N * 4), 0));
            }
            cb += 32;
            if (cb >= c) { cb = 0; rem &= rem - 1u; }
        } else {
            // a tap past the list's end has no weights; channels past the row's end (the next row's
            // numbers) meet weights of zero -- and if they are not finite, the plain sums are taken
            const int tap = taplist[min(a_tap, 31)];
#pragma unroll
            for (int q = 0; q < AU; ++q) {
                const int off = __mul24(idx[tap * ROWS + ar + 8 * q], c * 4);
                const int ch = (a_u * 8 + (ap & 1) * 4) * 4;
                ra[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, off < 0 ? off : off + ch, 0, 0));
            }
            a_tap += d_tap; a_u += d_u;
            if (a_u >= c8) { a_u -= c8; ++a_tap; }
            const int tb = taplist[min(b_tap, 31)];
            const bool ok = b_col && b_tap < n_present;
#pragma unroll
            for (int j = 0; j < UN; ++j) {
                const int k = b_u * 8 + bs + j;
                const int at = BT ? ((26 - tb) * N + n0 + bn) * c + k : (tb * c + k) * N + n0 + bn;
                rb[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, ok && k < c ? at * 4 : (int)OUT, 0, 0));
            }
            b_tap += d_tap; b_u += d_u;
            if (b_u >= c8) { b_u -= c8; ++b_tap; }
        }
    };
    auto stash_a = [&](const u32x4 *ra) {
#pragma unroll
        for (int q = 0; q < AU; ++q) {
            const int r = ar + 8 * q;
            *reinterpret_cast<u32x4 *>(a_lds + r * 128 + ((ap ^ row_swap(r)) << 4)) = ra[q];
        }
    };
    auto stash_b = [&](int stage, const float *rb) {
        unsigned char *dst = lds + L::O_B + stage * L::B + bk * L::LKS + (bn ^ unit_swap(bk)) * 16 + bs * 2;
        uint32_t p[3][UN / 2];
        split3n<UN / 2>(rb, p[0], p[1], p[2]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) __builtin_memcpy(__builtin_assume_aligned(dst + pl * L::PLANE, UN * 2), p[pl], UN * 2);
    };

    // the products of the leading pieces and the five smaller ones are summed apart: the large sums
    // are rounded by one instruction per 32 terms instead of six.  (Sums of one sign over very many terms lean
    // downwards, 4.6e-8 of the result with 27 taps of 512 channels and 3.5e-7 with 2048, where
    // v_mfma_f32_16x16x4_f32 leans by 7.0e-8 and 9.4e-7; sums of either sign by 2e-9 and less.)
    f32x4 acc[NT], low[NT];
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // FAST: the step being multiplied
    uint32_t rem_m = rem;
    int cb_m = cb;
    auto step = [&](int stage, u32x4 *ra, float *rb) {
        u32x4 raw[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            raw[h] = *reinterpret_cast<const u32x4 *>(a_lds + li * 128 + (((lk * 2 + h) ^ row_swap(li)) << 4));
        stash_a(ra);                                                       // step t + 1, after the reads of step t
        stash_b(stage ^ 1, rb);
        fetch(ra, rb);                                                     // step t + 3
        bool run = true;
        if constexpr (FAST) {
            run = (mine >> (rem_m ? __builtin_ctz(rem_m) : 0)) & 1u;
            cb_m += 32;
            if (cb_m >= c) { cb_m = 0; rem_m &= rem_m - 1u; }
        }
        if (run) {
            // the operands change places: a lane ends up with 4 neighbouring columns of one row
            float f[8];
            u32x4 x[3];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = __uint_as_float(raw[j >> 2][j & 3]);
            split3(f, x[0], x[1], x[2]);
            u32x4 w[NT][3];
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
        }
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
    const int vox = idx[13 * ROWS + li];
    if (__builtin_expect(__ballot(bad) != 0, 0)) {
        // An infinity or NaN among the operands, or a sum out of range: the sums of this slice with the
        // fp32 instruction, up to 32 channels of one tap at a time, added only where the row has the tap
        // (an absent row is not zero times an infinity).  From memory, without LDS or barriers.  Every number
        // a NaN, 32 -> 64 at 40 000 voxels: 110 us, 2.0 ms with the outputs summed one after the other; at
        // 280 000 voxels forward 365 us and data gradient 392, 139 and 150 with finite numbers.
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int u_end = min(s_end * 4, n_units);
        for (int u = s_beg * 4, cnt; u < u_end; u += cnt) {
            const int tap = taplist[u / c8], u_tap = u % c8, k0 = (u_tap + lk) * 8;
            cnt = min(min(4, c8 - u_tap), u_end - u);
            const int row = idx[tap * ROWS + li];
            if (__ballot(row >= 0) == 0) continue;
            const int have = lk < cnt ? c - k0 : 0;
            float x[8];
            load8(X + (int64_t)max(row, 0) * c + k0, row >= 0 ? have : 0, x);
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int col = n0 + b * 16 + li;
                float w[8];
                if constexpr (BT) load8(W + ((int64_t)(26 - tap) * N + min(col, N - 1)) * c + k0, col < N ? have : 0, w);
                else
#pragma unroll
                    for (int j = 0; j < 8; ++j) w[j] = j < have && col < N ? W[((int64_t)tap * c + k0 + j) * N + col] : 0.f;
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 8; ++j) t = mfma_f32(w[j], x[j], t);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[b][e] += row >= 0 ? t[e] : 0.f;
            }
        }
    }
    if (vox < 0) return;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        const int col = n0 + b * 16 + lk * 4;
        float *dst = C + (int64_t)vox * N + col;
        if (vec_out && col + 4 <= N) *reinterpret_cast<f32x4 *>(dst) = acc[b];
        else
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < N) dst[e] = acc[b][e];
    }
}

}  // namespace hch
