// Gathered product over general index rows (strided convolutions: forward through `field`, data
// gradient through `field_t`), out[i][n] = sum over the taps t and channels k of
// X[field[i][t]][k] * W(t, k, n), with fp32 operands on the bf16 matrix instruction: operands cut into three
// bf16 pieces as in split_wgrad.hip.hpp, six products per term.  Up to 32 taps.
#pragma once
#include "split_conv.hip.hpp"

namespace hch {

// The weights as the kernel below reads them: cut, 8 channels of one tap and one column to a piece of 16
// bytes, [tap][unit of 8 channels][16 columns][piece][column]; channels and columns past the end are zero.
// BT: W(t, k, n) = W[t][n][k], else W[t][k][n].  Cutting them where they are used would double the vector
// work of a product with 16 columns.
template <bool BT>
__global__ __launch_bounds__(256) void split_weights_kernel(const float *__restrict__ W, u32x4 *__restrict__ out, int taps, int c, int N)
{
    const int c8 = (c + 7) >> 3, n16 = (N + 15) >> 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)taps * c8 * n16 * 16) return;
    const int li = (int)(i & 15);
    const int64_t q = i >> 4, tu = q / n16;
    const int n = (int)(q - tu * n16) * 16 + li, t = (int)(tu / c8), k0 = (int)(tu - (int64_t)t * c8) * 8;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool ok = n < N && k0 + j < c;
        v[j] = ok ? W[BT ? ((int64_t)t * N + n) * c + k0 + j : ((int64_t)t * c + k0 + j) * N + n] : 0.f;
    }
    u32x4 p[3];
    split3(v, p[0], p[1], p[2]);
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) out[(q * 3 + pl) * 16 + li] = p[pl];
}

// A workgroup of 8 wavefronts takes 256 consecutive rows.  Rows of one stretch have few taps in common: of
// a stride S only those of one remainder per axis can have an owner.  So the workgroup first sorts its rows by
// their first tap, in LDS, and a wavefront multiplies 16 rows of that order at a time over the taps that those
// 16 have, in units of 8 channels of one tap, 4 units (32 terms) to an instruction, like conv_split_kernel but with
// a tap list of its own and without barriers.
// Bound by vector instructions (85 a step, 52 of them the cutting of the rows) with 16 columns, at 6 wavefronts per SIMD: the
// pipes issue 0.86 of the cycles, matrix pipes 0.11, LDS 0.29 (data gradient of 16 -> 32, 3^3, stride 2, 609 000 rows).  With
// more columns, at 4, by the waits of a step as well (weights from L2, rows, LDS): 0.63, 0.21 and 0.21 (its forward
// product).  Data gradient of 32 -> 16, 3^3, stride 2, 609 000 rows:
// 84 us, where the gradient of the column matrix and its gather took 208; forward 197 000 rows 32 -> 64 229 -> 175.  More
// requests ahead (rows two steps, weights one) at 4 wavefronts per SIMD were slower: 104 us and 188.
constexpr int FIELD_ROWS = 256, FIELD_WAVES = 8;
struct FieldLds {
    static constexpr int A = 16 * 128;                                    // one wavefront's rows of a step
    static constexpr int O_KEY = FIELD_WAVES * A, O_RANK = O_KEY + FIELD_ROWS * 4, O_ORDER = O_RANK + FIELD_ROWS * 4;
    static constexpr int O_MASK = O_ORDER + FIELD_ROWS * 4, O_TAP = O_MASK + FIELD_ROWS * 4, O_IDX = O_TAP + FIELD_WAVES * 32;
    static int bytes(int taps) { return O_IDX + FIELD_ROWS * (taps | 1) * 4; }
};

template <int NT, bool BT>
__global__ __launch_bounds__(64 * FIELD_WAVES, NT == 1 ? 6 : 4) void field_split_kernel(
    const float *__restrict__ X, const float *__restrict__ W, const u32x4 *__restrict__ Wp, float *__restrict__ C,
    const int32_t *__restrict__ field, int M, int N, int c, int taps, int64_t x_rows, unsigned n_tiles, int vec_out)
{
    typedef FieldLds L;
    constexpr int SRD3 = 0x00020000;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const unsigned tile = xcd_tile(blockIdx.x, gridDim.x / NUM_XCD);
    if (tile >= n_tiles) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = (int)tile * FIELD_ROWS, rows = min(FIELD_ROWS, M - row0), ts = taps | 1;
    unsigned char *a_lds = lds + wave * L::A;
    uint32_t *key = reinterpret_cast<uint32_t *>(lds + L::O_KEY), *mask = reinterpret_cast<uint32_t *>(lds + L::O_MASK);
    int32_t *rank = reinterpret_cast<int32_t *>(lds + L::O_RANK), *order = reinterpret_cast<int32_t *>(lds + L::O_ORDER);
    uint8_t *taplist = lds + L::O_TAP + wave * 32;
    int32_t *idx = reinterpret_cast<int32_t *>(lds + L::O_IDX);

    // index rows, then the order: number of rows with a smaller (first tap, row)
    const int32_t *src = field + (int64_t)row0 * taps;
    for (int e = tid; e < FIELD_ROWS * taps; e += 64 * FIELD_WAVES) {
        const int r = (int)((unsigned)e / (unsigned)taps);
        idx[r * ts + e - r * taps] = r < rows ? src[e] : -1;
    }
    __syncthreads();
    if (tid < FIELD_ROWS) {
        uint32_t m = 0;
#pragma unroll 9
        for (int t = 0; t < taps; ++t) m |= idx[tid * ts + t] >= 0 ? 1u << t : 0u;
        mask[tid] = m;
        key[tid] = (uint32_t)(m ? __builtin_ctz(m) : 32) << 16 | (uint32_t)tid;
        rank[tid] = 0;
    }
    __syncthreads();
    {
        const uint32_t mine = key[tid & (FIELD_ROWS - 1)];
        const u32x4 *k4 = reinterpret_cast<const u32x4 *>(key + tid / FIELD_ROWS * (FIELD_ROWS / 2));
        int before = 0;
#pragma unroll 8
        for (int q = 0; q < FIELD_ROWS / 8; ++q) {
            const u32x4 k = k4[q];
            before += (k[0] < mine) + (k[1] < mine) + (k[2] < mine) + (k[3] < mine);
        }
        atomicAdd(&rank[tid & (FIELD_ROWS - 1)], before);
    }
    __syncthreads();
    if (tid < FIELD_ROWS) order[rank[tid]] = tid;
    __syncthreads();

    const int n0 = (int)blockIdx.y * 16 * NT, n16 = (N + 15) >> 4, c8 = (c + 7) >> 3;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)(x_rows * c * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, taps * c8 * n16 * 768, SRD3);
    const int ap = lane & 7, ar = lane >> 3;           // gathered rows: piece ap (16 bytes) of rows ar and ar + 8
    const int d_tap = 4 / c8, d_u = 4 - d_tap * c8;
    for (int g = wave; g < FIELD_ROWS / 16; g += FIELD_WAVES) {
        const int my = order[g * 16 + li], r_a0 = order[g * 16 + ar], r_a1 = order[g * 16 + ar + 8];
        uint32_t present = mask[my];
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) present |= (uint32_t)__shfl_xor((int)present, d);
        present = (uint32_t)__builtin_amdgcn_readfirstlane((int)present);
        const int n_present = __popc(present);
        if (lane < 32) {
            if (lane >= n_present) taplist[lane] = 0;                      // past the last: multiplied with no weights
            if (present >> lane & 1u) taplist[__popc(present & ((1u << lane) - 1u))] = (uint8_t)lane;
        }
        __builtin_amdgcn_wave_barrier();
        const int n_units = n_present * c8, n_steps = (n_units + 3) >> 2;

        // list position and unit within the tap, of this lane's piece and of this lane's weights
        int a_tap = (ap >> 1) / c8, a_u = (ap >> 1) - a_tap * c8, b_tap = lk / c8, b_u = lk - b_tap * c8;
        auto fetch_rows = [&](u32x4 *ra) {
            const int tap = taplist[min(a_tap, 31)];
            const int ch = (a_u * 8 + (ap & 1) * 4) * 4;
            const int o0 = __mul24(idx[r_a0 * ts + tap], c * 4), o1 = __mul24(idx[r_a1 * ts + tap], c * 4);
            ra[0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, o0 < 0 ? o0 : o0 + ch, 0, 0));
            ra[1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, o1 < 0 ? o1 : o1 + ch, 0, 0));
            a_tap += d_tap; a_u += d_u;
            if (a_u >= c8) { a_u -= c8; ++a_tap; }
        };
        auto fetch_weights = [&](u32x4 (*w)[3]) {
            const int tap = taplist[min(b_tap, 31)];
            const int at = b_tap < n_present ? ((tap * c8 + b_u) * n16 * 48 + li) * 16 + n0 * 48 : (int)0x80000000u;
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int pl = 0; pl < 3; ++pl)
                    w[b][pl] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, at, n0 + 16 * b < N ? (b * 3 + pl) * 256 : 0, 0));
            b_tap += d_tap; b_u += d_u;
            if (b_u >= c8) { b_u -= c8; ++b_tap; }
        };

        f32x4 acc[NT], low[NT];
#pragma unroll
        for (int b = 0; b < NT; ++b) acc[b] = low[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        u32x4 ra[2];
        fetch_rows(ra);
        for (int s = 0; s < n_steps; ++s) {
            u32x4 w[NT][3];
            fetch_weights(w);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = ar + 8 * h;
                *reinterpret_cast<u32x4 *>(a_lds + r * 128 + ((ap ^ row_swap(r)) << 4)) = ra[h];
            }
            fetch_rows(ra);
            __builtin_amdgcn_wave_barrier();
            float f[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 raw = *reinterpret_cast<const u32x4 *>(a_lds + li * 128 + (((lk * 2 + h) ^ row_swap(li)) << 4));
#pragma unroll
                for (int e = 0; e < 4; ++e) f[4 * h + e] = __uint_as_float(raw[e]);
            }
            __builtin_amdgcn_wave_barrier();
            u32x4 x[3];
            split3(f, x[0], x[1], x[2]);
            constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
#pragma unroll
            for (int b = 0; b < NT; ++b) acc[b] = mfma_bf16(w[b][0], x[0], acc[b]);
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int b = 0; b < NT; ++b) low[b] = mfma_bf16(w[b][PB[t]], x[PA[t]], low[b]);
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
            // an infinity or NaN among the operands, or a sum out of range: the sums with the fp32 instruction, as in
            // conv_split_kernel
#pragma unroll
            for (int b = 0; b < NT; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int u = 0, cnt; u < n_units; u += cnt) {
                const int tap = taplist[u / c8], u_tap = u % c8, k0 = (u_tap + lk) * 8;
                cnt = min(min(4, c8 - u_tap), n_units - u);
                const int row = idx[my * ts + tap];
                const int have = lk < cnt ? c - k0 : 0;
                float x[8];
                load8(X + (int64_t)max(row, 0) * c + k0, row >= 0 ? have : 0, x);
#pragma unroll
                for (int b = 0; b < NT; ++b) {
                    const int col = n0 + b * 16 + li;
                    float v[8];
                    if constexpr (BT) load8(W + ((int64_t)tap * N + min(col, N - 1)) * c + k0, col < N ? have : 0, v);
                    else
#pragma unroll
                        for (int j = 0; j < 8; ++j) v[j] = j < have && col < N ? W[((int64_t)tap * c + k0 + j) * N + col] : 0.f;
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 8; ++j) t = mfma_f32(v[j], x[j], t);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][e] += row >= 0 ? t[e] : 0.f;
                }
            }
        }
        if (my < rows) {
#pragma unroll
            for (int b = 0; b < NT; ++b) {
                const int col = n0 + b * 16 + lk * 4;
                float *dst = C + (int64_t)(row0 + my) * N + col;
                if (vec_out && col + 4 <= N) *reinterpret_cast<f32x4 *>(dst) = acc[b];
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < N) dst[e] = acc[b][e];
            }
        }
    }
}

}  // namespace hch
