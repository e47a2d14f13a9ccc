// Weight gradient of a gathered convolution (Eq.7), dW[tap*c + ch][n] = sum over the voxels i of
// X[nbr[i][tap]][ch] * dY[i][n], with fp32 operands on the bf16 matrix instruction.
//
// An fp32 number is the exact sum of three bf16 numbers, each the rest of it rounded to 8 bits, a
// product of two therefore the sum of nine bf16 products; the six largest are computed, each exact,
// summed in fp32 by v_mfma_f32_16x16x32_bf16.  The second piece is at most 2^-8 of the number and the
// third 2^-17, of either sign, so what is left out is at most 2^-24 of the product (on random
// numbers 2^-27.4 in the mean square, without a preferred sign; pieces that are cut off instead lose up to 2^-21,
// always towards zero).  Six of those take 96 cycles for what takes v_mfma_f32_16x16x4_f32 256, and
// they round once per 8 terms instead of once per 4.
#pragma once
#include "gemm_bf16.hip.hpp"

namespace hch {

// two fp32 numbers rounded to the nearest bf16, the first in the lower half
__device__ __forceinline__ uint32_t round_bf16(float a, float b)
{
    typedef float f32x2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2v));
}

// The operands are scaled before they are split, sums of products of two of them scaled back: bf16 ends at
// 2^-133, so without it the third and then the second piece of numbers below 2^-110 would be lost
// (relative error of a product 2.7e-5 at 1e-36, 0.26 at 1e-40).  2^16 brings the last bit of the
// smallest fp32 number, 2^-149, to 2^-133.  At the other end sums beyond 2^96 become infinite and are
// taken plainly.  One multiplication per number: 32 -> 64 at 280 000 voxels, forward 136 -> 142 us, data
// gradient 144 -> 151, weight gradient 141 -> 144.
constexpr float SPLIT_SCALE = 0x1p16f, SPLIT_UNSCALE = 0x1p-32f;

// SPLIT_SCALE * x[0..7] = h + m + l, as three MFMA operands of 8 bf16 each.  Both differences are exact.  An
// infinity, a NaN or a number that goes beyond the largest bf16 makes m a NaN, so that whatever it is
// multiplied into comes out non-finite (the caller then takes the plain fp32 sum).
// (v_dot2_f32_bf16 with (-1, 0) would subtract straight from the packed pair, but its sum is not exact.)
template <int PAIRS, typename V>
__device__ __forceinline__ void split3n(const float *x, V &h, V &m, V &l)
{
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        const float a = x[2 * p] * SPLIT_SCALE, b = x[2 * p + 1] * SPLIT_SCALE;
        h[p] = round_bf16(a, b);
        const float ra = a - __uint_as_float(h[p] << 16), rb = b - __uint_as_float(h[p] & 0xFFFF0000u);
        m[p] = round_bf16(ra, rb);
        l[p] = round_bf16(ra - __uint_as_float(m[p] << 16), rb - __uint_as_float(m[p] & 0xFFFF0000u));
    }
}
__device__ __forceinline__ void split3(const float *x, u32x4 &h, u32x4 &m, u32x4 &l) { split3n<4>(x, h, m, l); }

__device__ __forceinline__ f32x4 mfma_bf16(const u32x4 &a, const u32x4 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// c[nt] += a * b[nt] for split operands, or c[nt] -= a * b[nt] (MINUS).  The leading products of the 32
// terms are summed by themselves and so are the five smaller ones, so that both sums are rounded once
// when they meet and the long sum in c once per 32 terms (a single product ends up as close as
// the fp32 instruction's: 2.5e-8 in the mean square, 3.4e-8 with the leading products added to the smaller
// ones by the instruction, which rounds less well there; 250 against 260 us, 64 -> 64 at 280 000
// voxels).  Consecutive instructions belong to different sums, so that none waits for the one before
// it.  The instruction rounds to the nearest where the sum exceeds the products, but drops the lowest bits
// of products downwards where they exceed the sum: the caller negates b and takes MINUS for every other
// stretch of 32 terms, so that this cancels (without it results are 1.5e-8 of their rms too low at
// a million voxels, with it 4e-10).
template <int NT, bool MINUS>
__device__ __forceinline__ void mfma_split(const u32x4 *a, const u32x4 (*b)[3], f32x4 *c)
{
    constexpr int PA[5] = {2, 0, 1, 1, 0}, PB[5] = {0, 2, 1, 0, 1};
    f32x4 t[NT], low[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) low[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 5; ++q)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) low[nt] = mfma_bf16(a[PA[q]], b[nt][PB[q]], low[nt]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) t[nt] = mfma_bf16(a[0], b[nt][0], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) c[nt] = MINUS ? c[nt] - (t[nt] + low[nt]) : c[nt] + (t[nt] + low[nt]);
}

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool non_finite(float v) { return (__float_as_uint(v) & 0x7F800000u) == 0x7F800000u; }

// A workgroup of 8 wavefronts computes 28 units of 16 rows of dW by 16*NT columns over the blocks of
// 128 voxels slice, slice + slices, ... of the pattern order (`order`; null: data order), so that
// every slice gets its share of the dense patterns.  Per block
//   * the rows of dY are split once and laid into LDS as the instruction reads them; the index rows
//     are laid beside them as byte offsets into X, with a bit set of the taps that each 32 voxels have;
//   * a wavefront takes its 7 units (one in four) over half of the block.  The 16 lanes of a group
//     load 16 consecutive channels of one row of X, 64 bytes, straight into the operand's layout (8
//     voxels per lane): a gathered row passes neither LDS nor a transpose.  A unit none of whose
//     taps occurs in the 32 voxels is left out: the zeros it would add are most of the work
//     (0.43 to 0.75 of the (32 voxels, tap) pairs are left at the levels of a 256^3 batch).
// The rows of the next unit are requested before a unit is multiplied, across blocks as well; the
// index rows run two blocks ahead, dY one.  The two halves of a block are added through LDS at the
// end, which halves the partial sums that go to memory.
// Bound by the wait for what a block needs next, at two wavefronts per SIMD (197 to 256 registers): of a busy
// CU's time the vector pipes work 0.49, the matrix pipes 0.26, LDS 0.17.  Against gemm_f32_kernel, which
// multiplies every tap: 32 -> 64 at 280 000 voxels 142 us (260), 64 -> 64 266 (540), 50 -> 50 288 (894).
// A form with the units in a loop and a switch over their sums copied the sums through other registers
// (1.7 times as long); requests further ahead than two units changed nothing.
constexpr int WG_VOX = 128, WG_UNITS = 28, WG_SLOTS = WG_UNITS + 1, WG_RS = WG_VOX + 4;
template <int NT>
struct WgradLds {
    static constexpr int BN = 16 * NT;
    static constexpr int DY = WG_VOX / 32 * 3 * 4 * BN * 16;              // bytes of one stage of dY
    static constexpr int IDX = WG_SLOTS * WG_RS * 4;                       // ... of one block's offsets
    static constexpr int O_IDX = 2 * DY, O_ORD = O_IDX + 3 * IDX, O_MASK = O_ORD + 3 * WG_VOX * 4;
    static constexpr int O_TAB = O_MASK + 3 * 8 * 4, TOTAL = O_TAB + WG_UNITS * 16 * 4;
    static constexpr int HALF = 4 * 7 * NT * 4 * 64 * 4;                   // the second half's sums
    static constexpr int BYTES = TOTAL > HALF ? TOTAL : HALF;
};

template <int NT, bool C16>
__global__ __launch_bounds__(512) void wgrad_split_kernel(
    const float *__restrict__ X, const float *__restrict__ dY, float *__restrict__ C,
    const int32_t *__restrict__ nbr, const int32_t *__restrict__ order, int M, int N, int n, int64_t x_rows, int c, int taps,
    int slices, int m_tiles, int n_tiles, int64_t c_split_stride)
{
    typedef WgradLds<NT> L;
    constexpr int BN = L::BN;
    constexpr int D = NT == 2 ? 7 : 2;                                     // units whose rows are on their way (divides 14)
    constexpr uint32_t OUT = 0x80000000u;                                  // a byte offset outside every buffer
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::BYTES];

    // all tiles of a slice on one XCD where the slices divide evenly (they read the same rows)
    const unsigned tiles = (unsigned)(m_tiles * n_tiles);
    unsigned slice, t;
    if (slices % (int)NUM_XCD == 0) {
        const unsigned q = blockIdx.x / NUM_XCD;
        t = q % tiles;
        slice = (q / tiles) * NUM_XCD + blockIdx.x % NUM_XCD;
    } else {
        t = blockIdx.x % tiles;
        slice = blockIdx.x / tiles;
    }
    const int m0 = (int)(t % (unsigned)m_tiles) * (WG_UNITS * 16), n0 = (int)(t / (unsigned)m_tiles) * BN;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = wave & 3, half = wave >> 2;
    const int tap0 = m0 / c;
    const int n_blocks = (n + WG_VOX - 1) / WG_VOX;
    const int my_blocks = (int)slice < n_blocks ? (n_blocks - 1 - (int)slice) / slices + 1 : 0;

    constexpr int SRD3 = 0x00020000;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)(x_rows * c * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void *)dY, 0, (int)((int64_t)n * N * 4), SRD3);
    const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, (int)((int64_t)n * taps * 4), SRD3);

    // per unit and lane: index slot and channel of the lane's row; rows past the end use the slot
    // that names nothing
    uint32_t *tab = reinterpret_cast<uint32_t *>(lds + L::O_TAB);
    if (tid < WG_UNITS * 16) {
        const int m = m0 + tid, tap = m / c;
        const bool real = m < M && tap - tap0 < WG_UNITS;
        tab[tid] = real ? (uint32_t)(tap - tap0) << 24 | (uint32_t)(m - tap * c) * 4u : (uint32_t)WG_UNITS << 24;
    }
    for (int q = tid; q < 3 * WG_RS; q += 512)
        reinterpret_cast<uint32_t *>(lds + L::O_IDX + (q / WG_RS) * L::IDX)[WG_UNITS * WG_RS + q % WG_RS] = OUT;
    // the slots that each of this wavefront's units reads
    uint32_t unit_slots[7];
    [[maybe_unused]] int unit_slot[7], unit_ch[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int a = m0 + (g + 4 * i) * 16, b = min(a + 15, M - 1);
        const int lo = a / c - tap0, hi = min(b / c - tap0, WG_UNITS - 1);
        unit_slots[i] = a < M && lo <= hi ? ((2u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
        unit_slot[i] = a < M ? lo : WG_UNITS;                              // C16: the only one, and its first channel
        unit_ch[i] = a < M ? a - (a / c) * c : 0;
    }

    // ---- staging: index rows two blocks ahead, dY one
    const int sr = tid >> 2, sq = (tid & 3) * 7;                           // this thread's voxel and first slot
    auto voxel = [&](int k) -> int {                                       // voxel sr of the slice's k-th block, or -1
        const int64_t p = ((int64_t)slice + (int64_t)k * slices) * WG_VOX + sr;
        const bool ok = k < my_blocks && p < n;
        const int v = order ? order[ok ? p : 0] : (int)p;
        return ok ? v : -1;
    };
    int32_t ix[7];
    auto fetch_idx = [&](int vox) {
        const uint32_t row = vox >= 0 ? (uint32_t)(vox * taps + tap0 + sq) * 4u : OUT;
#pragma unroll
        for (int j = 0; j < 7; ++j) ix[j] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_n, (int)(row + 4u * j), 0, 0);
    };
    // an absent neighbour (-1) becomes a negative, i.e. huge unsigned, byte offset; slots past the
    // last tap hold whatever follows in memory and are read by nobody
    auto store_idx = [&](int ring, int vox) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(lds + L::O_IDX + ring * L::IDX) + sq * WG_RS + sr;
        uint32_t have = 0;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int32_t q = vox >= 0 ? ix[j] : -1;
            dst[j * WG_RS] = (uint32_t)__mul24(q, c * 4);
            have |= (uint32_t)(~q >> 31) & (1u << j);
        }
        have <<= sq;
        if ((tid & 3) == 0)
            reinterpret_cast<uint32_t *>(lds + L::O_ORD)[ring * WG_VOX + sr] = vox >= 0 ? (uint32_t)vox * (uint32_t)(N * 4) : OUT;
        // or of the wavefront's 16 voxels, which ends up in its last lane
        int h = (int)have;
        h |= __builtin_amdgcn_update_dpp(0, h, 0x111, 0xF, 0xF, true);     // row_shr 1, 2, 4, 8
        h |= __builtin_amdgcn_update_dpp(0, h, 0x112, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x114, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x118, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x142, 0xA, 0xF, true);     // lane 15 of a row to the next, ...
        h |= __builtin_amdgcn_update_dpp(0, h, 0x143, 0xC, 0xF, true);     // ... lane 31 to the upper half
        if (lane == 63) reinterpret_cast<int *>(lds + L::O_MASK)[ring * 8 + wave] = h;
    };
    constexpr int YU = BN * (WG_VOX / 8) / 512;                            // (column, 8 voxels) units per thread
    static_assert(YU == 1 || YU == 2, "32 or 64 columns");
    float yv[8];
    const int yn = tid % BN, yg = tid / BN;                                // first group of 8 voxels
    const uint32_t y_off = n0 + yn < N ? (uint32_t)(n0 + yn) * 4u : OUT - 1u;    // (plus OUT, a missing voxel, still outside)
    auto fetch_dy = [&](int ring, int q) {
        const uint32_t *ord = reinterpret_cast<const uint32_t *>(lds + L::O_ORD) + ring * WG_VOX + (yg + q * (512 / BN)) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            yv[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_y, (int)(ord[j] + y_off), 0, 0));
    };
    auto store_dy = [&](int stage, int q) {
        const int vg = yg + q * (512 / BN);
        const uint32_t sign = vg & 4 ? 0x80000000u : 0u;                   // every other 32 voxels negated, see mfma_split
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = __uint_as_float(__float_as_uint(yv[j]) ^ sign);
        u32x4 p[3];
        split3(v, p[0], p[1], p[2]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
            *reinterpret_cast<u32x4 *>(lds + stage * L::DY + ((((vg >> 2) * 3 + pl) * 4 + (vg & 3)) * BN + yn) * 16) = p[pl];
    };

    f32x4 acc[7][NT];
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[i][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // taps that the two 32-voxel parts of the wavefront's half of a block have
    auto part_taps = [&](int ring, int part) -> uint32_t {
        const uint32_t *mk = reinterpret_cast<const uint32_t *>(lds + L::O_MASK) + ring * 8 + half * 4 + part * 2;
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(mk[0] | mk[1]));
    };
    // the rows behind unit i for 8 voxels per lane, in two steps: their byte offsets from LDS, then the
    // loads.  Rows of a multiple of 16 channels (C16): a unit lies within one tap, slot and first
    // channel are the same for all lanes
    auto fetch_off = [&](int ring, int part, int i, u32x4 *o) {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(lds + L::O_IDX + ring * L::IDX) + (half * 2 + part) * 32 + lk * 8;
        uint32_t ch = (uint32_t)li * 4u;
        if constexpr (C16) src += unit_slot[i] * WG_RS;
        else {
            const uint32_t e = tab[(g + 4 * i) * 16 + li];
            src += (e >> 24) * WG_RS;
            ch = e & 0xFFFFFFu;
        }
        o[0] = *reinterpret_cast<const u32x4 *>(src);
        o[1] = *reinterpret_cast<const u32x4 *>(src + 4);
        if constexpr (!C16)
            for (int j = 0; j < 4; ++j) { o[0][j] += ch; o[1][j] += ch; }
    };
    auto fetch_x = [&](int i, const u32x4 *o, float *raw) {
        const uint32_t ch = C16 ? (uint32_t)li * 4u : 0u;
        const int soff = C16 ? unit_ch[i] * 4 : 0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            raw[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_x, (int)(o[j >> 2][j & 3] + ch), soff, 0));
    };

    if (my_blocks > 0) {
        int v0 = voxel(0), v1 = voxel(1), v2 = voxel(2);
        fetch_idx(v0);
        store_idx(0, v0);
        fetch_idx(v1);
        store_idx(1, v1);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < YU; ++q) { fetch_dy(0, q); store_dy(0, q); }
        __syncthreads();
        float raw[D][8];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            u32x4 o[2];
            fetch_off(0, 0, i, o);
            fetch_x(i, o, raw[i]);
        }
        int r0 = 0, r1 = 1, r2 = 2;                                        // ring positions of blocks k, k+1, k+2
        for (int k = 0; k < my_blocks; ++k) {
            fetch_idx(v2);
            const int v3 = voxel(k + 3);
            fetch_dy(r1, 0);
            const unsigned char *dy = lds + (k & 1) * L::DY;
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                if (part == 1) {
                    // the first half of what this block stages has arrived: into LDS, and on to the second
                    store_idx(r2, v2);
                    store_dy((k + 1) & 1, 0);
                    if constexpr (YU == 2) fetch_dy(r1, 1);
                }
                const uint32_t have = part_taps(r0, part);
                u32x4 b[NT][3];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
                        b[nt][pl] = *reinterpret_cast<const u32x4 *>(dy + ((((half * 2 + part) * 3 + pl) * 4 + lk) * BN + nt * 16 + li) * 16);
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    const int it = part * 7 + i, next = (it + D) % 14;
                    u32x4 o[2];
                    fetch_off(it + D < 14 ? r0 : r1, next / 7, next % 7, o);
                    __builtin_amdgcn_sched_barrier(0);
                    if (have & unit_slots[i]) {
                        u32x4 a[3];
                        split3(raw[it % D], a[0], a[1], a[2]);
                        if (part == 0) mfma_split<NT, false>(a, b, acc[i]);
                        else mfma_split<NT, true>(a, b, acc[i]);
                    }
                    fetch_x(next % 7, o, raw[it % D]);
                }
            }
            if constexpr (YU == 2) store_dy((k + 1) & 1, 1);
            v2 = v3;
            const int r = r0; r0 = r1; r1 = r2; r2 = r;
            __syncthreads();
        }
    }

    // An infinity or NaN among the operands (or a sum out of range) has left a non-finite sum: such a
    // wavefront takes the fp32 sums of its voxels instead, which is what such numbers mean.
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 4; ++e) bad |= non_finite(acc[i][nt][e]);
    bad = __builtin_expect(__ballot(bad) != 0, 0);
    // (The fp32 instruction, 32 voxels at a time and tap by tap: dY counts only where the voxel has the tap --
    // an absent row is not zero times an infinity -- and of the result only the rows of that tap.  From
    // memory, without LDS or barriers.  Every number a NaN, 32 -> 64 at 40 000 voxels: 139 us, 9.1 ms with the
    // outputs summed one after the other; at 280 000 voxels 554 us, 141 with finite numbers.)
    if (bad) {
#pragma unroll
        for (int i = 0; i < 7; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[i][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int q = 0; q < 2 * my_blocks; ++q) {
            const int64_t p0 = ((int64_t)slice + (int64_t)(q >> 1) * slices) * WG_VOX + half * 64 + (q & 1) * 32 + lk * 8;
            int vox[8];
            float y[NT][8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool ok = p0 + j < n;
                const int v = order ? order[ok ? p0 + j : 0] : (int)(p0 + j);
                vox[j] = ok ? v : -1;
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int col = n0 + nt * 16 + li;
                    y[nt][j] = vox[j] >= 0 && col < N ? dY[(int64_t)vox[j] * N + col] : 0.f;
                }
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int a = m0 + (g + 4 * i) * 16, m = min(a + li, M - 1), ch = m - m / c * c;
                const int last = min(a + 15, M - 1) / c;
#pragma unroll 1
                for (int tap = a / c; tap <= last; ++tap) {
                    int row[8];
                    float x[8];
                    bool any = false;
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        row[j] = vox[j] >= 0 ? nbr[(int64_t)vox[j] * taps + tap] : -1;
                        any |= row[j] >= 0;
                    }
                    if (__ballot(any) == 0) continue;
#pragma unroll
                    for (int j = 0; j < 8; ++j) x[j] = row[j] >= 0 ? X[(int64_t)row[j] * c + ch] : 0.f;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int j = 0; j < 8; ++j) t = mfma_f32(x[j], row[j] >= 0 ? y[nt][j] : 0.f, t);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i][nt][e] += (a + lk * 4 + e) / c == tap ? t[e] : 0.f;
                    }
                }
            }
        }
    }
    const float unscale = bad ? 1.f : SPLIT_UNSCALE;

    // second half of every block -> LDS, added by the wavefront that has the first half
    f32x4 *sums = reinterpret_cast<f32x4 *>(lds) + g * 7 * NT * 64 + lane;
    if (half == 1) {
#pragma unroll
        for (int i = 0; i < 7; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sums[(i * NT + nt) * 64] = acc[i][nt] * unscale;
    }
    __syncthreads();
    if (half == 1) return;
    C += (int64_t)slice * c_split_stride;
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const f32x4 v = acc[i][nt] * unscale + sums[(i * NT + nt) * 64];
            const int col = n0 + nt * 16 + li;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = m0 + (g + 4 * i) * 16 + lk * 4 + e;
                if (m < M && col < N) C[(int64_t)m * N + col] = v[e];
            }
        }
}

// The same product with bf16 operands, which need no cutting.  Rows are taken in pairs of channels (a
// lane loads 32 bits and gives one half to each of two operands), so a unit is 32 rows of dW; a
// wavefront has 4 of the 16 units of a workgroup.  The second half of every block enters with the
// opposite sign and is subtracted at the end, for the reason given at mfma_split (inputs of one sign,
// a million voxels: results 1.2e-8 too small without it, 3e-10 with it).  64 -> 64 at 2.98 M voxels (512^3,
// thick shells): 1170 -> 877 us with the taps that 32 voxels lack left out.  Bound by memory there: the
// gathered rows, 0.31 of which are found in L2, are 5.3 GB from HBM, 6.0 TB/s; at 280 000 voxels 99 us
// (120 with every tap).
constexpr int WGB_UNITS = 16;
template <int NT>
struct WgradBfLds {
    static constexpr int BN = 16 * NT;
    static constexpr int DY = WG_VOX / 32 * 4 * BN * 16;
    static constexpr int IDX = WG_SLOTS * WG_RS * 4;
    static constexpr int O_IDX = 2 * DY, O_ORD = O_IDX + 3 * IDX, O_MASK = O_ORD + 3 * WG_VOX * 4;
    static constexpr int O_TAB = O_MASK + 3 * 8 * 4, TOTAL = O_TAB + WGB_UNITS * 16 * 4;
    static constexpr int HALF = 4 * 8 * NT * 4 * 64 * 4;
    static constexpr int BYTES = TOTAL > HALF ? TOTAL : HALF;
};

template <int NT>
__global__ __launch_bounds__(512) void wgrad_bf16_kernel(
    const uint16_t *__restrict__ X, const uint16_t *__restrict__ dY, float *__restrict__ C,
    const int32_t *__restrict__ nbr, const int32_t *__restrict__ order, int M, int N, int n, int64_t x_rows, int c, int taps,
    int slices, int m_tiles, int n_tiles, int64_t c_split_stride)
{
    typedef WgradBfLds<NT> L;
    constexpr int BN = L::BN;
    constexpr uint32_t OUT = 0x80000000u;
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::BYTES];

    const unsigned tiles = (unsigned)(m_tiles * n_tiles);
    unsigned slice, t;
    if (slices % (int)NUM_XCD == 0) {
        const unsigned q = blockIdx.x / NUM_XCD;
        t = q % tiles;
        slice = (q / tiles) * NUM_XCD + blockIdx.x % NUM_XCD;
    } else {
        t = blockIdx.x % tiles;
        slice = blockIdx.x / tiles;
    }
    const int m0 = (int)(t % (unsigned)m_tiles) * (WGB_UNITS * 32), n0 = (int)(t / (unsigned)m_tiles) * BN;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = wave & 3, half = wave >> 2;
    const int tap0 = m0 / c;
    const int n_blocks = (n + WG_VOX - 1) / WG_VOX;
    const int my_blocks = (int)slice < n_blocks ? (n_blocks - 1 - (int)slice) / slices + 1 : 0;

    constexpr int SRD3 = 0x00020000;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)(x_rows * c * 2), SRD3);
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void *)dY, 0, (int)((int64_t)n * N * 2), SRD3);
    const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc((void *)nbr, 0, (int)((int64_t)n * taps * 4), SRD3);

    uint32_t *tab = reinterpret_cast<uint32_t *>(lds + L::O_TAB);
    if (tid < WGB_UNITS * 16) {
        const int m = m0 + 2 * tid, tap = m / c;
        tab[tid] = m < M ? (uint32_t)(tap - tap0) << 24 | (uint32_t)(m - tap * c) * 2u : (uint32_t)WG_UNITS << 24;
    }
    for (int q = tid; q < 3 * WG_RS; q += 512)
        reinterpret_cast<uint32_t *>(lds + L::O_IDX + (q / WG_RS) * L::IDX)[WG_UNITS * WG_RS + q % WG_RS] = OUT;
    uint32_t unit_slots[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int a = m0 + (g + 4 * i) * 32, b = min(a + 31, M - 1);
        const int lo = a / c - tap0, hi = b / c - tap0;
        unit_slots[i] = a < M ? ((2u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
    }

    // ---- staging: index rows two blocks ahead, dY one
    const int sr = tid >> 2, sq = (tid & 3) * 7;                           // this thread's voxel and first slot
    auto voxel = [&](int k) -> int {                                       // voxel sr of the slice's k-th block, or -1
        const int64_t p = ((int64_t)slice + (int64_t)k * slices) * WG_VOX + sr;
        const bool ok = k < my_blocks && p < n;
        const int v = order ? order[ok ? p : 0] : (int)p;
        return ok ? v : -1;
    };
    int32_t ix[7];
    auto fetch_idx = [&](int vox) {
        const uint32_t row = vox >= 0 ? (uint32_t)(vox * taps + tap0 + sq) * 4u : OUT;
#pragma unroll
        for (int j = 0; j < 7; ++j) ix[j] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_n, (int)(row + 4u * j), 0, 0);
    };
    // an absent neighbour (-1) becomes a negative, i.e. huge unsigned, byte offset; slots past the
    // last tap hold whatever follows in memory and are read by nobody
    auto store_idx = [&](int ring, int vox) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(lds + L::O_IDX + ring * L::IDX) + sq * WG_RS + sr;
        uint32_t have = 0;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int32_t q = vox >= 0 ? ix[j] : -1;
            dst[j * WG_RS] = (uint32_t)__mul24(q, c * 2);
            have |= (uint32_t)(~q >> 31) & (1u << j);
        }
        have <<= sq;
        if ((tid & 3) == 0)
            reinterpret_cast<uint32_t *>(lds + L::O_ORD)[ring * WG_VOX + sr] = vox >= 0 ? (uint32_t)vox * (uint32_t)(N * 2) : OUT;
        // or of the wavefront's 16 voxels, which ends up in its last lane
        int h = (int)have;
        h |= __builtin_amdgcn_update_dpp(0, h, 0x111, 0xF, 0xF, true);     // row_shr 1, 2, 4, 8
        h |= __builtin_amdgcn_update_dpp(0, h, 0x112, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x114, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x118, 0xF, 0xF, true);
        h |= __builtin_amdgcn_update_dpp(0, h, 0x142, 0xA, 0xF, true);     // lane 15 of a row to the next, ...
        h |= __builtin_amdgcn_update_dpp(0, h, 0x143, 0xC, 0xF, true);     // ... lane 31 to the upper half
        if (lane == 63) reinterpret_cast<int *>(lds + L::O_MASK)[ring * 8 + wave] = h;
    };
    // columns come in pairs as well
    const int yn = tid % (BN / 2), yg = tid / (BN / 2);
    const bool y_mine = yg < WG_VOX / 8;
    const uint32_t y_off = n0 + 2 * yn < N ? (uint32_t)(n0 + 2 * yn) * 2u : OUT - 1u;
    uint32_t yv[8];
    auto fetch_dy = [&](int ring) {
        const uint32_t *ord = reinterpret_cast<const uint32_t *>(lds + L::O_ORD) + ring * WG_VOX + (yg % (WG_VOX / 8)) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) yv[j] = __builtin_amdgcn_raw_buffer_load_b32(rs_y, (int)(ord[j] + y_off), 0, 0);
    };
    auto store_dy = [&](int stage) {
        if (!y_mine) return;
        const uint32_t sign = yg & 8 ? 0x80008000u : 0u;                   // the second half of the block
        u32x4 e, o;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            e[p] = pack_lo(yv[2 * p], yv[2 * p + 1]) ^ sign;
            o[p] = pack_hi(yv[2 * p], yv[2 * p + 1]) ^ sign;
        }
        u32x4 *dst = reinterpret_cast<u32x4 *>(lds + stage * L::DY + (yg * BN + 2 * yn) * 16);
        dst[0] = e;
        dst[1] = o;
    };

    f32x4 acc[4][2][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[i][q][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto part_taps = [&](int ring, int part) -> uint32_t {
        const uint32_t *mk = reinterpret_cast<const uint32_t *>(lds + L::O_MASK) + ring * 8 + half * 4 + part * 2;
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(mk[0] | mk[1]));
    };
    auto fetch_off = [&](int ring, int part, int i, u32x4 *o) {
        const uint32_t e = tab[(g + 4 * i) * 16 + li], ch = e & 0xFFFFFFu;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(lds + L::O_IDX + ring * L::IDX) + (e >> 24) * WG_RS + (half * 2 + part) * 32 + lk * 8;
        o[0] = *reinterpret_cast<const u32x4 *>(src);
        o[1] = *reinterpret_cast<const u32x4 *>(src + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) { o[0][j] += ch; o[1][j] += ch; }
    };
    auto fetch_x = [&](const u32x4 *o, uint32_t *raw) {
#pragma unroll
        for (int j = 0; j < 8; ++j) raw[j] = __builtin_amdgcn_raw_buffer_load_b32(rs_x, (int)o[j >> 2][j & 3], 0, 0);
    };

    if (my_blocks > 0) {
        int v0 = voxel(0), v1 = voxel(1), v2 = voxel(2);
        fetch_idx(v0);
        store_idx(0, v0);
        fetch_idx(v1);
        store_idx(1, v1);
        __syncthreads();
        fetch_dy(0);
        store_dy(0);
        __syncthreads();
        constexpr int D = 4;                                               // units whose rows are on their way (divides 8)
        uint32_t raw[D][8];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            u32x4 o[2];
            fetch_off(0, 0, i, o);
            fetch_x(o, raw[i]);
        }
        int r0 = 0, r1 = 1, r2 = 2;
        for (int k = 0; k < my_blocks; ++k) {
            fetch_idx(v2);
            const int v3 = voxel(k + 3);
            fetch_dy(r1);
            const unsigned char *dy = lds + (k & 1) * L::DY;
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                if (part == 1) {
                    store_idx(r2, v2);
                    store_dy((k + 1) & 1);
                }
                const uint32_t have = part_taps(r0, part);
                u32x4 b[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    b[nt] = *reinterpret_cast<const u32x4 *>(dy + (((half * 2 + part) * 4 + lk) * BN + nt * 16 + li) * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int it = part * 4 + i, next = (it + D) % 8;
                    u32x4 o[2];
                    fetch_off(it + D < 8 ? r0 : r1, next / 4, next % 4, o);
                    __builtin_amdgcn_sched_barrier(0);
                    if (have & unit_slots[i]) {
                        u32x4 a[2];
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            a[0][p] = pack_lo(raw[it % D][2 * p], raw[it % D][2 * p + 1]);
                            a[1][p] = pack_hi(raw[it % D][2 * p], raw[it % D][2 * p + 1]);
                        }
#pragma unroll
                        for (int q = 0; q < 2; ++q)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt) acc[i][q][nt] = mfma_bf16(a[q], b[nt], acc[i][q][nt]);
                    }
                    fetch_x(o, raw[it % D]);
                }
            }
            v2 = v3;
            const int r = r0; r0 = r1; r1 = r2; r2 = r;
            __syncthreads();
        }
    }

    f32x4 *sums = reinterpret_cast<f32x4 *>(lds) + g * 8 * NT * 64 + lane;
    if (half == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) sums[((i * 2 + q) * NT + nt) * 64] = acc[i][q][nt];
    }
    __syncthreads();
    if (half == 1) return;
    C += (int64_t)slice * c_split_stride;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const f32x4 v = acc[i][q][nt] - sums[((i * 2 + q) * NT + nt) * 64];
                const int col = n0 + nt * 16 + li;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = m0 + (g + 4 * i) * 32 + 2 * (lk * 4 + e) + q;
                    if (m < M && col < N) C[(int64_t)m * N + col] = v[e];
                }
            }
}

}  // namespace hch
