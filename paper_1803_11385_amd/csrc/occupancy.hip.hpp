// Occupancy of the levels of a mini-batch on the device (Section 5.1: a coarse voxel is occupied iff one of the
// finer voxels below it is), and the checks of the finest level's positions: every one in the grid, none
// twice in a model.  One bit per position of every (level, model) grid; the coarse levels' voxels are the set
// bits in order of position.
#pragma once
#include "kernels.hip.hpp"

namespace hch {

constexpr int OCC_WORDS = 256;       // words of 64 bits per workgroup; a model's bits are padded to a multiple
struct OccupancySet {
    int n_levels, batch;
    int side[MAX_LEVELS], ratio[MAX_LEVELS];     // ratio of the finest side to this one's, as positions divide
    int64_t word_off[MAX_LEVELS];                // first word of a level; its models lie one behind the other
    int32_t blocks[MAX_LEVELS];                  // workgroups (OCC_WORDS words) per model
    int32_t block_off[MAX_LEVELS + 1];           // levels >= 1: first workgroup of a level among those of all
};

// Sets the bits of every level.  grid.y = model.  flags: 1 = a position outside the grid, 2 = one that occurs twice.
// Neighbouring lanes whose bits lie in one word (positions in order: runs along z) set them with one atomic, and
// at the coarse levels none where a look at the word, stale at worst, shows them set: with an atomic per voxel and
// level the kernel took 359 us for 609 000 voxels and 6 levels, so 36.
__global__ __launch_bounds__(256) void occupancy_mark_kernel(OccupancySet S, const int32_t *__restrict__ coords,
                                                             const int64_t *__restrict__ offsets, unsigned long long *bits,
                                                             int32_t *__restrict__ flags)
{
    const int v = blockIdx.y, lane = threadIdx.x & 63;
    const int64_t i = offsets[v] + (int64_t)blockIdx.x * 256 + threadIdx.x;
    const unsigned u = (unsigned)S.side[0];
    const bool have = i < offsets[v + 1];
    unsigned p0 = 0, p1 = 0, p2 = 0;
    if (have) { p0 = (unsigned)coords[3 * i]; p1 = (unsigned)coords[3 * i + 1]; p2 = (unsigned)coords[3 * i + 2]; }
    const bool good = have && p0 < u && p1 < u && p2 < u;
    if (have && !good) atomicOr(flags, 1);
    for (int l = 0; l < S.n_levels; ++l) {
        const unsigned d = (unsigned)S.ratio[l];
        const int64_t side = S.side[l], q = good ? ((int64_t)(p0 / d) * side + p1 / d) * side + p2 / d : -1;
        const int64_t word = q >> 6, before = __shfl_up(word, 1);
        const bool head = lane == 0 || word != before;
        const unsigned long long heads = __ballot(head);
        // the lanes up to the next head are this lane's run; its bits come together at the head
        const unsigned long long above = lane == 63 ? 0ull : heads >> (lane + 1);
        const int rest = above ? __builtin_ctzll(above) : 63 - lane;               // lanes of the run behind this one
        unsigned long long b = good ? 1ull << (q & 63) : 0ull;
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const unsigned long long other = __shfl_down(b, k);
            if (k <= rest) b |= other;
        }
        if (!good || !head) continue;
        unsigned long long *w = bits + S.word_off[l] + (int64_t)v * S.blocks[l] * OCC_WORDS + word;
        if (l == 0) {
            if (__popcll(b) != rest + 1 || (atomicOr(w, b) & b)) atomicOr(flags, 2);
        } else if ((*w & b) != b) atomicOr(w, b);
    }
}

__device__ __forceinline__ int occupancy_level(const OccupancySet &S, int block)
{
    int l = 1;
    while (l + 1 < S.n_levels && block >= S.block_off[l + 1]) ++l;
    return l;
}

// Set bits of every OCC_WORDS words of the levels >= 1, one workgroup each.
__global__ __launch_bounds__(OCC_WORDS) void occupancy_count_kernel(OccupancySet S, const unsigned long long *__restrict__ bits,
                                                                    int32_t *__restrict__ sums)
{
    __shared__ int32_t part[OCC_WORDS / 64];
    const int l = occupancy_level(S, (int)blockIdx.x);
    const int64_t w = S.word_off[l] + (int64_t)((int)blockIdx.x - S.block_off[l]) * OCC_WORDS + threadIdx.x;
    int32_t s = __popcll(bits[w]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Per (level >= 1, model), a workgroup each: the counts of its stretches become the voxels before them, and their sum
// the number of voxels.
__global__ __launch_bounds__(256) void occupancy_scan_kernel(OccupancySet S, int32_t *__restrict__ sums, int32_t *__restrict__ counts)
{
    __shared__ int32_t part[256];
    const int l = 1 + (int)blockIdx.x / S.batch, v = (int)blockIdx.x % S.batch, t = threadIdx.x;
    int32_t *mine = sums + S.block_off[l] + (int64_t)v * S.blocks[l];
    int32_t before = 0;
    for (int b0 = 0; b0 < S.blocks[l]; b0 += 256) {
        const int32_t s = b0 + t < S.blocks[l] ? mine[b0 + t] : 0;
        part[t] = s;
        __syncthreads();
        for (int d = 1; d < 256; d <<= 1) {
            const int32_t add = t >= d ? part[t - d] : 0;
            __syncthreads();
            part[t] += add;
            __syncthreads();
        }
        if (b0 + t < S.blocks[l]) mine[b0 + t] = before + part[t] - s;
        before += part[255];
        __syncthreads();
    }
    if (t == 0) counts[(l - 1) * S.batch + v] = before;
}

// The voxels of the levels >= 1 in order of position.  first[(l - 1) * batch + v]: a model's first voxel in its level.
struct OccupancyOut { int32_t *coords[MAX_LEVELS]; };
__global__ __launch_bounds__(OCC_WORDS) void occupancy_list_kernel(OccupancySet S, const unsigned long long *__restrict__ bits,
                                                                   const int32_t *__restrict__ sums, const int32_t *__restrict__ first,
                                                                   OccupancyOut out)
{
    __shared__ int32_t part[OCC_WORDS];
    const int l = occupancy_level(S, (int)blockIdx.x), t = threadIdx.x;
    const int flat = (int)blockIdx.x - S.block_off[l], v = flat / S.blocks[l];
    const int64_t w = (int64_t)(flat - v * S.blocks[l]) * OCC_WORDS + t;
    unsigned long long b = bits[S.word_off[l] + (int64_t)flat * OCC_WORDS + t];
    const int32_t s = __popcll(b);
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < OCC_WORDS; d <<= 1) {
        const int32_t add = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    const int64_t side = S.side[l];
    int32_t *dst = out.coords[l] + 3 * ((int64_t)first[(l - 1) * S.batch + v] + sums[blockIdx.x] + part[t] - s);
    for (; b; b &= b - 1, dst += 3) {
        const int64_t q = w * 64 + __builtin_ctzll(b);
        dst[0] = (int32_t)(q / (side * side));
        dst[1] = (int32_t)(q / side % side);
        dst[2] = (int32_t)(q % side);
    }
}

}  // namespace hch
