// Construction of the perfect spatial hash tables on the device (the paper leaves this as
// future work, Section 5.2 and the conclusion; its tables are built offline on the host).
//
// The structure and the sizes are the paper's (Section 3.1, 5.2): hash table side m with
// m^3 > n, offset table side r starting from 6 r^3 >= n and growing when an attempt fails,
// h(p) = (p mod m + Phi[p mod r]) mod m per axis, H holding data indices, T the position tags.
// The assignment of offsets is a parallel greedy one, made for thousands of threads instead
// of the one-bucket-at-a-time order of the host construction:
//   * every (level, model) pair of the batch is built in the same launches;
//   * buckets (voxels sharing p mod r) are placed in classes of decreasing size (9 and more,
//     8, 7, ..., 2, 1), one launch per class, all buckets of a class at once;
//   * before each class the free slots of every table are listed; a bucket's candidates are the
//     free slots (its first voxel goes there, which fixes the offset), starting at a hashed
//     position of the list;
//   * one wavefront per bucket: 64 candidates are examined at once (a lane looks whether the
//     slots of all the bucket's voxels are free), then the first lane that found room claims the
//     slots with compare-and-swap on H and, if another bucket was faster on one of them, gives
//     the claimed ones back and the next lane tries;
//   * buckets of one voxel need no search: the i-th of them takes the i-th free slot;
//   * a bucket that runs out of candidates fails its pair; failed pairs are cleared and repeated
//     with the next r.
// Which of two racing buckets gets a slot depends on timing, so the tables are valid but not
// reproducible bit for bit; everything computed THROUGH them (lookups, neighbour and child
// lists, convolutions) is the same for every valid table.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hch {

struct PairDesc {
    const int32_t *coords;   // [n][3] positions of this model at this level, data order
    int32_t *H;              // [m^3] this pair's part of H*, -1 = free
    uint16_t *T;             // [m^3][3]
    int32_t n, m, r;
    int32_t cell_base;       // first offset cell of the pair in this attempt's cell arrays
    int32_t vox_base;        // first entry of the pair in this attempt's member arrays
    int32_t slot_base;       // first entry of the pair in this attempt's free-slot list
    int32_t pair_id;         // index into the failure flags
};

constexpr int PSH_CLASSES = 10;      // class k holds the buckets of k voxels, class 9 those of 9 and more

// bucket number of every voxel, bucket sizes
__global__ __launch_bounds__(256) void psh_count_kernel(const PairDesc *__restrict__ pairs,
                                                        int32_t *__restrict__ cnt, int32_t *__restrict__ bucket_of)
{
    const PairDesc P = pairs[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= P.n) return;
    const int32_t *p = P.coords + 3 * (int64_t)i;
    const int r = P.r;
    const int g = ((p[0] % r) * r + (p[1] % r)) * r + (p[2] % r);
    bucket_of[P.vox_base + i] = g;
    atomicAdd(&cnt[P.cell_base + g], 1);
}

// Exclusive prefix sum of `n` counts in two launches: the sum of every PSH_SCAN counts, then each
// stretch on top of the stretches before it (a few hundred at most, added up by its workgroup).  One
// workgroup that walked through all of them took 290 us for the 140 000 cells of a 256^3 batch of 8.
constexpr int PSH_SCAN = 2048;       // 8 per thread, consecutive
__global__ __launch_bounds__(256) void psh_sum_kernel(const int32_t *__restrict__ in, int32_t *__restrict__ sums, int n)
{
    __shared__ int32_t part[4];
    int32_t s = 0;
#pragma unroll
    for (int q = 0; q < PSH_SCAN / 256; ++q) {
        const int i = (int)blockIdx.x * PSH_SCAN + q * 256 + (int)threadIdx.x;
        s += i < n ? in[i] : 0;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
__global__ __launch_bounds__(256) void psh_scan_kernel(const int32_t *__restrict__ in, const int32_t *__restrict__ sums,
                                                       int32_t *__restrict__ out, int n)
{
    __shared__ int32_t part[256];
    constexpr int PER = PSH_SCAN / 256;
    const int t = threadIdx.x, i0 = (int)blockIdx.x * PSH_SCAN + t * PER;
    int32_t before = 0;
    for (int q = t; q < (int)blockIdx.x; q += 256) before += sums[q];
    int32_t v[PER], s = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) { v[q] = i0 + q < n ? in[i0 + q] : 0; s += v[q]; }
    part[t] = before;
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
        if (t < d) part[t] += part[t + d];
        __syncthreads();
    }
    before = part[0];
    __syncthreads();
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int32_t add = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    int32_t run = before + part[t] - s;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (i0 + q < n) { out[i0 + q] = run; run += v[q]; }
}

// member lists: the voxels of every bucket (order inside a bucket is arbitrary) with their
// residues modulo m, packed x | y << 8 | z << 16
__global__ __launch_bounds__(256) void psh_fill_kernel(const PairDesc *__restrict__ pairs,
                                                       const int32_t *__restrict__ bucket_of,
                                                       const int32_t *__restrict__ first,
                                                       int32_t *__restrict__ fill, int32_t *__restrict__ members,
                                                       uint32_t *__restrict__ residues)
{
    const PairDesc P = pairs[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= P.n) return;
    const int cell = P.cell_base + bucket_of[P.vox_base + i];
    const int pos = first[cell] + atomicAdd(&fill[cell], 1);
    const int32_t *p = P.coords + 3 * (int64_t)i;
    const int m = P.m;
    members[pos] = i;
    residues[pos] = (uint32_t)(p[0] % m) | ((uint32_t)(p[1] % m) << 8) | ((uint32_t)(p[2] % m) << 16);
}

// The buckets of 2 and more voxels, listed by class: entry = (active pair, bucket number).  Positions
// are counted in LDS and a class's counter is advanced once per workgroup: with one advance per
// wavefront the atomics on these few addresses took 213 us (256^3, batch of 8).
__global__ __launch_bounds__(256) void psh_classify_kernel(const PairDesc *__restrict__ pairs,
                                                           const int32_t *__restrict__ cnt,
                                                           int32_t *__restrict__ class_count,
                                                           int2 *__restrict__ class_cells, int64_t class_stride)
{
    __shared__ int32_t count[PSH_CLASSES], base[PSH_CLASSES];
    const PairDesc P = pairs[blockIdx.y];
    const int cells = P.r * P.r * P.r;
    if ((int)blockIdx.x * 256 >= cells) return;       // whole workgroups
    const int g = blockIdx.x * 256 + threadIdx.x;
    const int c = g < cells ? cnt[P.cell_base + g] : 0;
    const int mine = c < 2 ? 0 : (c < PSH_CLASSES - 1 ? c : PSH_CLASSES - 1);
    if (threadIdx.x < PSH_CLASSES) count[threadIdx.x] = 0;
    __syncthreads();
    const int pos = mine ? atomicAdd(&count[mine], 1) : 0;
    __syncthreads();
    if (threadIdx.x < PSH_CLASSES && count[threadIdx.x]) base[threadIdx.x] = atomicAdd(&class_count[threadIdx.x], count[threadIdx.x]);
    __syncthreads();
    if (mine) class_cells[mine * class_stride + base[mine] + pos] = make_int2((int)blockIdx.y, g);
}

// The free slots of every table (any order), PSH_FREE slots per workgroup, which advances its table's
// counter once (one advance per wavefront: 155 us a launch, and a build has a dozen of them).
constexpr int PSH_FREE = 4096;
__global__ __launch_bounds__(256) void psh_free_list_kernel(const PairDesc *__restrict__ pairs,
                                                            int32_t *__restrict__ n_free, int32_t *__restrict__ free_list)
{
    __shared__ int32_t count, base;
    const PairDesc P = pairs[blockIdx.y];
    const int slots = P.m * P.m * P.m, e0 = (int)blockIdx.x * PSH_FREE;
    if (e0 >= slots) return;                          // whole workgroups
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    uint32_t is_free = 0;
#pragma unroll
    for (int q = 0; q < PSH_FREE / 256; ++q) {
        const int e = e0 + q * 256 + (int)threadIdx.x;
        is_free |= e < slots && P.H[min(e, slots - 1)] == -1 ? 1u << q : 0u;
    }
    int pos = atomicAdd(&count, __popc(is_free));
    __syncthreads();
    if (threadIdx.x == 0) base = atomicAdd(&n_free[blockIdx.y], count);
    __syncthreads();
    pos += base;
#pragma unroll
    for (int q = 0; q < PSH_FREE / 256; ++q)
        if (is_free >> q & 1u) free_list[P.slot_base + pos++] = e0 + q * 256 + (int)threadIdx.x;
}

__device__ __forceinline__ int32_t psh_peek(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// slot of a voxel with packed residues h under the offset (ox, oy, oz)
__device__ __forceinline__ int psh_slot_of(uint32_t h, int ox, int oy, int oz, int m)
{
    int x = (int)(h & 255u) + ox; if (x >= m) x -= m;
    int y = (int)((h >> 8) & 255u) + oy; if (y >= m) y -= m;
    int z = (int)(h >> 16) + oz; if (z >= m) z -= m;
    return (x * m + y) * m + z;
}

// Place the buckets of one class (2 voxels and more): one wavefront per bucket, 4 per workgroup.
// phi4[cell] receives the offset, packed x | y << 8 | z << 16.
constexpr int PSH_WIDE = 4;
__global__ __launch_bounds__(256) void psh_place_kernel(
    const PairDesc *__restrict__ pairs, const int2 *__restrict__ cells, int n_buckets,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ first, const int32_t *__restrict__ members,
    const uint32_t *__restrict__ residues, const int32_t *__restrict__ n_free,
    const int32_t *__restrict__ free_list, uint32_t *__restrict__ phi4, int32_t *__restrict__ fail)
{
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (b >= n_buckets) return;                       // whole wavefronts leave together
    const int2 ag = cells[b];
    const PairDesc P = pairs[ag.x];
    const int g = ag.y, cell = P.cell_base + g;
    const int c = cnt[cell], base = first[cell];
    const int m = P.m;
    const int nf = n_free[ag.x];
    int32_t *H = P.H;
    const int32_t *list = free_list + P.slot_base;
    const uint32_t h_first = residues[base];
    const int ax = h_first & 255u, ay = (h_first >> 8) & 255u, az = h_first >> 16;
    const int start = nf > 0 ? (int)(((uint32_t)g * 2654435761u) % (uint32_t)nf) : 0;

    // 64 candidates at first, the usual case; then four times as many at a time, their loads side by
    // side: a bucket that finds no room at all has to look at every free slot, and those buckets
    // (their pair then tries the next r) are what a launch waits for at the end
    for (int i0 = 0, wide = 1; i0 < nf; i0 += 64 * wide, wide = PSH_WIDE) {
        if (psh_peek(&fail[P.pair_id])) return;       // the pair is lost anyway
        int slot[PSH_WIDE];
        bool rooms[PSH_WIDE];
#pragma unroll
        for (int q = 0; q < PSH_WIDE; ++q) {
            const int i = i0 + q * 64 + lane;
            rooms[q] = q < wide && i < nf;
            int w = start + (rooms[q] ? i : 0); if (w >= nf) w -= nf;
            slot[q] = list[w];
        }
#pragma unroll
        for (int q = 0; q < PSH_WIDE; ++q) rooms[q] &= psh_peek(H + slot[q]) == -1;
        int off[PSH_WIDE];
#pragma unroll
        for (int q = 0; q < PSH_WIDE; ++q) {
            const int sx = slot[q] / (m * m), sy = (slot[q] / m) % m, sz = slot[q] % m;
            int x = sx - ax; if (x < 0) x += m;
            int y = sy - ay; if (y < 0) y += m;
            int z = sz - az; if (z < 0) z += m;
            off[q] = x | y << 8 | z << 16;
        }
        for (int k = 1; k < c; ++k) {
            bool any = false;
#pragma unroll
            for (int q = 0; q < PSH_WIDE; ++q) any |= rooms[q];
            if (!__ballot(any)) break;
            const uint32_t h = residues[base + k];
            int32_t seen[PSH_WIDE];
#pragma unroll
            for (int q = 0; q < PSH_WIDE; ++q)
                seen[q] = rooms[q] ? psh_peek(H + psh_slot_of(h, off[q] & 255, off[q] >> 8 & 255, off[q] >> 16, m)) : 0;
#pragma unroll
            for (int q = 0; q < PSH_WIDE; ++q) rooms[q] &= seen[q] == -1;
        }
        for (int q = 0; q < wide; ++q) {
            const bool room = q == 0 ? rooms[0] : q == 1 ? rooms[1] : q == 2 ? rooms[2] : rooms[3];
            const int o = q == 0 ? off[0] : q == 1 ? off[1] : q == 2 ? off[2] : off[3];
            const int ox = o & 255, oy = o >> 8 & 255, oz = o >> 16;
            unsigned long long cand = __ballot(room);
            while (cand) {                                // wave-uniform loop
                const int j = __builtin_ctzll(cand);
                cand &= cand - 1;
                int won = 0;
                if (lane == j) {
                    int got = 0;
                    bool twice = false;     // two voxels of the bucket on one slot: no offset can separate them
                    for (int k = 0; k < c && got == k; ++k) {
                        const int32_t old = atomicCAS(H + psh_slot_of(residues[base + k], ox, oy, oz, m), -1, members[base + k]);
                        if (old == -1) got = k + 1;
                        else for (int kk = 0; kk < k; ++kk) twice |= old == members[base + kk];
                    }
                    if (twice) { fail[P.pair_id] = 1; won = 1; }
                    if (got == c) {
                        for (int k = 0; k < c; ++k) {
                            const int32_t *p = P.coords + 3 * (int64_t)members[base + k];
                            uint16_t *tag = P.T + 3 * (int64_t)psh_slot_of(residues[base + k], ox, oy, oz, m);
                            tag[0] = (uint16_t)p[0]; tag[1] = (uint16_t)p[1]; tag[2] = (uint16_t)p[2];
                        }
                        phi4[cell] = (uint32_t)ox | ((uint32_t)oy << 8) | ((uint32_t)oz << 16);
                        won = 1;
                    } else {
                        for (int k = 0; k < got; ++k)     // give the claimed slots back
                            atomicExch(H + psh_slot_of(residues[base + k], ox, oy, oz, m), -1);
                    }
                }
                if (__ballot(won)) return;
            }
        }
    }
    if (lane == 0) fail[P.pair_id] = 1;
}

// Buckets of one voxel: the i-th of a table takes the i-th entry of its (fresh) free-slot list.
// Nothing else writes H during this launch.  One thread per offset cell.
__global__ __launch_bounds__(256) void psh_place_single_kernel(
    const PairDesc *__restrict__ pairs, const int32_t *__restrict__ cnt, const int32_t *__restrict__ first,
    const int32_t *__restrict__ members, const uint32_t *__restrict__ residues, const int32_t *__restrict__ n_free,
    const int32_t *__restrict__ free_list, int32_t *__restrict__ rank, uint32_t *__restrict__ phi4,
    int32_t *__restrict__ fail)
{
    const PairDesc P = pairs[blockIdx.y];
    const int g = blockIdx.x * 256 + threadIdx.x;
    if (g >= P.r * P.r * P.r) return;
    const int cell = P.cell_base + g;
    if (cnt[cell] != 1) return;
    const int i = atomicAdd(&rank[blockIdx.y], 1);
    if (i >= n_free[blockIdx.y]) { fail[P.pair_id] = 1; return; }   // cannot happen while m^3 > n
    const int e = free_list[P.slot_base + i];
    const int m = P.m;
    const uint32_t h = residues[first[cell]];
    const int32_t v = members[first[cell]];
    int ox = e / (m * m) - (int)(h & 255u); if (ox < 0) ox += m;
    int oy = (e / m) % m - (int)((h >> 8) & 255u); if (oy < 0) oy += m;
    int oz = e % m - (int)(h >> 16); if (oz < 0) oz += m;
    P.H[e] = v;
    const int32_t *p = P.coords + 3 * (int64_t)v;
    uint16_t *tag = P.T + 3 * (int64_t)e;
    tag[0] = (uint16_t)p[0]; tag[1] = (uint16_t)p[1]; tag[2] = (uint16_t)p[2];
    phi4[cell] = (uint32_t)ox | ((uint32_t)oy << 8) | ((uint32_t)oz << 16);
}

// Empties the tables of the pairs that failed, for their next attempt (grid as for the free-slot list).
__global__ __launch_bounds__(256) void psh_clear_kernel(const PairDesc *__restrict__ pairs, const int32_t *__restrict__ fail)
{
    const PairDesc P = pairs[blockIdx.y];
    if (!fail[P.pair_id]) return;
    const int slots = P.m * P.m * P.m, e1 = min(slots, (int)(blockIdx.x + 1) * PSH_FREE);
    for (int e = (int)blockIdx.x * PSH_FREE + (int)threadIdx.x; e < e1; e += 256) P.H[e] = -1;
    for (int e = 3 * (int)blockIdx.x * PSH_FREE + (int)threadIdx.x; e < 3 * e1; e += 256) P.T[e] = 0xFFFFu;
}

// One level's packed lookup records, model indices and byte offset table from H*, T* and the
// per-pair offset words.  grid.y = model.
struct PackDesc {
    const uint32_t *phi_src;  // this pair's offset words of its successful attempt
    int32_t m3, r3, M, R;     // sizes and bases inside the level's super tables
};

__global__ __launch_bounds__(256) void psh_pack_kernel(const PackDesc *__restrict__ desc, const int32_t *__restrict__ H,
                                                       const uint16_t *__restrict__ T, uint32_t *__restrict__ slot3,
                                                       int32_t *__restrict__ V, uint32_t *__restrict__ phi4,
                                                       uint8_t *__restrict__ Phi)
{
    const PackDesc D = desc[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < D.m3) {
        const int64_t q = (int64_t)D.M + i;
        slot3[SLOT_WORDS * q + 0] = (uint32_t)H[q];
        slot3[SLOT_WORDS * q + 1] = (uint32_t)T[3 * q] | ((uint32_t)T[3 * q + 1] << 16);
        slot3[SLOT_WORDS * q + 2] = (uint32_t)T[3 * q + 2];
        if (SLOT_WORDS > 3) slot3[SLOT_WORDS * q + 3] = 0u;
        V[q] = (int32_t)blockIdx.y;
    }
    if (i < D.r3) {
        const uint32_t w = D.phi_src[i];
        const int64_t q = (int64_t)D.R + i;
        phi4[q] = w;
        Phi[3 * q + 0] = (uint8_t)(w & 255u); Phi[3 * q + 1] = (uint8_t)((w >> 8) & 255u); Phi[3 * q + 2] = (uint8_t)((w >> 16) & 255u);
    }
}

}  // namespace hch
