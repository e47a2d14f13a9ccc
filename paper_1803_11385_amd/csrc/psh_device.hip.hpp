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
//   * a bit per slot says whether it is taken.  A lane looks at 64 offsets at once: those that differ
//     in z only, for which a bucket's voxels read one stretch of 64 bits each; a wavefront looks at
//     64 such rows side by side, starting at a hashed one;
//   * one wavefront per bucket: the first offset with room for all of its voxels is claimed, every voxel's
//     bit by a lane of its own and all at once; if another bucket was faster on one of them, the
//     claimed ones are given back and the next offset is tried;
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
    int32_t row_base;        // first word of the pair in this attempt's bits (psh_row_words a row, m^2 rows)
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

// A row of the bits of taken slots, m of them in z, goes round: behind bit m - 1 come bits 0 .. 62 again, so
// that 64 bits can be read from any of the m positions (two words, the second one always there).
__host__ __device__ __forceinline__ int psh_row_words(int m) { return (m - 1) / 64 + 2; }
__device__ __forceinline__ unsigned long long psh_peek_row(const unsigned long long *row, int at)
{
    const unsigned long long lo = __hip_atomic_load(row + (at >> 6), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(row + (at >> 6) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (at & 63) ? lo >> (at & 63) | hi << (64 - (at & 63)) : lo;
}

// Place the bucket of c voxels in cell g of pair P: a wavefront.  phi4 receives the offset, packed
// x | y << 8 | z << 16.
__device__ __forceinline__ void psh_place_bucket(
    const PairDesc &P, int g, int c, const int32_t *__restrict__ members, const uint32_t *__restrict__ residues,
    unsigned long long *__restrict__ taken, uint32_t *__restrict__ phi4, int32_t *__restrict__ fail)
{
    const int lane = threadIdx.x & 63, m = P.m, rows = m * m, words = psh_row_words(m);
    const uint32_t mine = residues[min(lane, c - 1)];             // lane k has voxel k; those beyond 64 come from memory
    auto residue = [&](int k) -> uint32_t { return k < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)mine, k) : residues[k]; };
    auto wrap = [&](int v) { return v >= m ? v - m : v; };
    const uint32_t hash = (uint32_t)g * 2654435761u;
    const int start = (int)(hash % (uint32_t)rows), bit0 = (int)(hash >> 26);

    bool raced = true, twins_checked = false;
    // an offset lost to another bucket that then gave its slots back is worth another look, a few times
    for (int pass = 0; pass < 4 && raced; ++pass) {
        raced = false;
        for (int i0 = 0; i0 < rows; i0 += 64) {
            int q = start + i0 + lane;
            if (q >= rows) q -= rows;
            const bool real = i0 + lane < rows;
            if (!real) q = 0;
            const int ox = q / m, oy = q - ox * m;
            for (int w = 0; w * 64 < m; ++w) {
                const int n_oz = m - w * 64;
                const unsigned long long offsets = !real ? 0ull : n_oz >= 64 ? ~0ull : (1ull << n_oz) - 1ull;
                unsigned long long tried = 0;
                for (;;) {                            // until these rows have no offset left: each turn tries one
                    const int lost = __builtin_amdgcn_readfirstlane(psh_peek(fail));
                    unsigned long long room = offsets & ~tried;
                    for (int k0 = 0; k0 < c; k0 += 4) {
                        unsigned long long seen[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const uint32_t h = residue(min(k0 + k, c - 1));
                            const int x = wrap((int)(h & 255u) + ox), y = wrap((int)(h >> 8 & 255u) + oy);
                            seen[k] = psh_peek_row(taken + (int64_t)(x * m + y) * words, wrap((int)(h >> 16) + w * 64));
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k) room &= ~seen[k];
                        if (!__ballot(room != 0)) break;
                    }
                    if (lost) return;                 // the pair is lost anyway
                    const unsigned long long lanes = __ballot(room != 0);
                    if (!lanes) break;
                    // the first lane with room, and its first offset from a hashed one on: buckets keep apart
                    const int j = __builtin_ctzll(lanes);
                    const unsigned long long later = room >> bit0 << bit0;
                    const int fz = room ? __builtin_ctzll(later ? later : room) : 0;
                    const int cx = __builtin_amdgcn_readlane(ox, j), cy = __builtin_amdgcn_readlane(oy, j);
                    const int cz = w * 64 + __builtin_amdgcn_readlane(fz, j);
                    if (lane == j) tried |= 1ull << fz;
                    // every voxel's bit, 64 of them at a time
                    auto row_of = [&](uint32_t h) { return taken + (int64_t)(wrap((int)(h & 255u) + cx) * m + wrap((int)(h >> 8 & 255u) + cy)) * words; };
                    auto give_back = [&](uint32_t h) {
                        const int z = wrap((int)(h >> 16) + cz);
                        __hip_atomic_fetch_and(row_of(h) + (z >> 6), ~(1ull << (z & 63)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    };
                    int turn = 0;
                    bool all = true;
                    for (; turn * 64 < c && all; ++turn) {
                        const int k = turn * 64 + lane;
                        const uint32_t h = turn == 0 ? mine : residues[min(k, c - 1)];
                        const int z = wrap((int)(h >> 16) + cz);
                        bool got = false;
                        if (k < c) got = !(__hip_atomic_fetch_or(row_of(h) + (z >> 6), 1ull << (z & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> (z & 63) & 1ull);
                        if (__ballot(k < c && !got)) {
                            all = false;
                            if (got) give_back(h);
                        }
                    }
                    if (!all) {
                        for (int t = 0; t < turn - 1; ++t) give_back(residues[t * 64 + lane]);    // whole turns before the one that failed
                        raced = true;
                        if (!twins_checked) {         // two voxels of the bucket on one slot: no offset can separate them
                            twins_checked = true;
                            bool twins = false;
                            for (int k = lane; k - lane < c; k += 64) {
                                const uint32_t h = residues[min(k, c - 1)];
                                for (int e = 0; e < c; ++e) twins |= residue(e) == h && e < k && k < c;
                            }
                            if (__ballot(twins)) {
                                if (lane == 0) *fail = 1;
                                return;
                            }
                        }
                        continue;                     // and a fresh look at the rows: others have moved on
                    }
                    for (int k = lane; k < c; k += 64) {
                        const uint32_t h = residues[k];
                        const int x = wrap((int)(h & 255u) + cx), y = wrap((int)(h >> 8 & 255u) + cy), z = wrap((int)(h >> 16) + cz);
                        if (z < 63) __hip_atomic_fetch_or(row_of(h) + ((z + m) >> 6), 1ull << ((z + m) & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const int32_t v = members[k];
                        const int64_t e = (int64_t)(x * m + y) * m + z;
                        P.H[e] = v;
                        const int32_t *p = P.coords + 3 * (int64_t)v;
                        uint16_t *tag = P.T + 3 * e;
                        tag[0] = (uint16_t)p[0]; tag[1] = (uint16_t)p[1]; tag[2] = (uint16_t)p[2];
                    }
                    if (lane == 0) *phi4 = (uint32_t)cx | ((uint32_t)cy << 8) | ((uint32_t)cz << 16);
                    return;
                }
            }
        }
    }
    if (lane == 0) *fail = 1;
}

// Place the buckets of one class (2 voxels and more), a wavefront at a time each, as many wavefronts as are
// launched.  Bound by round trips: what other workgroups may change is read and claimed past the caches of the
// XCDs, 1 to 2 us each time.  Two things keep buckets out of each other's way: after a lost claim the rows are looked
// at anew (the offsets of the first look were gone one after the other, thousands of them: 3.2 ms for the
// buckets of 9 and more voxels of a 256^3 batch of 8, now 0.4), and no more wavefronts are launched than claim
// one slot in 48 at a time.  A whole build with 6 levels: 10.6 -> 7.2 ms; one slot in 190 and one in 6 measured the
// same there, 4 shapes of 745 000 voxels take 45 ms with one in 190, 40 with one in 48.
__global__ __launch_bounds__(256) void psh_place_kernel(
    const PairDesc *__restrict__ pairs, const int2 *__restrict__ cells, int n_buckets,
    const int32_t *__restrict__ cnt, const int32_t *__restrict__ first, const int32_t *__restrict__ members,
    const uint32_t *__restrict__ residues, unsigned long long *__restrict__ bits, uint32_t *__restrict__ phi4,
    int32_t *__restrict__ fail)
{
    for (int b = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6))); b < n_buckets; b += (int)gridDim.x * 4) {
        const int2 ag = cells[b];
        const PairDesc P = pairs[ag.x];
        const int cell = P.cell_base + ag.y, base = first[cell];
        psh_place_bucket(P, ag.y, cnt[cell], members + base, residues + base, bits + P.row_base, phi4 + cell, fail + P.pair_id);
    }
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
