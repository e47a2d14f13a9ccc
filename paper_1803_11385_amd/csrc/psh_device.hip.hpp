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

// ---- the same construction with the taken bits of a table in LDS ----
//
// A workgroup of 16 wavefronts does a whole attempt at one table: bucket sizes, member lists, buckets by size,
// the placing and the buckets of one voxel.  The bits of a table of side m <= PSH_LDS_SIDE are m^2 words of 8 bytes in LDS,
// four times, side by side in x and y so that a look need not wrap round, so that a look at a row and a claim take some 100 cycles instead of the 1 to 2 us of
// memory past the caches, and nothing of an attempt returns to the host.  What is left of the parallelism is enough:
// a batch has some 50 tables, and where the chip has room for it (SIDES_AT_ONCE in place_in_lds) each table's next
// two offset sides are tried beside the first one, which a third of the tables find too small.
//   * Bucket sizes are counted in LDS where the offset cells fit it (else in memory), and the count before a
//     voxel was added is its place in the bucket.
//   * 4 lanes per bucket, 16 buckets to a wavefront: a lane looks at one row, all offsets of it at once, and the residues
//     of the bucket's voxels go round by DPP.  64 lanes would look at 4096 offsets where the first few have room.
//   * Offsets only are kept; psh_emit_kernel evaluates h(p) with them and fills H and T, on the whole chip.
// Bound by what 16 wavefronts of one CU issue, on the few CUs that have the finest level's largest tables: the looks of the last
// buckets at hundreds of rows each.  See psh_build_kernel for what it measured.
constexpr int PSH_LDS_SIDE = 64, PSH_LDS_BYTES = 144 << 10;
constexpr int PSH_THREADS = 1024;

struct AttemptDesc {
    const int32_t *coords;   // [n][3] positions of this model at this level
    int32_t n, m, r;
    int32_t cell_base;       // first offset cell in the arrays of cells (r^3 each)
    int32_t vox_base;        // first entry in the arrays of voxels (n each)
};

// the value that lane K of the 4 neighbouring ones holds (DPP quad_perm)
template <int K> __device__ __forceinline__ uint32_t psh_lane_of_4(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, K * 0x55, 0xF, 0xF, true);
}

// Places the buckets [from, to) of the list, `at_once` at a time (`next` starts at from + 3 at_once).  Four lanes have one, 16 of them to a wavefront, and every four take
// the next entry by themselves (it is requested two buckets ahead and its residues one).  A bucket that found nothing in
// PSH_ALONE rows, or one of the last PSH_FEW of a wavefront, is searched by all its lanes, 64 rows at a time: near the end of a full
// table a bucket looks at hundreds of rows, and an attempt is lost with the first that has looked at all.
// Every turn of the loops finishes a bucket, moves on to other rows or has one offset less to try.
constexpr int PSH_ALONE = 64, PSH_FEW = 3;
__device__ __forceinline__ void psh_place_list(
    const uint4 *__restrict__ list, const uint32_t *__restrict__ residues, uint32_t *__restrict__ phi, int from, int to, int at_once, int m,
    unsigned char *lds, int32_t *next, volatile int32_t *failed)
{
    typedef unsigned long long Row;                                         // bit z: the slot is taken
    const int tid = threadIdx.x, lane = tid & 63, gl = lane & 3, group = lane & ~3, rows = m * m;
    Row *const bits = reinterpret_cast<Row *>(lds);
    const int pitch = 2 * m;                                                // a row has copies at x + m, y + m and both
    const Row offsets = m >= 64 ? ~(Row)0 : ((Row)1 << m) - 1;
    const float inv_m = 1.f / (float)m;
    auto wrap = [&](int v) { return v >= m ? v - m : v; };
    auto of_group = [&](bool pred) -> uint32_t { return (uint32_t)(__ballot(pred) >> group) & 15u; };
    auto entry = [&](int b) -> uint4 { return b < to ? list[b] : make_uint4(0u, 0u, 0u, 0u); };
    // lane k of the four has voxels k, k + 4, ... of the first 16; in place of those beyond the last the last one
    auto fetch = [&](const uint4 &e, uint32_t *v) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = e.y ? residues[e.x + min(gl + 4 * j, (int)e.y - 1)] : 0u;
    };
    // a residue as a look wants it: the row's place, z above it
    auto place_of = [&](uint32_t h) -> uint32_t { return ((h & 255u) * (uint32_t)pitch + (h >> 8 & 255u)) | (h & 0xFFFF0000u); };
    // the first `at_once` fours, of all wavefronts in turn
    const int mine_of = (tid >> 2 & 15) * (PSH_THREADS / 64) + (tid >> 6), b0 = mine_of < at_once ? from + mine_of : to;
    uint4 e = entry(b0), e1 = entry(b0 + at_once), e2 = entry(b0 + 2 * at_once);
    uint32_t mine[4], mine1[4], at[4];
    fetch(e, mine);
    fetch(e1, mine1);
    bool raced = false, twins_checked = false;
    int c = 0, start = 0, bit0 = 0, i0 = 0, pass = 0;
    Row tried = 0;
    auto begin = [&]() {
        const uint32_t hash = e.z * 2654435761u;
        start = (int)(hash % (uint32_t)rows);
        bit0 = (int)((hash >> 16) * (uint32_t)m >> 16);
        c = (int)e.y;
#pragma unroll
        for (int t = 0; t < 4; ++t) at[t] = place_of(mine[t]);
        i0 = pass = 0;
        tried = 0;
        raced = twins_checked = false;
    };
    begin();
    while (!__builtin_amdgcn_readfirstlane(*failed)) {                      // an attempt that is lost ends
        const bool busy = c > 0;
        if (!__ballot(busy)) break;
        const unsigned long long busy_lanes = __ballot(busy);
        const unsigned long long stuck_lanes = __ballot(busy && i0 >= PSH_ALONE);
        const bool few = stuck_lanes || __popcll(busy_lanes) <= 4 * PSH_FEW;               // then all lanes look for one of them
        const int served = __builtin_ctzll(stuck_lanes ? stuck_lanes : busy_lanes) & ~3;
        int ox = 0, oy = 0;
        Row room = 0;
        auto row = [&](int q, bool real) {
            if (q >= rows) q -= rows;
            if (!real) q = 0;
            ox = (int)(((float)q + 0.5f) * inv_m);
            oy = q - ox * m;
            room = real ? offsets : (Row)0;
        };
        auto look = [&](uint32_t h) {                 // of place_of
            const int z = (int)(h >> 16);
            const Row w = bits[(h & 0xFFFFu) + (uint32_t)(ox * pitch + oy)];
            room &= ~(w >> z | w << ((m - z) & 63));  // (a row of 64: for z = 0 the second shift is one by 0 as well)
        };
        // all rows looked at: an offset lost to another bucket that then gave its slots back is worth another look, a few times
        auto next_rows = [&](int by) -> bool {
            i0 += by;
            tried = 0;
            if (i0 < rows) return true;
            i0 = 0;
            const bool again = raced && ++pass < 4;
            raced = false;
            if (!again) *failed = 1;
            return again;
        };
        if (!few) {
            // until three quarters of the buckets have an offset, PSH_ALONE rows at most
            bool looking = busy;
            for (int t = 0; t < PSH_ALONE / 4; ++t) {
                if (looking) {
                    row(start + i0 + gl, i0 + gl < rows);
                    room &= ~tried;
#define HCH_PSH_LOOK(K) look(psh_lane_of_4<(K) & 3>(at[(K) / 4]))
#define HCH_PSH_LOOK4(K) if (__ballot((K) < c)) { HCH_PSH_LOOK(K); HCH_PSH_LOOK(K + 1); if (__ballot((K) + 2 < c)) { HCH_PSH_LOOK(K + 2); HCH_PSH_LOOK(K + 3); } }
                    HCH_PSH_LOOK4(0) HCH_PSH_LOOK4(4) HCH_PSH_LOOK4(8) HCH_PSH_LOOK4(12)
#undef HCH_PSH_LOOK4
#undef HCH_PSH_LOOK
                    for (int k = 16; __ballot(k < c); ++k) look(place_of(residues[e.x + min(k, c - 1)]));
                    looking = of_group(room != 0) == 0 && next_rows(4);
                }
                if (4 * __popcll(__ballot(looking)) <= __popcll(busy_lanes)) break;
            }
        } else {
            const int c_s = __builtin_amdgcn_readlane(c, served), start_s = __builtin_amdgcn_readlane(start, served);
            const int first = __builtin_amdgcn_readlane((int)e.x, served);
            int i_s = __builtin_amdgcn_readlane(i0, served);
            uint32_t h[4];                            // most of the buckets that come here have no more
#pragma unroll
            for (int k = 0; k < 4; ++k) h[k] = (uint32_t)__builtin_amdgcn_readlane((int)at[0], served + k);
            for (;;) {                                // at most rows / 64 turns
                row(start_s + i_s + lane, i_s + lane < rows);
                look(h[0]);
                if (c_s > 1) look(h[1]);
                if (c_s > 2) look(h[2]);
                if (c_s > 3) look(h[3]);
#pragma unroll
                for (int k = 4; k < 16; ++k)
                    if (k < c_s) look((uint32_t)__builtin_amdgcn_readlane((int)at[k / 4], served + k % 4));
                for (int k = 16; k < c_s && __ballot(room != 0); ++k) look(place_of(residues[first + k]));
                if (__ballot(room != 0)) break;
                i_s += 64;
                if (i_s >= rows) break;
            }
            if (group == served) {
                i0 = i_s;
                if (i0 >= rows) next_rows(0);
            }
        }
        const unsigned long long lanes = __ballot(room != 0), has = few ? lanes : lanes >> group & 15ull;
        const bool claims = busy && (!few || group == served) && has != 0;
        // the first lane with room, and its first offset from a hashed one on: buckets keep apart
        const int ahead = has ? __builtin_ctzll(has) : 0, j = few ? ahead : group + ahead;
        const Row later = room >> bit0 << bit0, pick = later ? later : room;
        const int fz = pick ? __builtin_ctzll(pick) : 0;
        const int offer = __shfl(ox | oy << 8 | fz << 16, j);
        const int cx = offer & 255, cy = offer >> 8 & 255, cz = offer >> 16;
        // every voxel's bit by a lane of its own
        auto row_of = [&](uint32_t h) -> Row * {
            return bits + wrap((int)(h & 255u) + cx) * pitch + wrap((int)(h >> 8 & 255u) + cy);
        };
        auto claim = [&](uint32_t h) -> bool {
            const int z = wrap((int)(h >> 16) + cz);
            return !(atomicOr(row_of(h), 1ull << z) >> z & 1ull);
        };
        auto give_back = [&](uint32_t h) {
            const int z = wrap((int)(h >> 16) + cz);
            atomicAnd(row_of(h), ~(1ull << z));
        };
        bool got[4], missed = false;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            got[t] = false;
            if (claims && gl + 4 * t < c) {
                got[t] = claim(mine[t]);
                missed |= !got[t];
            }
        }
        bool lost = of_group(missed) != 0;
        int beyond = 16;                              // voxels before this one are claimed, from the 17th on
        for (int k0 = 16; __ballot(claims && !lost && k0 < c); k0 += 4) {
            const bool part_of = claims && !lost && k0 + gl < c;
            const uint32_t h = part_of ? residues[e.x + k0 + gl] : 0u;
            const bool have = part_of && claim(h);
            if (of_group(part_of && !have)) {
                lost = true;
                if (have) give_back(h);
            } else if (!lost) beyond = k0 + 4;
        }
        if (claims && lost) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (got[t]) give_back(mine[t]);
            for (int k = 16 + gl; k < min(beyond, c); k += 4) give_back(residues[e.x + k]);
            raced = true;
            if (few) next_rows(ahead + 1);            // go on behind that row
            else if (lane == j) tried |= (Row)1 << cz;
            if (!twins_checked) {                     // two voxels of the bucket on one slot: no offset can separate them
                twins_checked = true;
                bool twins = false;
                for (int k = gl; k < c; k += 4)
                    for (int f = 0; f < k; ++f) twins |= residues[e.x + k] == residues[e.x + f];
                if (twins) *failed = 1;
            }
        } else if (claims) {
            if (gl == 0) phi[e.z] = (uint32_t)offer;
            for (int k = gl; k < c; k += 4) {         // and the copies
                const uint32_t h = residues[e.x + k];
                const Row bit = 1ull << wrap((int)(h >> 16) + cz);
                Row *const row_at = row_of(h);
                atomicOr(row_at + m, bit);
                atomicOr(row_at + m * pitch, bit);
                atomicOr(row_at + m * pitch + m, bit);
            }
            e = e1; e1 = e2;
#pragma unroll
            for (int t = 0; t < 4; ++t) mine[t] = mine1[t];
            fetch(e1, mine1);
            int b = 0;
            if (gl == 0) b = atomicAdd(next, 1);
            e2 = entry(__shfl(b, group));
            begin();
        }
    }
}

// v mod d for 0 <= v < 2^15: the quotient from the reciprocal is exact or one off
__device__ __forceinline__ int psh_mod(int v, int d, float inv)
{
    const int q = v - (int)((float)v * inv) * d;
    return q < 0 ? q + d : q >= d ? q - d : q;
}

// One attempt at one table per workgroup; `ok` receives 1 where every bucket found its place.  cells: cnt, first
// and phi [cells], list [cells]; voxels: rank and residues.  Dynamic LDS: the larger of the bits and, up to
// PSH_LDS_BYTES, 4 bytes per offset cell.
// Every wait ends: a turn of the placing loop finishes the bucket, moves on to other rows or has one offset less to try.
// 256^3, batch of 8, 6 levels, 609 000 voxels: 1.1 ms for all tables, three sides tried at once (an attempt that succeeds at its
// second side 0.3, the ones that just succeed or fail at the first up to 1.1), where the launches over memory (psh_place_kernel
// and those around it) took 1.9 ms in two rounds with the host between them.
__global__ __launch_bounds__(PSH_THREADS) void psh_build_kernel(
    const AttemptDesc *__restrict__ attempts, int32_t *__restrict__ cnt_mem, int32_t *__restrict__ first_mem, uint32_t *__restrict__ phi_mem,
    uint4 *__restrict__ list_mem, int32_t *__restrict__ rank_mem, uint32_t *__restrict__ residue_mem, int32_t *__restrict__ ok, int lds_bytes)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ int32_t part[PSH_THREADS / 64], hist[PSH_CLASSES], cursor[PSH_CLASSES], next, failed;
    const AttemptDesc P = attempts[blockIdx.x];
    const int tid = threadIdx.x, n = P.n, m = P.m, r = P.r, cells = r * r * r;
    int32_t *rank = rank_mem + P.vox_base;
    uint32_t *residues = residue_mem + P.vox_base, *phi = phi_mem + P.cell_base;
    uint4 *list = list_mem + P.cell_base;
    const bool in_lds = (int64_t)cells * 4 <= lds_bytes;
    int32_t *cnt_l = reinterpret_cast<int32_t *>(lds), *cnt_g = cnt_mem + P.cell_base, *first_g = first_mem + P.cell_base;

    // ---- bucket sizes
    if (tid < PSH_CLASSES) hist[tid] = 0;
    if (tid == 0) failed = 0;
    for (int g = tid; g < cells; g += PSH_THREADS) {
        if (in_lds) cnt_l[g] = 0;
        else __hip_atomic_store(cnt_g + g, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const float inv_r = 1.f / (float)r, inv_m = 1.f / (float)m;
    auto bucket = [&](const int32_t *p) -> int { return (psh_mod(p[0], r, inv_r) * r + psh_mod(p[1], r, inv_r)) * r + psh_mod(p[2], r, inv_r); };
#pragma unroll 4
    for (int i = tid; i < n; i += PSH_THREADS) {
        const int g = bucket(P.coords + 3 * (int64_t)i);
        rank[i] = in_lds ? atomicAdd(cnt_l + g, 1) : __hip_atomic_fetch_add(cnt_g + g, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    // ---- first entries: thread t adds up its stretch of cells, then walks it again
    const int per = (cells + PSH_THREADS - 1) / PSH_THREADS, g0 = min(tid * per, cells), g1 = min(g0 + per, cells);
    auto count = [&](int g) -> int32_t { return in_lds ? cnt_l[g] : __hip_atomic_load(cnt_g + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto class_of = [](int c) -> int { return min(c, PSH_CLASSES - 1); };
    int32_t s = 0, all;
    for (int g = g0; g < g1; ++g) {
        const int c = count(g);
        s += c;
        if (c) atomicAdd(&hist[class_of(c)], 1);
    }
    int32_t at = block_scan(s, part, &all);
    __syncthreads();
    if (tid == 0)
        for (int k = PSH_CLASSES - 1, q = 0; k >= 1; --k) { cursor[k] = q; q += hist[k]; }     // largest first
    __syncthreads();
    const int n_single = hist[1], n_multi = cursor[1];
    __syncthreads();
    for (int g = g0; g < g1; ++g) {
        const int c = count(g);
        if (c) list[atomicAdd(&cursor[class_of(c)], 1)] = make_uint4((uint32_t)at, (uint32_t)c, (uint32_t)g, 0u);
        if (in_lds) cnt_l[g] = at; else first_g[g] = at;
        at += c;
    }
    __syncthreads();
    // ---- members' residues modulo m, packed x | y << 8 | z << 16, bucket by bucket
#pragma unroll 4
    for (int i = tid; i < n; i += PSH_THREADS) {
        const int32_t *p = P.coords + 3 * (int64_t)i;
        const int g = bucket(p);
        residues[(in_lds ? cnt_l[g] : first_g[g]) + rank[i]] =
            (uint32_t)psh_mod(p[0], m, inv_m) | (uint32_t)psh_mod(p[1], m, inv_m) << 8 | (uint32_t)psh_mod(p[2], m, inv_m) << 16;
    }
    __syncthreads();
    // ---- bits of taken slots
    const int rows = m * m, pitch = 2 * m;
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(lds);
    for (int q = tid; q < 4 * rows; q += PSH_THREADS) bits[q] = 0ull;
    __syncthreads();

    // one size after the other, largest first, and no more at a time than claim one slot in 48 (or tables come out with
    // larger sides: with all of them and all sizes at once hardly a first side was enough, see psh_place_kernel)
    for (int k = PSH_CLASSES - 1, from = 0; k >= 2; --k) {
        const int to = from + hist[k], at_once = min(max(rows * m / (48 * k), 1), PSH_THREADS / 4);
        if (tid == 0) next = from + 3 * at_once;
        __syncthreads();
        psh_place_list(list, residues, phi, from, to, at_once, m, lds, &next, &failed);
        __syncthreads();
        from = to;
    }
    __syncthreads();
    if (failed) {
        if (tid == 0) ok[blockIdx.x] = 0;
        return;
    }
    // ---- buckets of one voxel: the i-th takes the i-th free slot
    const unsigned long long offsets = m >= 64 ? ~0ull : (1ull << m) - 1ull;
    const int rper = (rows + PSH_THREADS - 1) / PSH_THREADS, q0 = min(tid * rper, rows), q1 = min(q0 + rper, rows);
    int32_t n_free = 0;
    for (int q = q0; q < q1; ++q) n_free += __popcll(~bits[q / m * pitch + q % m] & offsets);
    int i = block_scan(n_free, part, &all);       // m^3 > n: there are enough
    for (int q = q0; q < q1 && i < n_single; ++q)
        for (unsigned long long vacant = ~bits[q / m * pitch + q % m] & offsets; vacant && i < n_single; vacant &= vacant - 1ull, ++i) {
            const uint4 e = list[n_multi + i];
            const uint32_t h = residues[e.x];
            int px = q / m - (int)(h & 255u), py = q % m - (int)(h >> 8 & 255u), pz = __builtin_ctzll(vacant) - (int)(h >> 16);
            px += px < 0 ? m : 0; py += py < 0 ? m : 0; pz += pz < 0 ? m : 0;
            phi[e.z] = (uint32_t)px | ((uint32_t)py << 8) | ((uint32_t)pz << 16);
        }
    if (tid == 0) ok[blockIdx.x] = 1;
}

// What a table is written from: its offset words, and where its parts lie.
struct PackDesc {
    const int32_t *coords;    // [n][3] positions
    const uint32_t *phi_src;  // the offset words of its successful attempt
    int32_t *H;               // the parts of the level's super tables
    uint16_t *T;
    uint32_t *slot3, *phi4;
    int32_t *V;
    uint8_t *Phi;
    int32_t n, m, r, model;
};

// H and T from the offsets (Eq.1), for tables of psh_build_kernel.  grid.y = table.
__global__ __launch_bounds__(256) void psh_emit_kernel(const PackDesc *__restrict__ desc)
{
    const PackDesc D = desc[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= D.n) return;
    const int32_t *p = D.coords + 3 * (int64_t)i;
    const int x = p[0], y = p[1], z = p[2], m = D.m, r = D.r;
    const uint32_t w = D.phi_src[((x % r) * r + (y % r)) * r + (z % r)];
    const int e = (((x % m + (int)(w & 255u)) % m) * m + (y % m + (int)(w >> 8 & 255u)) % m) * m + (z % m + (int)(w >> 16)) % m;
    D.H[e] = i;
    uint16_t *tag = D.T + 3 * (int64_t)e;
    tag[0] = (uint16_t)x; tag[1] = (uint16_t)y; tag[2] = (uint16_t)z;
}

// Packed lookup records, model indices and byte offset tables from H, T and the offset words.  grid.y = table.
__global__ __launch_bounds__(256) void psh_pack_kernel(const PackDesc *__restrict__ desc)
{
    const PackDesc D = desc[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < D.m * D.m * D.m) {
        D.slot3[SLOT_WORDS * (int64_t)i + 0] = (uint32_t)D.H[i];
        D.slot3[SLOT_WORDS * (int64_t)i + 1] = (uint32_t)D.T[3 * (int64_t)i] | ((uint32_t)D.T[3 * (int64_t)i + 1] << 16);
        D.slot3[SLOT_WORDS * (int64_t)i + 2] = (uint32_t)D.T[3 * (int64_t)i + 2];
        if (SLOT_WORDS > 3) D.slot3[SLOT_WORDS * (int64_t)i + 3] = 0u;
        D.V[i] = D.model;
    }
    if (i < D.r * D.r * D.r) {
        const uint32_t w = D.phi_src[i];
        D.phi4[i] = w;
        D.Phi[3 * (int64_t)i + 0] = (uint8_t)(w & 255u); D.Phi[3 * (int64_t)i + 1] = (uint8_t)((w >> 8) & 255u); D.Phi[3 * (int64_t)i + 2] = (uint8_t)((w >> 16) & 255u);
    }
}

}  // namespace hch
