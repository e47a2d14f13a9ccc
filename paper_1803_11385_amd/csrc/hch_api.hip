// C ABI of the hch library: host logic, table upload and kernel launches.
#include "../../include/hch.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "kernels.hip.hpp"
#include "direct.hip.hpp"
#include "gemm_bf16.hip.hpp"
#include "split_wgrad.hip.hpp"
#include "split_conv.hip.hpp"
#include "conv_small.hip.hpp"
#include "split_columns.hip.hpp"
#include "split_dcol.hip.hpp"
#include "split_field.hip.hpp"
#include "conv_bf16.hip.hpp"
#include "psh_device.hip.hpp"
#include "occupancy.hip.hpp"
#include "profile.hpp"
#include "psh_build.hpp"

// Every kernel launch of the library: carries the two timing events of the enclosing LaunchTimer,
// if there is one and timing is on; an ordinary launch otherwise.
#define HCH_LAUNCH(kernel, grid, block, lds, stream, ...)                                          \
    do {                                                                                           \
        hipEvent_t ev_a_ = hch::tls_start_event, ev_b_ = hch::tls_stop_event;                      \
        hch::tls_start_event = hch::tls_stop_event = nullptr;                                      \
        if (ev_a_) hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, ev_a_, ev_b_, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);                    \
    } while (0)

namespace {

thread_local std::string g_err;

hch_status fail(hch_status st, const std::string &msg)
{
    g_err = msg;
    return st;
}

// Every allocation of the library on the device.  The runtime keeps a failed one as its last error over later calls that
// succeed; taken back here, or the next HCH_LAUNCH_CHECK, of this call or of another one, would report it as its own.
hipError_t device_malloc(void **p, size_t bytes)
{
    const hipError_t e = hipMalloc(p, bytes ? bytes : 16);
    if (e != hipSuccess) { *p = nullptr; (void)hipGetLastError(); }
    return e;
}

#define HCH_HIP(call)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (call);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(HCH_EHIP, std::string(#call) + ": " + hipGetErrorString(e_));      \
    } while (0)

#define HCH_LAUNCH_CHECK(name)                                                             \
    do {                                                                                   \
        hipError_t e_ = hipGetLastError();                                                 \
        if (e_ != hipSuccess)                                                              \
            return fail(HCH_EHIP, std::string("launch ") + name + ": " + hipGetErrorString(e_)); \
    } while (0)

// One level of the super-PSH, host and device side.
struct Level {
    int32_t ubar = 0, b = 0;
    int32_t ratio = 1;                         // side of the next finer level / side of this one (1 at level 0)
    int64_t n_total = 0, m_total = 0, r_total = 0;
    int32_t max_n = 0;                         // largest model of the level
    int64_t nbr_valid = 0;                     // occupied entries of nbr27 (incl. the centre)
    std::vector<int32_t> mbar, rbar, attempts, coords;
    std::vector<int64_t> M, R, N;
    std::vector<int32_t> H, V;                 // host copies of the super tables
    std::vector<uint16_t> T;
    std::vector<uint8_t> Phi;
    // ... and where the host copies are in hch_levels' own blocks instead (tables built on the device)
    const int32_t *hH = nullptr, *hV = nullptr, *hcoords = nullptr;
    const uint16_t *hT = nullptr;
    const uint8_t *hPhi = nullptr;
    // device
    bool in_block = false;                     // tables and lists lie in blocks of the whole level set
    int32_t *dH = nullptr, *dV = nullptr, *dcoords = nullptr, *dnbr = nullptr, *dchild = nullptr;
    int32_t *dnbr_t = nullptr;                 // tap-major copy of dnbr ([27][n_total]), built on request
    uint32_t *dmask27 = nullptr;               // [n_total] bit k: neighbour k exists
    uint32_t *dtilemask = nullptr;             // [ceil(n_total/64)] taps present in each tile of the pattern order
    const int32_t *dorder = nullptr;           // [n_total] the level's voxels in pattern order (into hch_levels' sort output)
    const int32_t *dforder = nullptr;          // the same in the fine order, and its tiles' taps; null on small levels
    uint32_t *dftilemask = nullptr;
    const int32_t *rows() const { return dforder ? dforder : dorder; }            // the order the products walk
    const uint32_t *row_taps() const { return dforder ? dftilemask : dtilemask; }
    uint16_t *dT = nullptr;
    uint8_t *dPhi = nullptr;
    uint32_t *dslot3 = nullptr, *dphi4 = nullptr;   // packed copies of H*,T* and Phi* for the lookups
    int32_t *dmeta = nullptr;                  // mbar[b] rbar[b] M[b+1] R[b+1] N[b+1] as int32

    hch::PshView view() const
    {
        hch::PshView v;
        v.slot3 = dslot3; v.phi4 = dphi4;
        v.mbar = dmeta; v.rbar = dmeta + b; v.M = dmeta + 2 * b; v.R = dmeta + 3 * b + 1;
        v.N = dmeta + 4 * b + 2; v.ubar = ubar;
        return v;
    }
    const int32_t *dN() const { return dmeta + 4 * b + 2; }
};

void free_level(Level &L)
{
    if (L.in_block) {                          // everything but the tap-major copy belongs to hch_levels::blocks
        void *own = L.dnbr_t;
        L = Level();
        if (own) (void)hipFree(own);
        return;
    }
    void *ptrs[] = {L.dH, L.dV, L.dcoords, L.dnbr, L.dchild, L.dT, L.dPhi, L.dmeta, L.dslot3, L.dphi4, L.dnbr_t, L.dmask27, L.dtilemask};
    for (void *p : ptrs) if (p) (void)hipFree(p);
    L.dH = L.dV = L.dcoords = L.dnbr = L.dchild = L.dmeta = L.dnbr_t = nullptr;
    L.dmask27 = L.dtilemask = L.dftilemask = nullptr; L.dorder = L.dforder = nullptr;
    L.dT = nullptr; L.dPhi = nullptr; L.dslot3 = L.dphi4 = nullptr;
}

inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Host memory that the device copies into (tables built there, for hch_level_info).  Copies into ordinary memory go by pieces through a buffer of the
// runtime's and a copy by the host: builds of a 256^3 batch of 8 (17 MB) one after the other 3.3 ms, with pinned memory 2.7, of a 64^3 batch of 32
// 1.04 and 0.94.  Making such a block costs what it saves the first time (twenty level sets that stay 6.2 ms each either way; the first build of a
// single model of 90 000 voxels 2.5 and 2.0), so blocks of level sets that are gone are kept for the next ones: HOST_KEPT bytes at most, the longest
// unused given back first.  In use and kept there are HOST_PINNED bytes at most; beyond that, for more than HOST_KEPT at once (192 MB in each build
// 33.4 ms, ordinary 32.4) and where the runtime has no pinned memory it is ordinary memory.  By any thread: a block has one owner, whose copies are
// over before it is freed.
constexpr size_t HOST_KEPT = (size_t)128 << 20, HOST_PINNED = 2 * HOST_KEPT, HOST_STEP = (size_t)256 << 10;

class HostBlocks {
    struct Block { char *p; size_t bytes; };
    std::mutex mu;
    std::vector<Block> kept;                   // longest unused first
    size_t held = 0, pinned = 0;               // bytes kept; of all pinned blocks
    void unpin(const Block &b)
    {
        (void)hipHostFree(b.p);
        std::lock_guard<std::mutex> lock(mu);
        pinned -= b.bytes;
    }
public:
    static HostBlocks &get() { static HostBlocks *const all = new HostBlocks; return *all; }      // outlives every level set
    char *take(size_t *bytes)                  // null: ordinary memory will do
    {
        *bytes = round_up(*bytes, HOST_STEP);
        {
            std::lock_guard<std::mutex> lock(mu);
            size_t best = kept.size();
            for (size_t i = 0; i < kept.size(); ++i)
                if (kept[i].bytes >= *bytes && kept[i].bytes <= 4 * *bytes && (best == kept.size() || kept[i].bytes < kept[best].bytes)) best = i;
            if (best < kept.size()) {
                char *p = kept[best].p;
                *bytes = kept[best].bytes;
                held -= *bytes;
                kept.erase(kept.begin() + (std::ptrdiff_t)best);
                return p;
            }
            if (*bytes > HOST_KEPT || pinned + *bytes > HOST_PINNED) return nullptr;
            pinned += *bytes;
        }
        void *p = nullptr;
        if (hipHostMalloc(&p, *bytes, hipHostMallocPortable) == hipSuccess) return (char *)p;
        (void)hipGetLastError();
        std::lock_guard<std::mutex> lock(mu);
        pinned -= *bytes;
        return nullptr;
    }
    void keep(char *p, size_t bytes)
    {
        Block out{nullptr, 0};
        {
            std::lock_guard<std::mutex> lock(mu);
            try {
                kept.push_back(Block{p, bytes});
                held += bytes;
            } catch (const std::bad_alloc &) {
                out = Block{p, bytes};
            }
        }
        if (out.p) unpin(out);
        for (;;) {                             // (the runtime takes its time over a block: not while others wait)
            {
                std::lock_guard<std::mutex> lock(mu);
                if (held <= HOST_KEPT) return;
                out = kept.front();
                held -= out.bytes;
                kept.erase(kept.begin());
            }
            unpin(out);
        }
    }
};

class HostBlock {
    char *p = nullptr;
    size_t bytes = 0;
    std::unique_ptr<char[]> ordinary;
public:
    HostBlock() = default;
    HostBlock(const HostBlock &) = delete;
    HostBlock &operator=(const HostBlock &) = delete;
    ~HostBlock() { if (p) HostBlocks::get().keep(p, bytes); }
    char *get() const { return p ? p : ordinary.get(); }
    bool pinned() const { return p != nullptr; }
    void make(size_t n)                        // once
    {
        bytes = std::max<size_t>(n, 1);
        p = HostBlocks::get().take(&bytes);
        if (!p) ordinary.reset(new char[n]);
    }
};

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline unsigned blocks_for(int64_t items) { return (unsigned)((items + 255) / 256); }

// levels with a fine order (see corner_key): below, what it saves no longer pays for its launches
constexpr int64_t FINE_MIN_VOXELS = 32768;
static_assert(hch::PATTERN_SMALL < FINE_MIN_VOXELS, "pattern_small_kernel makes no fine order");
constexpr int64_t MAX_GRID_ITEMS = (int64_t)2147483647 * 256;   // grid.x limit * block size

}  // namespace

struct hch_levels {
    std::vector<Level> lv;
    // one-launch index-list kernels: all levels as a kernel argument, and the tile prefix
    // arrays (host copy + device) of the neighbour and child kernels
    hch::LevelSet set{};
    std::vector<int32_t> nbr_prefix, child_prefix;
    int32_t *d_nbr_prefix = nullptr, *d_child_prefix = nullptr;
    // pattern order of every level's voxels (level l at sort_off[l]): keys and tile histograms
    // written by the neighbour kernel, the sorted data indices
    std::vector<int32_t> sort_off;
    uint8_t *d_sort_key = nullptr;
    int32_t *d_tile_hist = nullptr, *d_key_total = nullptr, *d_order = nullptr;
    uint32_t *d_fine = nullptr;                // everything of the fine order, in one allocation
    std::vector<void *> blocks;                // allocations: the orders and prefixes; device construction: what is known before it, and after
    HostBlock host_block, host_phi;            // its host copies: positions, H*, T*, V*; offset tables
};

extern "C" const char *hch_last_error(void) { return g_err.c_str(); }

extern "C" void hch_free_levels(hch_levels *levels)
{
    if (!levels) return;
    for (Level &L : levels->lv) free_level(L);
    for (void *p : levels->blocks) (void)hipFree(p);
    delete levels;
}

extern "C" int32_t hch_num_levels(const hch_levels *levels)
{
    return levels ? (int32_t)levels->lv.size() : 0;
}

// ---------------------------------------------------------------------------------------
// build
// ---------------------------------------------------------------------------------------

static hch_status upload(void **dst, const void *src, size_t bytes, hipStream_t s)
{
    const hipError_t e = device_malloc(dst, bytes);
    if (e != hipSuccess) return fail(HCH_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    if (bytes) HCH_HIP(hipMemcpyAsync(*dst, src, bytes, hipMemcpyHostToDevice, s));
    return HCH_OK;
}

// dnbr_t[t][i] = dnbr[i][t], if the level has the copy
static hch_status transpose_neighbours(const Level &L, hipStream_t s)
{
    if (!L.dnbr_t || L.n_total == 0) return HCH_OK;
    hch::LaunchTimer lt(HCH_KERNEL_ID("index_transpose_kernel"), s, 216.0 * (double)L.n_total, 0.0);
    HCH_LAUNCH(hch::index_transpose_kernel, dim3(blocks_for(L.n_total)), dim3(256), 0, s, L.dnbr, L.dnbr_t, L.n_total, 27);
    HCH_LAUNCH_CHECK("index_transpose_kernel");
    return HCH_OK;
}

// index lists of levels [l0, l1) in one launch
// (orders: and the row orders of the fused products)
static hch_status launch_index_lists(const hch_levels *hl, int l0, int l1, hipStream_t s, bool orders = true)
{
    const int b = hl->lv[0].b;
    const int n_entries = (int)hl->lv.size() * b;
    {
        const int first = hl->nbr_prefix[(size_t)l0 * b], last = hl->nbr_prefix[(size_t)l1 * b];
        if (last > first) {
            double bytes = 0.0;   // per voxel: its position in, 27 indices out; the level's tables once
            for (int l = l0; l < l1; ++l)
                bytes += (double)hl->lv[l].n_total * 120.0 + (double)hl->lv[l].m_total * 10.0 + (double)hl->lv[l].r_total * 3.0;
            // per coarse voxel: position in, 8 indices out; the finer tables once
            for (int l = std::max(l0, 1); l < l1; ++l)
                if (hl->lv[l].ratio == 2) bytes += (double)hl->lv[l].n_total * 44.0 + (double)hl->lv[l - 1].m_total * 10.0 + (double)hl->lv[l - 1].r_total * 3.0;
            const int child_first = hl->child_prefix[(size_t)l0 * b];
            const unsigned n_tiles = (unsigned)(last - first), n_child = (unsigned)(hl->child_prefix[(size_t)l1 * b] - child_first);
            const unsigned nbr_grid = (n_tiles + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD;
            const unsigned grid = nbr_grid + (n_child + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD;
            hch::LaunchTimer lt(HCH_KERNEL_ID("neighbour_kernel"), s, bytes, 0.0);
            HCH_LAUNCH(hch::neighbour_kernel, dim3(grid), dim3(256), 0, s, hl->set, hl->d_nbr_prefix,
                               n_entries, first, n_tiles, nbr_grid, hl->d_child_prefix, child_first, n_child);
        }
        HCH_LAUNCH_CHECK("neighbour_kernel");
        for (int l = l0; l < l1; ++l) {            // keep the tap-major copies in step
            hch_status st = transpose_neighbours(hl->lv[l], s);
            if (st != HCH_OK) return st;
        }
        // pattern order of the levels' voxels (stable counting sort by pattern key), then the tap
        // masks of its 64-row tiles
        const int64_t cnt = (int64_t)hl->sort_off[l1] - hl->sort_off[l0];
        int64_t most = 0;
        for (int l = l0; l < l1; ++l) most = std::max(most, hl->lv[l].n_total);
        if (orders && cnt > 0 && most <= hch::PATTERN_SMALL) {
            hch::PatternSmallArgs A{};
            for (int l = l0; l < l1; ++l) A.tile_mask[l] = hl->lv[l].dtilemask;
            hch::LaunchTimer lt(HCH_KERNEL_ID("pattern_small_kernel"), s, 17.0 * (double)cnt, 0.0);
            HCH_LAUNCH(hch::pattern_small_kernel, dim3((unsigned)(l1 - l0)), dim3(1024), 0, s, hl->set, A, l0, hl->d_order);
            HCH_LAUNCH_CHECK("pattern_small_kernel");
        } else if (orders && cnt > 0) {
            {
                hch::LaunchTimer lt(HCH_KERNEL_ID("pattern_scan_kernel"), s, 8.0 * 64.0 * (double)(last - first), 0.0);
                HCH_LAUNCH(hch::pattern_scan_kernel, dim3(hch::PATTERN_BINS, (unsigned)(l1 - l0)), dim3(256), 0, s, hl->set,
                           hl->d_key_total, l0);
            }
            HCH_LAUNCH_CHECK("pattern_scan_kernel");
            {
                hch::LaunchTimer lt(HCH_KERNEL_ID("pattern_scatter_kernel"), s, 5.0 * (double)cnt, 0.0);
                HCH_LAUNCH(hch::pattern_scatter_kernel, dim3((unsigned)(last - first)), dim3(256), 0, s, hl->set,
                           hl->d_nbr_prefix, n_entries, first, (unsigned)(last - first), hl->d_key_total, hl->d_order);
            }
            HCH_LAUNCH_CHECK("pattern_scatter_kernel");
            hch::TileMaskArgs A{}, F{};           // tile masks of the pattern order, of the fine order
            A.n_levels = F.n_levels = l1 - l0;
            int fine_most = 0;
            for (int l = l0; l < l1; ++l) {
                const Level &L = hl->lv[l];
                const int q = l - l0, stretches = (int)((L.n_total + hch::FINE_TILE - 1) / hch::FINE_TILE);
                A.tile_mask[q] = L.dtilemask; F.tile_mask[q] = L.dftilemask;
                A.off[q] = F.off[q] = hl->sort_off[l];
                A.n[q] = F.n[q] = (int32_t)L.n_total;
                A.hist_off[q] = hl->set.fine_off[l]; A.hist_tiles[q] = hl->set.fine_tiles[l];
                A.tile_prefix[q + 1] = A.tile_prefix[q] + stretches;
                F.tile_prefix[q + 1] = F.tile_prefix[q] + (L.dforder ? stretches : 0);
                fine_most = std::max(fine_most, hl->set.fine_tiles[l]);
            }
            {
                hch::LaunchTimer lt(HCH_KERNEL_ID("tile_mask_kernel<true>"), s, 4.0 * (double)cnt, 0.0);
                HCH_LAUNCH(hch::tile_mask_kernel<true>, dim3((unsigned)A.tile_prefix[A.n_levels]), dim3(256), 0, s, A,
                           (const uint32_t *)hl->set.sorted_mask, hl->set.fine_hist);
            }
            HCH_LAUNCH_CHECK("tile_mask_kernel");
            if (fine_most > 0) {
                {
                    hch::LaunchTimer lt(HCH_KERNEL_ID("fine_scan_kernel"), s, 8.0 * hch::FINE_BINS * F.tile_prefix[F.n_levels], 0.0);
                    HCH_LAUNCH(hch::fine_scan_kernel, dim3(hch::FINE_BINS, (unsigned)(l1 - l0)), dim3(256), 0, s, hl->set, l0);
                }
                HCH_LAUNCH_CHECK("fine_scan_kernel");
                {
                    hch::LaunchTimer lt(HCH_KERNEL_ID("fine_scatter_kernel"), s, 16.0 * (double)cnt, 0.0);
                    HCH_LAUNCH(hch::fine_scatter_kernel, dim3((unsigned)fine_most, (unsigned)(l1 - l0)), dim3(256), 0, s, hl->set,
                               (const int32_t *)hl->d_order, l0);
                }
                HCH_LAUNCH_CHECK("fine_scatter_kernel");
                hch::LaunchTimer lt(HCH_KERNEL_ID("tile_mask_kernel<false>"), s, 4.0 * (double)cnt, 0.0);
                HCH_LAUNCH(hch::tile_mask_kernel<false>, dim3((unsigned)F.tile_prefix[F.n_levels]), dim3(256), 0, s, F,
                           (const uint32_t *)hl->set.fine_mask, (int32_t *)nullptr);
            }
            HCH_LAUNCH_CHECK("tile_mask_kernel");
        }
    }
    return HCH_OK;
}

extern "C" hch_status hch_build_neighbours(hch_levels *levels, int32_t level, void *stream)
{
    if (!levels || level < -1 || level >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_build_neighbours: bad level");
    if (!levels->d_nbr_prefix) return fail(HCH_EINVAL, "hch_build_neighbours: levels were built without device tables");
    if (level < 0) return launch_index_lists(levels, 0, (int)levels->lv.size(), (hipStream_t)stream);
    return launch_index_lists(levels, level, level + 1, (hipStream_t)stream);
}

extern "C" hch_status hch_build_tap_major(hch_levels *levels, int32_t level, void *stream)
{
    if (!levels || level < -1 || level >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_build_tap_major: bad level");
    if (!levels->d_nbr_prefix) return fail(HCH_EINVAL, "hch_build_tap_major: levels were built without device tables");
    const int l0 = level < 0 ? 0 : level, l1 = level < 0 ? (int)levels->lv.size() : level + 1;
    for (int l = l0; l < l1; ++l) {
        Level &L = levels->lv[l];
        if (!L.dnbr_t && L.n_total > 0 && device_malloc((void **)&L.dnbr_t, (size_t)L.n_total * 27 * 4) != hipSuccess)
            return fail(HCH_ENOMEM, "hch_build_tap_major: hipMalloc failed");
        hch_status st = transpose_neighbours(L, (hipStream_t)stream);
        if (st != HCH_OK) return st;
    }
    return HCH_OK;
}

extern "C" hch_status hch_build_neighbours_range(hch_levels *levels, int32_t first, int32_t count, void *stream)
{
    if (!levels || first < 0 || count < 0 || (int64_t)first + count > (int64_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_build_neighbours_range: bad level range");
    if (!levels->d_nbr_prefix) return fail(HCH_EINVAL, "hch_build_neighbours_range: levels were built without device tables");
    if (count == 0) return HCH_OK;
    return launch_index_lists(levels, first, first + count, (hipStream_t)stream);
}

extern "C" hch_status hch_build_index_lists(hch_levels *levels, int32_t first, int32_t count, void *stream)
{
    if (!levels || first < 0 || count < 0 || (int64_t)first + count > (int64_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_build_index_lists: bad level range");
    if (!levels->d_nbr_prefix) return fail(HCH_EINVAL, "hch_build_index_lists: levels were built without device tables");
    if (count == 0) return HCH_OK;
    return launch_index_lists(levels, first, first + count, (hipStream_t)stream, false);
}

// ---- PSH construction on the device (psh_device.hip.hpp) ----

namespace {
// Device memory by the piece, 256-byte aligned, out of one allocation: sized first (null base), then
// handed out in the same order.
struct Pieces {
    char *base = nullptr;
    size_t used = 0;
    template <typename T> void take(T *&p, size_t bytes)
    {
        if (base) p = reinterpret_cast<T *>(base + used);
        used += round_up(std::max<size_t>(bytes, 16), 256);
    }
};
struct DeviceBlocks {            // device allocations that live until the end of the build call, unless released before
    std::vector<void *> ptrs;
    ~DeviceBlocks() { release(); }
    void release()
    {
        for (void *p : ptrs) (void)hipFree(p);
        ptrs.clear();
    }
    hipError_t try_get(void **out, size_t bytes)
    {
        const hipError_t e = device_malloc(out, bytes);
        if (e == hipSuccess) ptrs.push_back(*out);
        return e;
    }
    hch_status get(void **out, size_t bytes)
    {
        const hipError_t e = try_get(out, bytes);
        return e == hipSuccess ? HCH_OK : fail(HCH_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
};
// Occupancy of the levels on the device (occupancy.hip.hpp), between the checks and the tables
struct Occupancy {
    DeviceBlocks mem;
    hch::OccupancySet set{};
    const int32_t *host_coords = nullptr;      // the caller's
    int32_t *d_coords = nullptr, *d_sums = nullptr, *d_first = nullptr;
    unsigned long long *d_bits = nullptr;
    std::vector<int32_t> first;
    bool ready = false;
};
struct PairWork {
    int l, v;
    int32_t n, m, r, attempts;
    const uint32_t *phi;         // offset words of the successful attempt (device)
    bool done;
};
}  // namespace

// Checks the positions and fills ubar, ratio, b, N, n_total and max_n of every level on the device; the
// coarse levels' voxels stay a bit set until device_construct lists them.  On the host the checks and the coarse
// levels were 3.4 ms of a 256^3 batch of 8.  Not `ready` where a bit per position is too much memory, altogether or for the
// few voxels there are: the host does it then.  Clearing and reading the bits costs 2.5 us a MB, the host 50 to 90 ns a voxel
// of one model and, from a few models on, its threads.  Whole builds, device and host: 1024^3, one model (153 MB), 300 voxels
// 1.23 and 0.71 ms, 4000 1.85 and 1.65, 8000 2.26 and 2.32, 16 000 2.14 and 2.74; 512^3 (19 MB), 600 voxels 1.14 and 1.06, 2500
// 1.05 and 1.10; 512^3, 4 models, 2400 voxels 1.61 and 1.49, 10 000 2.04 and 2.05; 256^3, 16 models (38 MB), 640 voxels 0.81 and 2.27.
constexpr size_t OCCUPANCY_BYTES = (size_t)512 << 20, OCCUPANCY_PER_VOXEL = 16 << 10, OCCUPANCY_PER_MODEL = 4 << 20;
static hch_status device_occupancy(hch_levels *hl, const int32_t *coords, const int64_t *offsets, int32_t batch,
                                   const std::vector<int32_t> &side, const std::vector<int32_t> &ratio_of, int n_levels,
                                   hipStream_t s, Occupancy &o)
{
    if (n_levels > hch::MAX_LEVELS) return HCH_OK;
    hch::OccupancySet &S = o.set;
    S.n_levels = n_levels; S.batch = batch;
    int64_t words = 0, blocks = 0, divide = 1;
    for (int l = 0; l < n_levels; ++l) {
        const int64_t u = side[l], per_model = ((u * u * u + 63) / 64 + hch::OCC_WORDS - 1) / hch::OCC_WORDS;
        divide *= ratio_of[l];
        if ((uint64_t)per_model * hch::OCC_WORDS * 8 > OCCUPANCY_BYTES / (size_t)batch) return HCH_OK;
        S.side[l] = side[l]; S.ratio[l] = (int32_t)std::min<int64_t>(divide, 65536);       // past the side all divide to 0
        divide = S.ratio[l];
        S.word_off[l] = words; S.blocks[l] = (int32_t)per_model;
        words += per_model * batch * hch::OCC_WORDS;
        S.block_off[l] = (int32_t)blocks;
        if (l > 0) blocks += per_model * batch;
        S.block_off[l + 1] = (int32_t)blocks;
    }
    const int64_t n = offsets[batch], pairs = (int64_t)(n_levels - 1) * batch;
    if ((size_t)words * 8 > std::min(OCCUPANCY_BYTES, (size_t)n * OCCUPANCY_PER_VOXEL + (size_t)batch * OCCUPANCY_PER_MODEL)) return HCH_OK;
    int32_t *d_flags = nullptr;                // [0] flags, then the number of voxels of every (level >= 1, model)
    int64_t *d_offsets = nullptr;
    auto lay = [&](Pieces &P, size_t *zeroed) {
        P.take(o.d_bits, (size_t)words * 8);
        P.take(d_flags, (size_t)(1 + pairs) * 4);
        *zeroed = P.used;
        P.take(d_offsets, ((size_t)batch + 1) * 8);
        P.take(o.d_coords, (size_t)n * 12);
        P.take(o.d_sums, (size_t)blocks * 4);
        P.take(o.d_first, (size_t)pairs * 4);
    };
    Pieces size, place;
    size_t zeroed = 0;
    lay(size, &zeroed);
    if (o.mem.try_get((void **)&place.base, size.used) != hipSuccess) return HCH_OK;
    lay(place, &zeroed);
    HCH_HIP(hipMemsetAsync(place.base, 0, zeroed, s));
    HCH_HIP(hipMemcpyAsync(d_offsets, offsets, ((size_t)batch + 1) * 8, hipMemcpyHostToDevice, s));
    HCH_HIP(hipMemcpyAsync(o.d_coords, coords, (size_t)n * 12, hipMemcpyHostToDevice, s));
    int64_t most = 0;
    for (int v = 0; v < batch; ++v) most = std::max(most, offsets[v + 1] - offsets[v]);
    HCH_LAUNCH(hch::occupancy_mark_kernel, dim3(blocks_for(most), (unsigned)batch), dim3(256), 0, s, S, (const int32_t *)o.d_coords,
               (const int64_t *)d_offsets, o.d_bits, d_flags);
    HCH_LAUNCH_CHECK("occupancy_mark_kernel");
    if (blocks > 0) {
        HCH_LAUNCH(hch::occupancy_count_kernel, dim3((unsigned)blocks), dim3(hch::OCC_WORDS), 0, s, S, (const unsigned long long *)o.d_bits, o.d_sums);
        HCH_LAUNCH(hch::occupancy_scan_kernel, dim3((unsigned)pairs), dim3(256), 0, s, S, o.d_sums, d_flags + 1);
        HCH_LAUNCH_CHECK("occupancy_scan_kernel");
    }
    std::vector<int32_t> got((size_t)(1 + pairs));
    HCH_HIP(hipMemcpyAsync(got.data(), d_flags, got.size() * 4, hipMemcpyDeviceToHost, s));
    HCH_HIP(hipStreamSynchronize(s));
    if (got[0] & 1) return fail(HCH_EINVAL, "hch_build_levels: coordinate outside [0, resolution)");
    if (got[0] & 2) return fail(HCH_EINVAL, "hch_build_levels: duplicate voxel inside a model");
    o.first.resize((size_t)pairs);
    for (int l = 0; l < n_levels; ++l) {
        Level &L = hl->lv[l];
        L.ubar = side[l]; L.ratio = ratio_of[l]; L.b = batch;
        L.N.assign((size_t)batch + 1, 0);
        for (int v = 0; v < batch; ++v) {
            const int64_t nv = l == 0 ? offsets[v + 1] - offsets[v] : got[(size_t)(1 + (int64_t)(l - 1) * batch + v)];
            if (l > 0) o.first[(size_t)((int64_t)(l - 1) * batch + v)] = (int32_t)L.N[v];
            L.N[v + 1] = L.N[v] + nv;
            L.max_n = std::max<int32_t>(L.max_n, (int32_t)nv);
        }
        L.n_total = L.N[batch];
    }
    o.host_coords = coords;
    o.ready = true;
    return HCH_OK;
}

// Offsets of every table by launches over memory, H* and T* with them.
template <typename Fn>
static hch_status place_in_memory(hch_levels *hl, std::vector<PairWork> &work, DeviceBlocks &tmp, Fn &host_copies, hipStream_t s)
{
    hch_status st;
    const int n_pairs = (int)work.size();
    int32_t *d_fail = nullptr;
    if ((st = tmp.get((void **)&d_fail, (size_t)n_pairs * 4)) != HCH_OK) return st;
    std::vector<int32_t> h_fail((size_t)n_pairs);

    std::vector<int> active((size_t)n_pairs);
    for (int i = 0; i < n_pairs; ++i) active[i] = i;
    for (int round = 0; !active.empty(); ++round) {
        if (round >= 24) return fail(HCH_EBUILD, "hch_build_levels_device: perfect hash construction failed");
        const int na = (int)active.size();
        std::vector<hch::PairDesc> desc((size_t)na);
        int64_t cells = 0, vox = 0, slots = 0, words = 0;       // words of taken bits: no more than slots, but 2 where m is 1
        int32_t max_n = 0, max_r3 = 0, max_m3 = 0;
        for (int a = 0; a < na; ++a) {
            PairWork &w = work[active[a]];
            Level &L = hl->lv[w.l];
            if (w.r > 1024 || w.r > 2 * L.ubar + 1)   // beyond one cell per grid position nothing can improve
                return fail(HCH_EBUILD, "hch_build_levels_device: perfect hash construction failed");
            const int32_t r3 = w.r * w.r * w.r, m3 = w.m * w.m * w.m;
            desc[a] = hch::PairDesc{L.dcoords + 3 * L.N[w.v], L.dH + L.M[w.v], L.dT + 3 * L.M[w.v], w.n, w.m, w.r,
                                    (int32_t)cells, (int32_t)vox, (int32_t)slots, (int32_t)words, active[a]};
            cells += r3; vox += w.n; slots += m3; words += (int64_t)w.m * w.m * hch::psh_row_words(w.m);
            max_n = std::max(max_n, w.n); max_r3 = std::max(max_r3, r3); max_m3 = std::max(max_m3, m3);
            ++w.attempts;
        }
        if (cells >= ((int64_t)1 << 31) / hch::PSH_CLASSES || vox >= ((int64_t)1 << 31) || slots >= ((int64_t)1 << 31))
            return fail(HCH_EUNSUPPORTED, "hch_build_levels_device: offset tables exceed 32-bit indexing");
        hch::PairDesc *d_desc = nullptr;
        int32_t *d_cnt = nullptr, *d_first = nullptr, *d_sums = nullptr, *d_fill = nullptr, *d_bucket = nullptr, *d_members = nullptr;
        int32_t *d_counters = nullptr, *d_free = nullptr;
        uint32_t *d_phi = nullptr, *d_res = nullptr;
        unsigned long long *d_bits = nullptr;
        int2 *d_cells = nullptr;
        // counters: [0, CLASSES) buckets per class, then per active pair: free slots, singles placed
        const size_t n_counters = (size_t)hch::PSH_CLASSES + 2 * (size_t)na;
        auto lay_round = [&](Pieces &P, size_t *zeroed) {      // the arrays that start from zero first
            P.take(d_cnt, (size_t)cells * 4);
            P.take(d_fill, (size_t)cells * 4);
            P.take(d_phi, (size_t)cells * 4);
            P.take(d_counters, n_counters * 4);
            P.take(d_bits, (size_t)words * 8);
            *zeroed = P.used;
            P.take(d_desc, desc.size() * sizeof(hch::PairDesc));
            P.take(d_first, (size_t)cells * 4);
            P.take(d_sums, ((size_t)cells / hch::PSH_SCAN + 1) * 4);
            P.take(d_bucket, (size_t)vox * 4);
            P.take(d_members, (size_t)vox * 4);
            P.take(d_res, (size_t)vox * 4);
            P.take(d_free, (size_t)slots * 4);
            P.take(d_cells, (size_t)cells * hch::PSH_CLASSES * sizeof(int2));
        };
        Pieces size, place;
        size_t zeroed = 0;
        lay_round(size, &zeroed);
        if ((st = tmp.get((void **)&place.base, size.used)) != HCH_OK) return st;
        lay_round(place, &zeroed);
        HCH_HIP(hipMemsetAsync(place.base, 0, zeroed, s));
        HCH_HIP(hipMemcpyAsync(d_desc, desc.data(), desc.size() * sizeof(hch::PairDesc), hipMemcpyHostToDevice, s));
        int32_t *d_class_count = d_counters, *d_nfree = d_counters + hch::PSH_CLASSES, *d_rank = d_nfree + na;
        HCH_HIP(hipMemsetAsync(d_fail, 0, (size_t)n_pairs * 4, s));

        const dim3 gv((unsigned)((max_n + 255) / 256), (unsigned)na), gc((unsigned)((max_r3 + 255) / 256), (unsigned)na);
        const dim3 gs((unsigned)((max_m3 + hch::PSH_FREE - 1) / hch::PSH_FREE), (unsigned)na);
        HCH_LAUNCH(hch::psh_count_kernel, gv, dim3(256), 0, s, d_desc, d_cnt, d_bucket);
        const unsigned stretches = (unsigned)((cells + hch::PSH_SCAN - 1) / hch::PSH_SCAN);
        HCH_LAUNCH(hch::psh_sum_kernel, dim3(stretches), dim3(256), 0, s, d_cnt, d_sums, (int)cells);
        HCH_LAUNCH(hch::psh_scan_kernel, dim3(stretches), dim3(256), 0, s, d_cnt, d_sums, d_first, (int)cells);
        HCH_LAUNCH(hch::psh_fill_kernel, gv, dim3(256), 0, s, d_desc, d_bucket, d_first, d_fill, d_members, d_res);
        HCH_LAUNCH(hch::psh_classify_kernel, gc, dim3(256), 0, s, d_desc, d_cnt, d_class_count, d_cells, cells);
        HCH_LAUNCH_CHECK("psh construction");
        int32_t class_count[hch::PSH_CLASSES];
        HCH_HIP(hipMemcpyAsync(class_count, d_class_count, sizeof class_count, hipMemcpyDeviceToHost, s));
        HCH_HIP(hipStreamSynchronize(s));
        // largest buckets first: all of 9 voxels and more in one launch, then one size per launch
        for (int k = hch::PSH_CLASSES - 1; k >= 2; --k) {
            if (class_count[k] <= 0) continue;
            const int64_t waves = std::max<int64_t>(64, slots / (48 * k));     // see psh_place_kernel
            HCH_LAUNCH(hch::psh_place_kernel, dim3((unsigned)((std::min<int64_t>(class_count[k], waves) + 3) / 4)), dim3(256), 0, s, d_desc,
                               d_cells + (size_t)k * cells, class_count[k], d_cnt, d_first, d_members, d_res, d_bits,
                               d_phi, d_fail);
        }
        HCH_LAUNCH(hch::psh_free_list_kernel, gs, dim3(256), 0, s, d_desc, d_nfree, d_free);
        HCH_LAUNCH(hch::psh_place_single_kernel, gc, dim3(256), 0, s, d_desc, d_cnt, d_first, d_members, d_res,
                           d_nfree, d_free, d_rank, d_phi, d_fail);
        HCH_LAUNCH(hch::psh_clear_kernel, gs, dim3(256), 0, s, d_desc, d_fail);
        HCH_LAUNCH_CHECK("psh construction");
        if (round == 0) host_copies();
        HCH_HIP(hipMemcpyAsync(h_fail.data(), d_fail, (size_t)n_pairs * 4, hipMemcpyDeviceToHost, s));
        HCH_HIP(hipStreamSynchronize(s));

        std::vector<int> again;
        for (int a = 0; a < na; ++a) {
            PairWork &w = work[active[a]];
            if (!h_fail[active[a]]) {
                w.done = true;
                w.phi = d_phi + desc[a].cell_base;
                continue;
            }
            w.r = hch::offset_side_next(w.r, w.m);
            again.push_back(active[a]);
        }
        active.swap(again);
    }
    return HCH_OK;
}

// Offsets of every table by a workgroup each (psh_build_kernel).  Up to three sides at once where that leaves a CU to each: the
// second is needed by a third of the tables, the third by one or two of a batch, and they are known at the same time.
constexpr int SIDES_AT_ONCE = 3;
template <typename Fn>
static hch_status place_in_lds(hch_levels *hl, std::vector<PairWork> &work, DeviceBlocks &tmp, Fn &host_copies, hipStream_t s)
{
    hch_status st;
    const int n_pairs = (int)work.size();
    std::vector<int> active((size_t)n_pairs);
    for (int i = 0; i < n_pairs; ++i) active[i] = i;
    for (int round = 0; !active.empty(); ++round) {
        if (round >= 24) return fail(HCH_EBUILD, "hch_build_levels_device: perfect hash construction failed");
        const int na = (int)active.size(), at_once = std::max(1, std::min(SIDES_AT_ONCE, (int)hch::NUM_CU / na));
        std::vector<hch::AttemptDesc> desc;
        std::vector<int> pair_of;
        int64_t cells = 0, vox = 0;
        size_t lds = 0;
        for (int a = 0; a < na; ++a) {
            const PairWork &w = work[active[a]];
            const Level &L = hl->lv[w.l];
            int r = w.r;
            for (int k = 0; k < at_once; ++k, r = hch::offset_side_next(r, w.m)) {
                if (k > 0 && r > 100) break;                  // no memory for a second side that is large
                if (r > 1024 || r > 2 * L.ubar + 1) {         // beyond one cell per grid position nothing can improve
                    if (k == 0) return fail(HCH_EBUILD, "hch_build_levels_device: perfect hash construction failed");
                    break;
                }
                desc.push_back(hch::AttemptDesc{L.dcoords + 3 * L.N[w.v], w.n, w.m, r, (int32_t)cells, (int32_t)vox});
                pair_of.push_back(active[a]);
                const int64_t r3 = (int64_t)r * r * r;
                cells += r3; vox += w.n;
                lds = std::max({lds, (size_t)w.m * w.m * 32, r3 * 4 <= hch::PSH_LDS_BYTES ? (size_t)r3 * 4 : (size_t)0});
            }
        }
        if (cells >= ((int64_t)1 << 31) / hch::PSH_CLASSES || vox >= ((int64_t)1 << 31))
            return fail(HCH_EUNSUPPORTED, "hch_build_levels_device: offset tables exceed 32-bit indexing");
        hch::AttemptDesc *d_desc = nullptr;
        int32_t *d_ok = nullptr, *d_cnt = nullptr, *d_first = nullptr, *d_rank = nullptr;
        uint32_t *d_phi = nullptr, *d_res = nullptr;
        uint4 *d_list = nullptr;
        auto lay_round = [&](Pieces &P, size_t *zeroed) {
            P.take(d_phi, (size_t)cells * 4);
            *zeroed = P.used;
            P.take(d_ok, desc.size() * 4);
            P.take(d_desc, desc.size() * sizeof(hch::AttemptDesc));
            P.take(d_cnt, (size_t)cells * 4);
            P.take(d_first, (size_t)cells * 4);
            P.take(d_list, (size_t)cells * sizeof(uint4));
            P.take(d_rank, (size_t)vox * 4);
            P.take(d_res, (size_t)vox * 4);
        };
        Pieces size, place;
        size_t zeroed = 0;
        lay_round(size, &zeroed);
        if ((st = tmp.get((void **)&place.base, size.used)) != HCH_OK) return st;
        lay_round(place, &zeroed);
        HCH_HIP(hipMemsetAsync(d_phi, 0, zeroed, s));          // unused cells keep (0, 0, 0)
        HCH_HIP(hipMemcpyAsync(d_desc, desc.data(), desc.size() * sizeof(hch::AttemptDesc), hipMemcpyHostToDevice, s));
        const int total = (int)desc.size();
        HCH_LAUNCH(hch::psh_build_kernel, dim3((unsigned)total), dim3(hch::PSH_THREADS), lds, s, d_desc, d_cnt, d_first, d_phi, d_list, d_rank, d_res,
                   d_ok, (int)lds);
        HCH_LAUNCH_CHECK("psh_build_kernel");
        if (round == 0) host_copies();
        std::vector<int32_t> ok((size_t)total);
        HCH_HIP(hipMemcpyAsync(ok.data(), d_ok, (size_t)total * 4, hipMemcpyDeviceToHost, s));
        HCH_HIP(hipStreamSynchronize(s));
        std::vector<int> again;
        for (int q = 0; q < total; ++q) {
            PairWork &w = work[pair_of[q]];
            if (w.done) continue;                     // its smaller side was enough
            ++w.attempts;
            if (ok[q]) { w.r = desc[q].r; w.phi = d_phi + desc[q].cell_base; w.done = true; }
            else {
                w.r = hch::offset_side_next(desc[q].r, w.m);
                if (q + 1 == total || pair_of[q + 1] != pair_of[q]) again.push_back(pair_of[q]);
            }
        }
        active.swap(again);
    }
    return HCH_OK;
}

// Fills, for every level: mbar, rbar, attempts, M, R, m_total, r_total, the device tables dH, dT,
// dV, dPhi, dslot3, dphi4, dcoords, dmeta and the host copies.  Levels must have ubar, b, N, n_total and, unless
// `occ` has them, coords.
static hch_status device_construct(hch_levels *hl, Occupancy &occ, hipStream_t s)
{
    const int n_levels = (int)hl->lv.size();
    const int batch = hl->lv[0].b;
    DeviceBlocks tmp;
    std::vector<PairWork> work;
    hch_status st;
    for (int l = 0; l < n_levels; ++l) {
        Level &L = hl->lv[l];
        L.mbar.assign((size_t)batch, 0); L.rbar.assign((size_t)batch, 0); L.attempts.assign((size_t)batch, 0);
        L.M.assign((size_t)batch + 1, 0); L.R.assign((size_t)batch + 1, 0);
        for (int v = 0; v < batch; ++v) {
            const int64_t n = L.N[v + 1] - L.N[v];
            const int m = hch::hash_side(n);
            if (m > 256) return fail(HCH_EUNSUPPORTED, "hch_build_levels_device: a model needs a hash table side above 256");
            L.mbar[v] = m;
            L.M[v + 1] = L.M[v] + (int64_t)m * m * m;
            work.push_back(PairWork{l, v, (int32_t)n, m, hch::offset_side_first(n, m), 0, nullptr, false});
        }
        L.m_total = L.M[batch];
        if (L.m_total >= ((int64_t)1 << 31)) return fail(HCH_EUNSUPPORTED, "hch_build_levels_device: super table exceeds 32-bit indexing");
    }
    // what the level set keeps and whose size is known now, in one allocation (one by one the
    // allocations and frees of a build took 6 ms); H* and T* first, so that one fill empties them, then the
    // positions, so that one copy brings all of them to the host
    size_t copied = 0;
    auto lay = [&](Pieces &P, size_t *tables) {
        for (Level &L : hl->lv) { P.take(L.dH, (size_t)L.m_total * 4); P.take(L.dT, (size_t)L.m_total * 6); }
        *tables = P.used;
        for (int l = 1; l < n_levels; ++l) P.take(hl->lv[l].dcoords, (size_t)hl->lv[l].n_total * 12);
        copied = P.used;
        P.take(hl->lv[0].dcoords, (size_t)hl->lv[0].n_total * 12);
        for (Level &L : hl->lv) {
            const size_t n = (size_t)L.n_total;
            P.take(L.dV, (size_t)L.m_total * 4);
            P.take(L.dslot3, (size_t)L.m_total * 4 * hch::SLOT_WORDS);
            P.take(L.dnbr, n * 27 * 4);
            if (&L != &hl->lv[0] && L.ratio == 2) P.take(L.dchild, n * 8 * 4);
            P.take(L.dmask27, std::max<size_t>(n, 64) * 4);
            P.take(L.dtilemask, std::max<size_t>((n + hch::PATTERN_TILE - 1) / hch::PATTERN_TILE, 64) * 4);
        }
    };
    {
        Pieces size, place;
        size_t tables = 0;
        lay(size, &tables);
        void *block = nullptr;
        hipError_t e = device_malloc(&block, size.used);
        if (e != hipSuccess) return fail(HCH_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        hl->blocks.push_back(block);
        place.base = (char *)block;
        for (Level &L : hl->lv) L.in_block = true;
        lay(place, &tables);
        HCH_HIP(hipMemsetAsync(block, 0xFF, tables, s));      // H* = -1: free slot; T* = 0xFFFF: no position
        if (!occ.ready) {
            for (Level &L : hl->lv) HCH_HIP(hipMemcpyAsync(L.dcoords, L.coords.data(), L.coords.size() * 4, hipMemcpyHostToDevice, s));
        } else {
            HCH_HIP(hipMemcpyAsync(hl->lv[0].dcoords, occ.d_coords, (size_t)hl->lv[0].n_total * 12, hipMemcpyDeviceToDevice, s));
            hch::OccupancyOut out{};
            for (int l = 1; l < n_levels; ++l) out.coords[l] = hl->lv[l].dcoords;
            if (n_levels > 1) {
                HCH_HIP(hipMemcpyAsync(occ.d_first, occ.first.data(), occ.first.size() * 4, hipMemcpyHostToDevice, s));
                HCH_LAUNCH(hch::occupancy_list_kernel, dim3((unsigned)occ.set.block_off[n_levels]), dim3(hch::OCC_WORDS), 0, s, occ.set,
                           (const unsigned long long *)occ.d_bits, (const int32_t *)occ.d_sums, (const int32_t *)occ.d_first, out);
                HCH_LAUNCH_CHECK("occupancy_list_kernel");
            }
        }
    }
    // The host copies: a mirror of the first `copied` bytes, the finest positions, V*.  Fresh memory costs more to
    // touch than to fill, so that is done while the device builds.
    const char *const mirrored = (const char *)hl->lv[0].dH;
    auto host_copies = [&]() {
        const size_t finest = (size_t)hl->lv[0].n_total * 12;
        size_t slots = 0;
        for (const Level &L : hl->lv) slots += (size_t)L.m_total;
        hl->host_block.make(copied + finest + slots * 4);
        char *h = hl->host_block.get();
        for (size_t at = 0; at < copied && !hl->host_block.pinned(); at += 4096) h[at] = 0;
        memcpy(h + copied, occ.ready ? occ.host_coords : hl->lv[0].coords.data(), finest);
        int32_t *V = (int32_t *)(h + copied + finest);
        for (Level &L : hl->lv) {
            L.hH = (const int32_t *)(h + ((const char *)L.dH - mirrored));
            L.hT = (const uint16_t *)(h + ((const char *)L.dT - mirrored));
            L.hcoords = (const int32_t *)(&L == &hl->lv[0] ? h + copied : h + ((const char *)L.dcoords - mirrored));
            L.hV = V;
            for (int v = 0; v < batch; ++v) std::fill(V + L.M[v], V + L.M[v + 1], v);
            V += L.m_total;
            std::vector<int32_t>().swap(L.coords);
        }
    };
    const int n_pairs = (int)work.size();
    // A workgroup per table, where rows fit 64 bits and the largest table is not most of the work (then a chip full of wavefronts on that one is as
    // fast).  Whole builds with 3 levels, there and by launches over memory: 40 models of 4000 voxels 0.78 and 1.89 ms, 1 of 3000 0.46 and 0.80, 1 of
    // 25 000 0.69 and 0.70, 2 of 150 000 1.83 and 2.04, 3 of 230 000 3.7 and 4.3; 1 of 90 000 1.45 and 1.38, 1 of 250 000 3.5 and 3.2, 2 of 250 000
    // 7.5 and 6.9; one level of 2 of 100 000 1.4 and 1.2, of 200 000 2.7 and 2.2; rows of 128 bits, 1 of 400 000 8.0 and 3.8, 4 of them 11 and 16.
    int32_t widest_m = 0;
    int64_t largest = 0, all_voxels = 0;
    for (const PairWork &w : work) {
        widest_m = std::max(widest_m, w.m);
        largest = std::max<int64_t>(largest, w.n);
        all_voxels += w.n;
    }
    const bool in_lds = widest_m <= hch::PSH_LDS_SIDE && (largest <= 32768 || (double)all_voxels >= (largest > 229376 ? 3.0 : 2.2) * (double)largest);
    st = in_lds ? place_in_lds(hl, work, tmp, host_copies, s) : place_in_memory(hl, work, tmp, host_copies, s);
    if (st != HCH_OK) return st;

    // super tables of every level from the pairs' results
    std::vector<hch::PackDesc> pd((size_t)n_pairs);
    std::vector<int32_t> meta;
    const size_t meta_len = 5 * (size_t)batch + 3;            // mbar, rbar, M, R, N
    for (int l = 0; l < n_levels; ++l) {
        Level &L = hl->lv[l];
        for (int v = 0; v < batch; ++v) {
            const PairWork &w = work[(size_t)l * batch + v];
            L.rbar[v] = w.r; L.attempts[v] = w.attempts;
            L.R[v + 1] = L.R[v] + (int64_t)w.r * w.r * w.r;
        }
        L.r_total = L.R[batch];
        if (L.r_total >= ((int64_t)1 << 31) / 3) return fail(HCH_EUNSUPPORTED, "hch_build_levels_device: super table exceeds 32-bit indexing");
        meta.insert(meta.end(), L.mbar.begin(), L.mbar.end());
        meta.insert(meta.end(), L.rbar.begin(), L.rbar.end());
        for (int64_t x : L.M) meta.push_back((int32_t)x);
        for (int64_t x : L.R) meta.push_back((int32_t)x);
        for (int64_t x : L.N) meta.push_back((int32_t)x);
    }
    int32_t *d_meta = nullptr;
    hch::PackDesc *d_pd = nullptr;
    size_t phi_bytes = 0;
    {
        auto lay_offsets = [&](Pieces &P) {
            for (Level &L : hl->lv) P.take(L.dPhi, (size_t)L.r_total * 3);
            phi_bytes = P.used;
            for (Level &L : hl->lv) P.take(L.dphi4, (size_t)L.r_total * 4);
            P.take(d_meta, meta.size() * 4);
            P.take(d_pd, pd.size() * sizeof(hch::PackDesc));
        };
        Pieces size, place;
        lay_offsets(size);
        void *block = nullptr;
        hipError_t e = device_malloc(&block, size.used);
        if (e != hipSuccess) return fail(HCH_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
        hl->blocks.push_back(block);
        place.base = (char *)block;
        lay_offsets(place);
    }
    int32_t most = 0, widest = 0;
    for (const PairWork &w : work) {
        const Level &L = hl->lv[w.l];
        pd[(size_t)w.l * batch + w.v] = hch::PackDesc{L.dcoords + 3 * L.N[w.v], w.phi, L.dH + L.M[w.v], L.dT + 3 * L.M[w.v],
                                                      L.dslot3 + hch::SLOT_WORDS * L.M[w.v], L.dphi4 + L.R[w.v], L.dV + L.M[w.v], L.dPhi + 3 * L.R[w.v],
                                                      w.n, w.m, w.r, w.v};
        most = std::max(most, w.n);
        widest = std::max({widest, w.m * w.m * w.m, w.r * w.r * w.r});
    }
    HCH_HIP(hipMemcpyAsync(d_pd, pd.data(), pd.size() * sizeof(hch::PackDesc), hipMemcpyHostToDevice, s));
    HCH_HIP(hipMemcpyAsync(d_meta, meta.data(), meta.size() * 4, hipMemcpyHostToDevice, s));
    for (int l = 0; l < n_levels; ++l) hl->lv[l].dmeta = d_meta + (size_t)l * meta_len;
    // a grid's second side ends at 65535 tables
    for (int p0 = 0; p0 < n_pairs; p0 += 65535) {
        const unsigned tables = (unsigned)std::min(65535, n_pairs - p0);
        if (in_lds) HCH_LAUNCH(hch::psh_emit_kernel, dim3(blocks_for(most), tables), dim3(256), 0, s, (const hch::PackDesc *)d_pd + p0);
        HCH_LAUNCH(hch::psh_pack_kernel, dim3(blocks_for(widest), tables), dim3(256), 0, s, (const hch::PackDesc *)d_pd + p0);
    }
    HCH_LAUNCH_CHECK("psh_pack_kernel");
    // host copies for hch_level_info
    hl->host_phi.make(phi_bytes);
    HCH_HIP(hipMemcpyAsync(hl->host_block.get(), mirrored, copied, hipMemcpyDeviceToHost, s));
    HCH_HIP(hipMemcpyAsync(hl->host_phi.get(), hl->lv[0].dPhi, phi_bytes, hipMemcpyDeviceToHost, s));
    for (Level &L : hl->lv) L.hPhi = (const uint8_t *)(hl->host_phi.get() + (L.dPhi - hl->lv[0].dPhi));
    HCH_HIP(hipStreamSynchronize(s));         // `meta`, `pd` and the coordinates' copies are done
    // (as soon as the coarse levels are listed it could go, but a hipFree between the launches costs 0.3 of 4.8 ms)
    occ.mem.release();
    return HCH_OK;
}

// ratios == nullptr: every level halves the resolution (a power of two); else ratios[l] >= 2 is
// the ratio between level l and level l+1, whose side is ceil(side_l / ratios[l])
// Run `fn` on up to `nthr` host threads (the caller's included) and wait for all of them.  An
// exception inside a worker (std::bad_alloc from its vectors, std::system_error) must not leave
// the thread function: it is caught there and reported as false.  Threads that were started are
// always joined, also when starting a further one fails.
template <typename Fn>
static bool run_on_threads(unsigned nthr, Fn fn)
{
    std::atomic<int> failed(0);
    auto guarded = [&]() {
        try { fn(); } catch (...) { failed = 1; }
    };
    std::vector<std::thread> pool;
    struct Joiner {
        std::vector<std::thread> &p;
        ~Joiner() { for (auto &th : p) if (th.joinable()) th.join(); }
    } joiner{pool};
    try {
        pool.reserve(nthr);
        for (unsigned i = 1; i < nthr; ++i) pool.emplace_back(guarded);
    } catch (...) {
        failed = 1;             // fewer threads than wanted: the work is still done below
    }
    guarded();
    for (auto &th : pool) th.join();
    return failed == 0;
}

static hch_status build_impl(const int32_t *coords_xyz, const int64_t *model_offsets,
                             int32_t batch, int32_t resolution, int32_t n_levels, const int32_t *ratios,
                             void *stream, bool with_device, bool device_tables, hch_levels **out, bool host_checks = false)
{
    if (out) *out = nullptr;
    if (!coords_xyz || !model_offsets || !out) return fail(HCH_EINVAL, "hch_build_levels: null pointer");
    if (batch <= 0 || batch > 65535) return fail(HCH_EINVAL, "hch_build_levels: batch must be 1..65535");
    std::vector<int32_t> side((size_t)std::max(n_levels, 1), resolution), ratio_of((size_t)std::max(n_levels, 1), 1);
    if (!ratios) {
        if (resolution < 2 || resolution > 32768 || (resolution & (resolution - 1)))
            return fail(HCH_EINVAL, "hch_build_levels: resolution must be a power of two in 2..32768");
        if (n_levels < 1 || (resolution >> (n_levels - 1)) < 1)
            return fail(HCH_EINVAL, "hch_build_levels: n_levels out of range for this resolution");
        for (int l = 1; l < n_levels; ++l) { side[l] = resolution >> l; ratio_of[l] = 2; }
    } else {
        if (resolution < 2 || resolution > 32768)
            return fail(HCH_EINVAL, "hch_build_levels_ratios: resolution must be in 2..32768");
        if (n_levels < 1) return fail(HCH_EINVAL, "hch_build_levels_ratios: n_levels must be at least 1");
        for (int l = 1; l < n_levels; ++l) {
            if (ratios[l - 1] < 2 || side[l - 1] < 2)
                return fail(HCH_EINVAL, "hch_build_levels_ratios: every ratio must be >= 2 and every level but the last have side >= 2");
            ratio_of[l] = ratios[l - 1];
            side[l] = (side[l - 1] + ratios[l - 1] - 1) / ratios[l - 1];
        }
    }
    if (model_offsets[0] != 0) return fail(HCH_EINVAL, "hch_build_levels: model_offsets[0] must be 0");
    for (int v = 0; v < batch; ++v)
        if (model_offsets[v + 1] <= model_offsets[v])
            return fail(HCH_EINVAL, "hch_build_levels: empty model or decreasing model_offsets");
    const int64_t n_total = model_offsets[batch];
    if (n_total >= ((int64_t)1 << 31) / 27)
        return fail(HCH_EUNSUPPORTED, "hch_build_levels: more than 2^31/27 voxels in a batch");
    hipStream_t s = (hipStream_t)stream;
    hch_levels *hl = nullptr;
    Occupancy occ;
    hch_status st = HCH_OK;
    if (device_tables && !host_checks) {
        hl = new (std::nothrow) hch_levels;
        if (!hl) return fail(HCH_ENOMEM, "hch_build_levels: out of host memory");
        try {
            hl->lv.resize((size_t)n_levels);
            st = device_occupancy(hl, coords_xyz, model_offsets, batch, side, ratio_of, n_levels, s, occ);
        } catch (const std::bad_alloc &) {
            st = fail(HCH_ENOMEM, "hch_build_levels: out of host memory");
        }
        if (st != HCH_OK || !occ.ready) { hch_free_levels(hl); hl = nullptr; }
        if (st != HCH_OK) return st;
    }
    for (int64_t i = 0; i < 3 * n_total && !occ.ready; ++i)
        if (coords_xyz[i] < 0 || coords_xyz[i] >= resolution)
            return fail(HCH_EINVAL, "hch_build_levels: coordinate outside [0, resolution)");
    // duplicates inside a model (models in parallel on host threads)
    if (!occ.ready) {
        std::atomic<int> next_model(0), dup(0);
        auto check = [&]() {
            std::vector<int64_t> lin;
            for (;;) {
                const int v = next_model.fetch_add(1);
                if (v >= batch) break;
                const int64_t a = model_offsets[v], n = model_offsets[v + 1] - a;
                lin.resize((size_t)n);
                for (int64_t i = 0; i < n; ++i) {
                    const int32_t *p = coords_xyz + 3 * (a + i);
                    lin[i] = ((int64_t)p[0] * resolution + p[1]) * resolution + p[2];
                }
                if (!std::is_sorted(lin.begin(), lin.end())) std::sort(lin.begin(), lin.end());
                if (std::adjacent_find(lin.begin(), lin.end()) != lin.end()) dup = 1;
            }
        };
        const unsigned nthr = std::max(1u, std::min({std::thread::hardware_concurrency(), 16u, (unsigned)batch}));
        if (!run_on_threads(nthr, check)) return fail(HCH_ENOMEM, "hch_build_levels: out of host memory");
        if (dup) return fail(HCH_EINVAL, "hch_build_levels: duplicate voxel inside a model");
    }

    if (!hl) hl = new (std::nothrow) hch_levels;
    if (!hl) return fail(HCH_ENOMEM, "hch_build_levels: out of host memory");

    try {
        hl->lv.resize((size_t)n_levels);
        // ---- occupancy of every level (host) ----
        for (int l = 0; l < n_levels && !occ.ready; ++l) {
            Level &L = hl->lv[l];
            L.ubar = side[l];
            L.ratio = ratio_of[l];
            L.b = batch;
            L.N.assign((size_t)batch + 1, 0);
            if (l == 0) {
                L.coords.assign(coords_xyz, coords_xyz + 3 * n_total);
                for (int v = 0; v <= batch; ++v) L.N[v] = model_offsets[v];
            } else {
                const Level &Lf = hl->lv[l - 1];
                std::vector<std::vector<int32_t>> per_model((size_t)batch);
                std::atomic<int> next_model(0);
                auto coarsen = [&]() {
                    for (;;) {
                        const int v = next_model.fetch_add(1);
                        if (v >= batch) break;
                        hch::coarsen_model(Lf.coords.data() + 3 * Lf.N[v], Lf.N[v + 1] - Lf.N[v], Lf.ubar, L.ratio, per_model[v]);
                    }
                };
                {
                    const unsigned nthr = std::max(1u, std::min({std::thread::hardware_concurrency(), 16u, (unsigned)batch}));
                    if (!run_on_threads(nthr, coarsen)) throw std::bad_alloc();
                }
                for (int v = 0; v < batch; ++v) {
                    L.coords.insert(L.coords.end(), per_model[v].begin(), per_model[v].end());
                    L.N[v + 1] = L.N[v] + (int64_t)per_model[v].size() / 3;
                }
            }
            L.n_total = L.N[batch];
            L.max_n = 0;
            for (int v = 0; v < batch; ++v) L.max_n = std::max<int32_t>(L.max_n, (int32_t)(L.N[v + 1] - L.N[v]));
        }

        if (device_tables) {
            if (n_levels > hch::MAX_LEVELS) st = fail(HCH_EUNSUPPORTED, "hch_build_levels: too many levels");
            if (st == HCH_OK) st = device_construct(hl, occ, s);
        }
        // ---- PSH construction of every (level, model), spread over host threads ----
        std::vector<std::vector<hch::ModelTables>> tabs((size_t)n_levels);
        for (auto &t : tabs) t.resize((size_t)batch);
        const int n_tasks = device_tables ? 0 : n_levels * batch;
        std::vector<int> result((size_t)n_tasks, 0);
        std::atomic<int> next(0);
        auto worker = [&]() {
            for (;;) {
                const int t = next.fetch_add(1);
                if (t >= n_tasks) break;
                const int l = t / batch, v = t % batch;     // finest (largest) levels first
                const Level &L = hl->lv[l];
                result[t] = (int)hch::build_model_tables(L.coords.data() + 3 * L.N[v],
                                                         L.N[v + 1] - L.N[v], L.ubar, tabs[l][v]);
            }
        };
        {
            unsigned nthr = std::thread::hardware_concurrency();
            nthr = std::max(1u, std::min(nthr, 16u));
            nthr = std::min<unsigned>(nthr, (unsigned)std::max(1, n_tasks));
            if (!run_on_threads(nthr, worker)) throw std::bad_alloc();
        }
        for (int t = 0; t < n_tasks && st == HCH_OK; ++t) {
            if (result[t] == hch::BUILD_UNSUPPORTED)
                st = fail(HCH_EUNSUPPORTED, "hch_build_levels: a model needs a hash table side above 256");
            else if (result[t] == hch::BUILD_FAILED)
                st = fail(HCH_EBUILD, "hch_build_levels: perfect hash construction failed");
        }

        // ---- super tables (Section 3.2) and upload ----
        for (int l = 0; l < n_levels && st == HCH_OK; ++l) {
            Level &L = hl->lv[l];
            if (device_tables) continue;              // all of it is in the blocks of device_construct
            L.mbar.resize((size_t)batch); L.rbar.resize((size_t)batch); L.attempts.resize((size_t)batch);
            L.M.assign((size_t)batch + 1, 0); L.R.assign((size_t)batch + 1, 0);
            for (int v = 0; v < batch; ++v) {
                const hch::ModelTables &t = tabs[l][v];
                L.mbar[v] = t.m; L.rbar[v] = t.r; L.attempts[v] = t.attempts;
                L.M[v + 1] = L.M[v] + (int64_t)t.m * t.m * t.m;
                L.R[v + 1] = L.R[v] + (int64_t)t.r * t.r * t.r;
            }
            L.m_total = L.M[batch]; L.r_total = L.R[batch];
            if (L.m_total >= ((int64_t)1 << 31) || L.r_total >= ((int64_t)1 << 31) / 3) {
                st = fail(HCH_EUNSUPPORTED, "hch_build_levels: super table exceeds 32-bit indexing");
                break;
            }
            L.H.resize((size_t)L.m_total); L.V.resize((size_t)L.m_total);
            L.T.resize((size_t)L.m_total * 3); L.Phi.resize((size_t)L.r_total * 3);
            for (int v = 0; v < batch; ++v) {
                hch::ModelTables &t = tabs[l][v];
                std::copy(t.H.begin(), t.H.end(), L.H.begin() + L.M[v]);
                std::copy(t.T.begin(), t.T.end(), L.T.begin() + 3 * L.M[v]);
                std::copy(t.Phi.begin(), t.Phi.end(), L.Phi.begin() + 3 * L.R[v]);
                std::fill(L.V.begin() + L.M[v], L.V.begin() + L.M[v + 1], v);
                t = hch::ModelTables();
            }
            if (!with_device) continue;
            std::vector<int32_t> meta;
            meta.insert(meta.end(), L.mbar.begin(), L.mbar.end());
            meta.insert(meta.end(), L.rbar.begin(), L.rbar.end());
            for (int64_t x : L.M) meta.push_back((int32_t)x);
            for (int64_t x : L.R) meta.push_back((int32_t)x);
            for (int64_t x : L.N) meta.push_back((int32_t)x);

            if ((st = upload((void **)&L.dH, L.H.data(), L.H.size() * 4, s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dV, L.V.data(), L.V.size() * 4, s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dT, L.T.data(), L.T.size() * 2, s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dPhi, L.Phi.data(), L.Phi.size(), s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dcoords, L.coords.data(), L.coords.size() * 4, s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dmeta, meta.data(), meta.size() * 4, s)) != HCH_OK) break;
            constexpr int SW = hch::SLOT_WORDS;
            std::vector<uint32_t> slot3((size_t)L.m_total * SW, 0u), phi4((size_t)L.r_total);
            for (int64_t q = 0; q < L.m_total; ++q) {
                slot3[SW * q + 0] = (uint32_t)L.H[q];
                slot3[SW * q + 1] = (uint32_t)L.T[3 * q] | ((uint32_t)L.T[3 * q + 1] << 16);
                slot3[SW * q + 2] = (uint32_t)L.T[3 * q + 2];
            }
            for (int64_t q = 0; q < L.r_total; ++q)
                phi4[q] = (uint32_t)L.Phi[3 * q] | ((uint32_t)L.Phi[3 * q + 1] << 8) | ((uint32_t)L.Phi[3 * q + 2] << 16);
            if ((st = upload((void **)&L.dslot3, slot3.data(), slot3.size() * 4, s)) != HCH_OK) break;
            if ((st = upload((void **)&L.dphi4, phi4.data(), phi4.size() * 4, s)) != HCH_OK) break;
            if (device_malloc((void **)&L.dnbr, (size_t)L.n_total * 27 * 4) != hipSuccess) {
                st = fail(HCH_ENOMEM, "hipMalloc(nbr27) failed"); break;
            }
            if (l > 0 && L.ratio == 2 && device_malloc((void **)&L.dchild, (size_t)L.n_total * 8 * 4) != hipSuccess) {
                st = fail(HCH_ENOMEM, "hipMalloc(child8) failed"); break;
            }
            // the staging vectors die at the end of this iteration: finish the copies first
            hipError_t e = hipStreamSynchronize(s);
            if (e != hipSuccess) { st = fail(HCH_EHIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(e)); break; }
        }
        if (st == HCH_OK && with_device) {
            if (n_levels > hch::MAX_LEVELS) st = fail(HCH_EUNSUPPORTED, "hch_build_levels: too many levels");
        }
        if (st == HCH_OK && with_device) {
            // buffers of the pattern order (see launch_index_lists)
            hl->sort_off.assign((size_t)n_levels + 1, 0);
            for (int l = 0; l < n_levels; ++l) hl->sort_off[l + 1] = hl->sort_off[l] + (int32_t)hl->lv[l].n_total;
            const size_t n_all = (size_t)hl->sort_off[n_levels];
            int64_t nbr_tiles = 0;
            for (int l = 0; l < n_levels; ++l)
                for (int v = 0; v < batch; ++v) nbr_tiles += (hl->lv[l].N[v + 1] - hl->lv[l].N[v] + 255) / 256;
            // the fine order: neighbour sets by position in both orders, the order, its tiles' taps,
            // the histograms and their totals
            const size_t na = round_up(std::max<size_t>(n_all, 64), 64);
            size_t fine_tiles = 0, hist = 0;
            for (int l = 0; l < n_levels; ++l) {
                const int64_t n = hl->lv[l].n_total;
                hl->set.n_total[l] = (int32_t)n;
                hl->set.fine_off[l] = (int32_t)hist;
                hl->set.fine_tiles[l] = n >= FINE_MIN_VOXELS ? (int32_t)((n + hch::FINE_TILE - 1) / hch::FINE_TILE) : 0;
                hist += (size_t)hl->set.fine_tiles[l] * hch::FINE_BINS;
                if (hl->set.fine_tiles[l]) fine_tiles += (size_t)((n + hch::PATTERN_TILE - 1) / hch::PATTERN_TILE);
            }
            const size_t totals = hist ? (size_t)hch::MAX_LEVELS * hch::FINE_BINS : 0;
            auto lay = [&](Pieces &P) {            // one allocation: seven took 0.5 ms of a build
                P.take(hl->d_sort_key, std::max<size_t>(n_all, 64));
                P.take(hl->d_order, std::max<size_t>(n_all, 64) * 4);
                P.take(hl->d_tile_hist, (size_t)std::max<int64_t>(nbr_tiles, 1) * hch::PATTERN_BINS * 4);
                P.take(hl->d_key_total, (size_t)hch::MAX_LEVELS * hch::PATTERN_BINS * 4);
                P.take(hl->d_fine, (na + (hist ? 2 * na : 0) + fine_tiles + hist + totals) * 4);
                P.take(hl->d_nbr_prefix, ((size_t)n_levels * batch + 1) * 4);
                P.take(hl->d_child_prefix, ((size_t)n_levels * batch + 1) * 4);
            };
            Pieces size, place;
            lay(size);
            if (device_malloc((void **)&place.base, size.used) != hipSuccess) st = fail(HCH_ENOMEM, "hipMalloc(pattern and fine order) failed");
            else {
                hl->blocks.push_back(place.base);
                lay(place);
            }
            for (int l = 0; l < n_levels && st == HCH_OK; ++l) {
                Level &L = hl->lv[l];
                const size_t tiles = (size_t)((L.n_total + hch::PATTERN_TILE - 1) / hch::PATTERN_TILE);
                L.dorder = hl->d_order + hl->sort_off[l];
                if (L.in_block) continue;
                if (device_malloc((void **)&L.dmask27, std::max<size_t>((size_t)L.n_total, 64) * 4) != hipSuccess) { st = fail(HCH_ENOMEM, "hipMalloc(mask27) failed"); break; }
                if (device_malloc((void **)&L.dtilemask, std::max<size_t>(tiles, 64) * 4) != hipSuccess) { st = fail(HCH_ENOMEM, "hipMalloc(tile masks) failed"); break; }
            }
            if (st == HCH_OK) {
                uint32_t *p = hl->d_fine;
                hl->set.sorted_mask = p; p += na;
                if (hist) {
                    hl->set.fine_mask = p; p += na;
                    hl->set.fine_order = (int32_t *)p; p += na;
                    hl->set.fine_hist = (int32_t *)p; p += hist;
                    hl->set.fine_total = (int32_t *)p; p += totals;
                    for (int l = 0; l < n_levels; ++l)
                        if (hl->set.fine_tiles[l]) {
                            hl->lv[l].dforder = hl->set.fine_order + hl->sort_off[l];
                            hl->lv[l].dftilemask = p;
                            p += (hl->lv[l].n_total + hch::PATTERN_TILE - 1) / hch::PATTERN_TILE;
                        }
                }
            }
        }
        if (st == HCH_OK && with_device) {
            hl->set.batch = batch;
            hl->nbr_prefix.assign((size_t)n_levels * batch + 1, 0);
            hl->child_prefix.assign((size_t)n_levels * batch + 1, 0);
            for (int l = 0; l < n_levels; ++l) {
                Level &L = hl->lv[l];
                hl->set.view[l] = L.view();
                hl->set.coords[l] = L.dcoords;
                hl->set.nbr[l] = L.dnbr;
                hl->set.child[l] = L.dchild;
                hl->set.mask27[l] = L.dmask27;
                hl->set.sort_off[l] = hl->sort_off[l];
                hl->set.level_tile0[l] = hl->nbr_prefix[(size_t)l * batch];
                for (int v = 0; v < batch; ++v) {
                    const int32_t tiles = (int32_t)((L.N[v + 1] - L.N[v] + 255) / 256);
                    const size_t e = (size_t)l * batch + v;
                    hl->nbr_prefix[e + 1] = hl->nbr_prefix[e] + tiles;
                    hl->child_prefix[e + 1] = hl->child_prefix[e] + (l > 0 && L.ratio == 2 ? tiles : 0);
                }
            }
            hl->set.sort_key = hl->d_sort_key;
            hl->set.tile_hist = hl->d_tile_hist;
            for (int l = 0; l < n_levels; ++l) {
                hl->set.level_tile0[l] = hl->nbr_prefix[(size_t)l * batch];
                hl->set.level_tiles[l] = hl->nbr_prefix[(size_t)(l + 1) * batch] - hl->nbr_prefix[(size_t)l * batch];
                hl->set.hist_off[l] = hl->set.level_tile0[l] * hch::PATTERN_BINS;
            }
            hipError_t e = hipMemcpyAsync(hl->d_nbr_prefix, hl->nbr_prefix.data(), hl->nbr_prefix.size() * 4, hipMemcpyHostToDevice, s);
            if (e == hipSuccess) e = hipMemcpyAsync(hl->d_child_prefix, hl->child_prefix.data(), hl->child_prefix.size() * 4, hipMemcpyHostToDevice, s);
            if (e != hipSuccess) st = fail(HCH_EHIP, std::string("hipMemcpyAsync: ") + hipGetErrorString(e));
            if (st == HCH_OK) st = hch_build_neighbours(hl, -1, s);
        }
        if (st == HCH_OK && with_device) {
            hipError_t e = hipStreamSynchronize(s);
            if (e != hipSuccess) st = fail(HCH_EHIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(e));
        }
        // occupied-neighbour count of every level (for the algorithmic traffic that is reported, and conv_bf16_ok)
        if (st == HCH_OK && with_device) {
            unsigned long long *d_cnt = nullptr;
            std::vector<unsigned long long> h_cnt((size_t)n_levels, 0);
            if (device_malloc((void **)&d_cnt, (size_t)n_levels * 8) != hipSuccess) st = fail(HCH_ENOMEM, "hipMalloc failed");
            if (st == HCH_OK) {
                hipError_t e = hipMemsetAsync(d_cnt, 0, (size_t)n_levels * 8, s);
                for (int l = 0; l < n_levels && e == hipSuccess; ++l) {
                    const int64_t n = hl->lv[l].n_total;
                    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(512, (n + 1023) / 1024));
                    HCH_LAUNCH(hch::count_taps_kernel, dim3(grid), dim3(256), 0, s, (const uint32_t *)hl->lv[l].dmask27, n, d_cnt + l);
                    e = hipGetLastError();
                }
                if (e == hipSuccess) e = hipMemcpyAsync(h_cnt.data(), d_cnt, (size_t)n_levels * 8, hipMemcpyDeviceToHost, s);
                if (e == hipSuccess) e = hipStreamSynchronize(s);
                if (e != hipSuccess) st = fail(HCH_EHIP, std::string("neighbour count: ") + hipGetErrorString(e));
                for (int l = 0; l < n_levels; ++l) hl->lv[l].nbr_valid = (int64_t)h_cnt[l];
            }
            if (d_cnt) (void)hipFree(d_cnt);
        }
    } catch (const std::bad_alloc &) {
        st = fail(HCH_ENOMEM, "hch_build_levels: out of host memory");
    }

    if (st != HCH_OK) {
        hch_free_levels(hl);
        // out of memory while the checks on the device held some (up to OCCUPANCY_BYTES and the positions): once more
        // without it
        if (st != HCH_ENOMEM || occ.mem.ptrs.empty()) return st;
        occ.mem.release();
        return build_impl(coords_xyz, model_offsets, batch, resolution, n_levels, ratios, stream, with_device, device_tables, out, true);
    }
    *out = hl;
    return HCH_OK;
}

extern "C" hch_status hch_build_levels(const int32_t *coords_xyz, const int64_t *model_offsets,
                                       int32_t batch, int32_t resolution, int32_t n_levels,
                                       void *stream, hch_levels **out)
{
    return build_impl(coords_xyz, model_offsets, batch, resolution, n_levels, nullptr, stream, true, false, out);
}

extern "C" hch_status hch_build_levels_device(const int32_t *coords_xyz, const int64_t *model_offsets,
                                              int32_t batch, int32_t resolution, int32_t n_levels,
                                              void *stream, hch_levels **out)
{
    return build_impl(coords_xyz, model_offsets, batch, resolution, n_levels, nullptr, stream, true, true, out);
}

extern "C" hch_status hch_build_levels_ratios(const int32_t *coords_xyz, const int64_t *model_offsets,
                                              int32_t batch, int32_t resolution, int32_t n_levels,
                                              const int32_t *ratios, int32_t device_tables,
                                              void *stream, hch_levels **out)
{
    if (n_levels > 1 && !ratios) {
        if (out) *out = nullptr;
        return fail(HCH_EINVAL, "hch_build_levels_ratios: null ratios");
    }
    static const int32_t none[1] = {2};
    return build_impl(coords_xyz, model_offsets, batch, resolution, n_levels, ratios ? ratios : none, stream, true,
                      device_tables != 0, out);
}

extern "C" hch_status hch_build_tables_host(const int32_t *coords_xyz, const int64_t *model_offsets,
                                            int32_t batch, int32_t resolution, int32_t n_levels,
                                            hch_levels **out)
{
    return build_impl(coords_xyz, model_offsets, batch, resolution, n_levels, nullptr, nullptr, false, false, out);
}

extern "C" hch_status hch_level_info(const hch_levels *levels, int32_t level, hch_level_desc *out)
{
    if (!levels || !out || level < 0 || level >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_level_info: bad argument");
    const Level &L = levels->lv[level];
    out->ubar = L.ubar; out->batch = L.b;
    out->n_total = L.n_total; out->m_total = L.m_total; out->r_total = L.r_total;
    out->nbr_valid = L.nbr_valid;
    out->mbar = L.mbar.data(); out->rbar = L.rbar.data(); out->attempts = L.attempts.data();
    out->M = L.M.data(); out->R = L.R.data(); out->N = L.N.data();
    out->coords_host = L.hcoords ? L.hcoords : L.coords.data();
    out->H_host = L.hH ? L.hH : L.H.data(); out->T_host = L.hT ? L.hT : L.T.data(); out->Phi_host = L.hPhi ? L.hPhi : L.Phi.data();
    out->V_host = L.hV ? L.hV : L.V.data();
    out->H = L.dH; out->T = L.dT; out->Phi = L.dPhi; out->V = L.dV; out->coords = L.dcoords;
    out->nbr27 = L.dnbr; out->child8 = L.dchild;
    out->row_order = L.dorder; out->tile_taps = L.dtilemask;
    return HCH_OK;
}

// ---------------------------------------------------------------------------------------
// hash2col / col2hash
// ---------------------------------------------------------------------------------------

static hch_status get_level(const hch_levels *levels, int32_t level, const Level **L, const char *who)
{
    if (!levels || level < 0 || level >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, std::string(who) + ": bad level");
    *L = &levels->lv[level];
    if (!(*L)->dnbr) return fail(HCH_EINVAL, std::string(who) + ": levels were built without device tables");
    return HCH_OK;
}

static inline int elem_size(hch_dtype d) { return d == HCH_BF16 ? 2 : 4; }

// voxels per workgroup for the gather / scatter kernels: large tiles when there are many voxels,
// smaller ones when the level is small so that the chip still gets a few thousand workgroups
static int tile_voxels(int64_t n, int lo, int hi)
{
    int64_t tv = n / 2048;
    tv = std::max<int64_t>(lo, std::min<int64_t>(hi, tv));
    return (int)tv;
}

static hch_status do_hash2col(const Level &L, hch_dtype dtype, const void *X, int c_in,
                              int64_t row_begin, int64_t rows, void *col, hipStream_t s)
{
    if (rows == 0) return HCH_OK;
    const int es = elem_size(dtype);
    const int row_bytes = c_in * es;
    // per voxel: 27 indices and its own feature row in (neighbour re-reads are cache hits),
    // 27 rows out (zeros included: the GEMM operand needs them)
    const double bytes = (double)rows * (108.0 + 28.0 * row_bytes);
    const int tv = tile_voxels(rows, 8, 128);
    const size_t lds = (size_t)tv * 27 * 4;
    const unsigned n_tiles = (unsigned)((rows + tv - 1) / tv);
    const unsigned grid = (n_tiles + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD;
    if (row_bytes % 16 == 0 && aligned16(X) && aligned16(col)) {
        hch::LaunchTimer lt(HCH_KERNEL_ID("hash2col_kernel<unsigned int __vector(4)>"), s, bytes, 0.0);
        HCH_LAUNCH(hch::hash2col_kernel<hch::u32x4>, dim3(grid), dim3(256), lds, s,
                           (const hch::u32x4 *)X, L.dnbr, (hch::u32x4 *)col, row_begin, rows, row_bytes / 16, tv, n_tiles);
    } else {
        hch::LaunchTimer lt(dtype == HCH_F32 ? HCH_KERNEL_ID("hash2col_kernel<float>") : HCH_KERNEL_ID("hash2col_kernel<unsigned short>"), s, bytes, 0.0);
        if (dtype == HCH_F32)
            HCH_LAUNCH(hch::hash2col_kernel<float>, dim3(grid), dim3(256), lds, s,
                               (const float *)X, L.dnbr, (float *)col, row_begin, rows, c_in, tv, n_tiles);
        else
            HCH_LAUNCH(hch::hash2col_kernel<uint16_t>, dim3(grid), dim3(256), lds, s,
                               (const uint16_t *)X, L.dnbr, (uint16_t *)col, row_begin, rows, c_in, tv, n_tiles);
    }
    HCH_LAUNCH_CHECK("hash2col");
    return HCH_OK;
}

extern "C" hch_status hch_hash2col(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                   const void *X, int32_t c_in, int64_t row_begin,
                                   int64_t row_count, void *col, void *stream)
{
    const Level *L;
    hch_status st = get_level(levels, level, &L, "hch_hash2col");
    if (st != HCH_OK) return st;
    if (!X || !col || c_in <= 0 || (dtype != HCH_F32 && dtype != HCH_BF16))
        return fail(HCH_EINVAL, "hch_hash2col: bad argument");
    if (row_begin < 0 || row_count < 0 || row_begin + row_count > L->n_total)
        return fail(HCH_EINVAL, "hch_hash2col: row range outside the level");
    return do_hash2col(*L, dtype, X, c_in, row_begin, row_count, col, (hipStream_t)stream);
}

// planes: dcol is stored tap-major, [27][n][c_in] (the library's own layout between the data
// gradient product and this gather; needs c_in % 4 == 0), instead of [n][27*c_in]
static hch_status do_col2hash(const Level &L, const float *dcol, int c_in, float *dX, bool planes, hipStream_t s)
{
    if (L.n_total == 0) return HCH_OK;
    // per voxel: 27 indices in, one c_in row per occupied neighbour in, one row out
    const double bytes = (double)L.n_total * (108.0 + 4.0 * c_in) + (double)L.nbr_valid * 4.0 * c_in;
    const bool vec = c_in % 4 == 0 && aligned16(dcol) && aligned16(dX);
    if (planes && !vec) return fail(HCH_EINVAL, "col2hash: tap-major layout needs aligned 4-channel units");
    hch::LaunchTimer lt(planes ? HCH_KERNEL_ID("col2hash_kernel<4, true>")
                               : (vec ? HCH_KERNEL_ID("col2hash_kernel<4, false>") : HCH_KERNEL_ID("col2hash_kernel<1, false>")),
                        s, bytes, (double)L.nbr_valid * c_in);
    const int cu = vec ? c_in / 4 : c_in;
    const int tv = std::max(4, std::min(128, 256 / cu));
    const size_t lds = (size_t)tv * 27 * 4;
    const unsigned n_tiles = (unsigned)((L.n_total + tv - 1) / tv);
    const unsigned grid = (n_tiles + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD;
    if (planes)
        HCH_LAUNCH((hch::col2hash_kernel<4, true>), dim3(grid), dim3(256), lds, s, dcol, L.dnbr, dX,
                           L.n_total, c_in, tv, n_tiles);
    else if (vec)
        HCH_LAUNCH((hch::col2hash_kernel<4, false>), dim3(grid), dim3(256), lds, s, dcol, L.dnbr, dX,
                           L.n_total, c_in, tv, n_tiles);
    else
        HCH_LAUNCH((hch::col2hash_kernel<1, false>), dim3(grid), dim3(256), lds, s, dcol, L.dnbr, dX,
                           L.n_total, c_in, tv, n_tiles);
    HCH_LAUNCH_CHECK("col2hash");
    return HCH_OK;
}

extern "C" hch_status hch_col2hash(const hch_levels *levels, int32_t level, const float *dcol,
                                   int32_t c_in, float *dX, void *stream)
{
    const Level *L;
    hch_status st = get_level(levels, level, &L, "hch_col2hash");
    if (st != HCH_OK) return st;
    if (!dcol || !dX || c_in <= 0) return fail(HCH_EINVAL, "hch_col2hash: bad argument");
    return do_col2hash(*L, dcol, c_in, dX, false, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------
// GEMM launches
// ---------------------------------------------------------------------------------------

// slices of a split reduction are multiples of the reduction length of one tile
static inline int k_gran(hch_dtype dtype) { return dtype == HCH_BF16 ? hch::BF16_BK : hch::GEMM_BK; }

// tile shape and split of one product
// hch_set_lean_loops: 0 = every product of launch_gemm_* takes the pointer-based form of its main loop
static std::atomic<int> g_lean_loops{1};

struct GemmPlan {
    int bm, bn, wm;
    int splits, k_per_split;
};

// fwd-like products (M = voxels): wide tiles when there are many row tiles, 64-row tiles and a
// split of the reduction when the level is too small to fill the chip
static GemmPlan plan_rows(int64_t M, int N, int K, bool allow_split, int gran = hch::GEMM_BK)
{
    GemmPlan p;
    p.bn = N <= 16 ? 16 : (N <= 32 ? 32 : 64);
    p.bm = 128; p.wm = 4;
    const int64_t n_tiles = (N + p.bn - 1) / p.bn;
    int64_t blocks = (M + 127) / 128 * n_tiles;
    if (p.bn == 64 && blocks < 1024) { p.bm = 64; p.wm = 2; blocks = (M + 63) / 64 * n_tiles; }
    p.splits = 1; p.k_per_split = K + hch::GEMM_BK;
    if (allow_split && blocks < 512 && K >= 512) {
        // as many slices as fit the chip in one round of workgroups (4 per CU with the 64-row
        // tile, 3 with the 128-row ones): a second, nearly empty round costs as much as a full one
        const int64_t resident = p.bm == 64 ? 1024 : 768;
        int64_t want = std::min<int64_t>(resident / blocks, K / 256);
        want = std::max<int64_t>(1, want);
        int64_t kps = (K + want - 1) / want;
        kps = (kps + gran - 1) / gran * gran;
        p.k_per_split = (int)kps;
        p.splits = (int)((K + kps - 1) / kps);
    }
    return p;
}

// weight-gradient product (M = 27*c_in, N = c_out, reduction over n voxels split in slices)
static GemmPlan plan_wgrad(int64_t n, int c_in, int c_out, int taps = 27, int gran = hch::GEMM_BK)
{
    GemmPlan p;
    const int Kc = taps * c_in;
    p.bn = c_out <= 16 ? 16 : (c_out <= 32 ? 32 : 64);
    p.bm = 128; p.wm = 4;
    const int64_t tiles = (int64_t)((Kc + 127) / 128) * ((c_out + p.bn - 1) / p.bn);
    int64_t want = std::max<int64_t>(1, 768 / tiles);   // one round of workgroups, 3 per CU
    // bf16 kernel: a multiple of 8 slices, each XCD (32 CUs, 96 workgroups at a time) taking
    // whole slices, if that still fills most of the chip
    if (gran == hch::BF16_BK && tiles <= 96 && (96 / tiles) * tiles >= 64) want = 8 * (96 / tiles);
    want = std::min<int64_t>(want, std::max<int64_t>(1, (n + 255) / 256));
    // fp32 kernel: a multiple of 8 slices as well (each XCD takes whole slices and gathers their
    // voxels once for all its tiles) where that costs at most an eighth of the slices
    if (gran != hch::BF16_BK && want >= 8) want = want / 8 * 8;
    int64_t rows = (n + want - 1) / want;
    rows = std::max<int64_t>(gran, (rows + gran - 1) / gran * gran);
    p.k_per_split = (int)rows;
    p.splits = (int)std::max<int64_t>(1, (n + rows - 1) / rows);
    // keep the count a multiple of 8 (rounding the slice length up may have dropped a few slices;
    // the extra ones are empty and write zeros)
    if (want >= 8 && want % 8 == 0 && p.splits <= want) p.splits = (int)((p.splits + 7) / 8 * 8);
    return p;
}

static inline bool k_split_aligned(const GemmPlan &p) { return p.k_per_split % 4 == 0; }

template <typename TIN, int AMODE, bool B_KC>
static hch_status launch_gemm_t(const GemmPlan &plan, const void *A, const void *B, float *C,
                                const int32_t *nbr, int M, int N, int K, int64_t lda, int64_t ldb,
                                int64_t ldc, int64_t c_split_stride, double alg_bytes, hipStream_t s,
                                int c_planes = 0, int taps = 27, int b_wrap = 0, int64_t b_tap_stride = 0,
                                const int32_t *rowmap = nullptr, const uint32_t *tilemask = nullptr, int64_t a_rows = 0,
                                const uint32_t *rowmask = nullptr, int mask_c = 1)
{
    if (M <= 0 || N <= 0) return HCH_OK;
    GemmPlan p = plan;
    // vector path: every 4-element unit is aligned and wholly inside or outside its matrix
    const uintptr_t amask = sizeof(TIN) * 4 - 1;
    const bool a_fast_ok = (AMODE == hch::A_COLS) ? (M % 4 == 0) : (K % 4 == 0 || AMODE == hch::A_GATHER_T);
    const bool b_fast_ok = B_KC ? (K % 4 == 0) : (N % 4 == 0);
    const bool vec = (lda % 4 == 0) && (ldb % 4 == 0) && a_fast_ok && b_fast_ok &&
                     !(reinterpret_cast<uintptr_t>(A) & amask) && !(reinterpret_cast<uintptr_t>(B) & amask) &&
                     (k_split_aligned(p));
    if (b_wrap && !vec) return fail(HCH_EINVAL, "gemm: in-place weight reading needs aligned operands");
    if (!vec || AMODE != hch::A_GATHER || taps != 27) rowmap = nullptr;     // rows in pattern order and tap skipping:
    if (!rowmap) tilemask = nullptr;                                        // the vector path of the 3x3x3 gather only
    if (!vec && p.bm == 64) { p.bm = 128; p.wm = 4; }   // the generic path has the 128-row tiles only
    const int c_vec_ok = (c_planes > 0 ? c_planes % 4 == 0 : ldc % 4 == 0) && (c_split_stride % 4 == 0) && aligned16(C);
    const unsigned m_tiles = (unsigned)((M + p.bm - 1) / p.bm);
    // XCD-contiguous row tiles only where rows are voxels and there are enough tiles to keep
    // every XCD busy (an exact multiple of 8 cannot be told apart from the plain order, so
    // pad it by 8 as well)
    // (in pattern order neighbouring tiles have the same amount of work: chunks of tiles go to the
    // XCDs in turn, see xcd_chunk_tile, and the grid is a whole number of rounds of chunks)
    const bool remap = (AMODE == hch::A_GATHER || AMODE == hch::A_ROWS) && m_tiles >= 256 && !tilemask;
    const unsigned gx = tilemask ? hch::skip_grid(m_tiles, hch::skip_chunk(m_tiles * (unsigned)(p.bm / 64), (unsigned)(p.bm / 64)))
                                 : (remap ? (m_tiles / hch::NUM_XCD + 1) * hch::NUM_XCD : m_tiles);
    const unsigned n_tiles = (unsigned)((N + p.bn - 1) / p.bn);
    // reductions over the voxels cut into a multiple of 8 slices: one XCD per slice
    const int flat = ((AMODE == hch::A_GATHER_T || AMODE == hch::A_COLS) && p.splits >= 8 && p.splits % (int)hch::NUM_XCD == 0) ? p.splits : 0;
    const dim3 grid = flat ? dim3((unsigned)p.splits * m_tiles * n_tiles) : dim3(gx, n_tiles, (unsigned)p.splits);
    // the kernel's name as a profiler prints it: gemm_f32_kernel<TIN, BM, BN, BK, WM, AMODE, B_KC>
    static int ids[2][3][2][4];                        // [lean][planes / skipping][vector path][tile shape]
    static const bool ids_ready = [] { memset(ids, 0xFF, sizeof ids); return true; }();
    (void)ids_ready;
    const int cfg = p.bm == 64 ? 0 : (p.bn == 16 ? 1 : (p.bn == 32 ? 2 : 3));
    const int v = vec ? 1 : 0, pl = c_planes > 0 ? 1 : (tilemask ? 2 : 0);
    if (pl == 1 && p.bn != 64) return fail(HCH_EINVAL, "gemm: plane-wise output needs the 64-column tile");
    // The lean loop (buffer loads, scalar offsets): float gathers of a 3x3x3 neighbourhood whose
    // operands stay below 2 GiB each, so that 32-bit byte offsets reach everything and a negative
    // offset is out of range; row indices must fit the 24-bit multiply.  Gathering along the
    // reduction axis a tile must lie within one tap (rows of a multiple of 32 channels).
    constexpr bool gather_mode = (AMODE == hch::A_GATHER || AMODE == hch::A_GATHER_T);
    constexpr bool lean_mode = (AMODE == hch::A_GATHER || AMODE == hch::A_ROWS || ((AMODE == hch::A_GATHER_T || AMODE == hch::A_COLS) && !B_KC)) &&
                               sizeof(TIN) == 4;
    bool lean = false;
    // rows of 16 channels (not a multiple of 32): tiles of 16 reduction indices, one tap each
    const bool lean16 = AMODE == hch::A_GATHER && !B_KC && lda % 32 == 16 && p.bm == 128 && p.bn == 32 &&
                        (p.splits == 1 || p.k_per_split % 16 == 0);
    if constexpr (lean_mode) {
        const int64_t lim = (int64_t)1 << 31;
        if constexpr (gather_mode) {
            const int64_t idx_rows = AMODE == hch::A_GATHER ? M : K;
            int64_t b_bytes;
            if (AMODE == hch::A_GATHER_T) b_bytes = (int64_t)K * ldb * 4;
            else if (B_KC) b_bytes = ((int64_t)(taps - 1) * (b_tap_stride < 0 ? -b_tap_stride : b_tap_stride) + (int64_t)N * ldb) * 4;
            else b_bytes = (int64_t)taps * lda * ldb * 4;
            lean = vec && c_planes == 0 && taps == 27 && nbr && a_rows > 0 && a_rows < ((int64_t)1 << 23) && lda * 4 < ((int64_t)1 << 23) &&
                   a_rows * lda * 4 < lim && idx_rows * taps * 4 < lim && b_bytes < lim &&
                   (AMODE == hch::A_GATHER_T || ((lda % 32 == 0 || lean16) && (B_KC ? b_wrap == (int)lda : b_wrap == 0)));
        } else {
            // plain operands (the products of the columns algorithm): row-major A needs whole tiles,
            // K and the slices multiples of 32; k-major A and B may end anywhere (their buffers are
            // described slice by slice)
            const int64_t a_bytes = (int64_t)(AMODE == hch::A_ROWS ? M : K) * lda * 4;
            const int64_t b_bytes = (int64_t)(B_KC ? N : K) * ldb * 4;
            lean = vec && c_planes == 0 && b_wrap == 0 && a_bytes < lim && b_bytes < lim &&
                   (AMODE == hch::A_COLS || (K % 32 == 0 && (p.splits == 1 || p.k_per_split % 32 == 0)));
        }
    }
    if (!g_lean_loops.load(std::memory_order_relaxed)) lean = false;
    if (tilemask) lean = false;        // rows in an order, taps left out: conv_split_kernel, or operands beyond the lean loop's reach
    const int ln = lean ? 1 : 0;
    if (ids[ln][pl][v][cfg] < 0) {
        char nm[128];
        // all eleven template arguments, as a profiler prints the instantiation
        snprintf(nm, sizeof nm, "gemm_f32_kernel<%s, %d, %d, 32, %d, %d, %s, %s, %s, %s, %s>",
                 sizeof(TIN) == 4 ? "float" : "unsigned short", p.bm, p.bm == 64 ? 64 : p.bn, p.wm,
                 (int)AMODE, B_KC ? "true" : "false", v ? "true" : "false", pl == 1 ? "true" : "false",
                 pl == 2 ? "true" : "false", lean ? "true" : "false");
        ids[ln][pl][v][cfg] = hch::Profiler::get().id_for(nm);
    }
    int kid = ids[ln][pl][v][cfg];
    if (lean && lean16)
        kid = HCH_KERNEL_ID("gemm_f32_kernel<float, 128, 32, 16, 4, 2, false, true, false, false, true>");
    const bool short_k = AMODE == hch::A_ROWS && B_KC && pl == 1 && vec && p.bm == 128 && K <= 16 && p.splits == 1;
    if (short_k) kid = HCH_KERNEL_ID("gemm_f32_kernel<float, 128, 64, 16, 4, 0, true, true, true, false, false>");
    hch::LaunchTimer lt(kid, s, alg_bytes, 2.0 * M * (double)N * K);
#define HCH_GEMM_ARGS (const TIN *)A, (const TIN *)B, C, nbr, M, N, K, lda, ldb, ldc, p.k_per_split, c_split_stride, c_vec_ok, \
                      m_tiles, c_planes, taps, b_wrap, b_tap_stride, rowmap, tilemask, flat, rowmask, mask_c
#define HCH_GEMM_CASE(BM_, BN_, BK_, WM_, VEC_, PL_)                                                                \
    HCH_LAUNCH((hch::gemm_f32_kernel<TIN, BM_, BN_, BK_, WM_, AMODE, B_KC, VEC_, PL_>), grid, dim3(256), 0, s, HCH_GEMM_ARGS)
#define HCH_GEMM_SKIP_CASE(BM_, BN_, WM_)                                                                           \
    HCH_LAUNCH((hch::gemm_f32_kernel<TIN, BM_, BN_, 32, WM_, hch::A_GATHER, B_KC, true, false, true>), grid, dim3(256), 0, s, HCH_GEMM_ARGS)
    if constexpr (AMODE == hch::A_ROWS && B_KC) {
        if (pl == 1) {
            if (vec) {
                if (p.bm == 64) HCH_GEMM_CASE(64, 64, 32, 2, true, true);
                else if (short_k) HCH_GEMM_CASE(128, 64, 16, 4, true, true);      // a reduction of at most 16: one half-size tile
                else HCH_GEMM_CASE(128, 64, 32, 4, true, true);
            }
            else HCH_GEMM_CASE(128, 64, 32, 4, false, true);
            HCH_LAUNCH_CHECK("gemm_f32_kernel");
            return HCH_OK;
        }
    }
#define HCH_GEMM_LEAN_CASE(BM_, BN_, WM_)                                                                            \
    HCH_LAUNCH((hch::gemm_f32_kernel<TIN, BM_, BN_, 32, WM_, AMODE, B_KC, true, false, false, true>), grid, dim3(256), 0, s, HCH_GEMM_ARGS)
    if constexpr (lean_mode) {
        if (lean) {
            if constexpr (AMODE == hch::A_GATHER && !B_KC) {
                if (lean16) {
                    HCH_LAUNCH((hch::gemm_f32_kernel<TIN, 128, 32, 16, 4, AMODE, B_KC, true, false, false, true>), grid, dim3(256), 0, s, HCH_GEMM_ARGS);
                    HCH_LAUNCH_CHECK("gemm_f32_kernel");
                    return HCH_OK;
                }
            }
            if (p.bm == 64) HCH_GEMM_LEAN_CASE(64, 64, 2);
            else if (p.bn == 16) HCH_GEMM_LEAN_CASE(128, 16, 4);
            else if (p.bn == 32) HCH_GEMM_LEAN_CASE(128, 32, 4);
            else HCH_GEMM_LEAN_CASE(128, 64, 4);
            HCH_LAUNCH_CHECK("gemm_f32_kernel");
            return HCH_OK;
        }
    }
#undef HCH_GEMM_LEAN_CASE
    if constexpr (AMODE == hch::A_GATHER) {
        if (vec && tilemask) {      // rows in pattern order, absent taps left out
            if (p.bm == 64) HCH_GEMM_SKIP_CASE(64, 64, 2);
            else if (p.bn == 16) HCH_GEMM_SKIP_CASE(128, 16, 4);
            else if (p.bn == 32) HCH_GEMM_SKIP_CASE(128, 32, 4);
            else HCH_GEMM_SKIP_CASE(128, 64, 4);
            HCH_LAUNCH_CHECK("gemm_f32_kernel");
            return HCH_OK;
        }
    }
    if (vec) {
        if (p.bm == 64) HCH_GEMM_CASE(64, 64, 32, 2, true, false);
        else if (p.bn == 16) HCH_GEMM_CASE(128, 16, 32, 4, true, false);
        else if (p.bn == 32) HCH_GEMM_CASE(128, 32, 32, 4, true, false);
        else HCH_GEMM_CASE(128, 64, 32, 4, true, false);
    } else {
        // odd channel counts / unaligned operands: one generic shape is enough
        if (p.bn == 16) HCH_GEMM_CASE(128, 16, 32, 4, false, false);
        else if (p.bn == 32) HCH_GEMM_CASE(128, 32, 32, 4, false, false);
        else HCH_GEMM_CASE(128, 64, 32, 4, false, false);
    }
#undef HCH_GEMM_CASE
#undef HCH_GEMM_SKIP_CASE
#undef HCH_GEMM_ARGS
    HCH_LAUNCH_CHECK("gemm_f32_kernel");
    return HCH_OK;
}

// bf16 operands on the bf16 matrix instruction (gemm_bf16_kernel): whether the operands meet its
// alignment rules; products that do not go to the kernel that widens to fp32 on load
template <int AMODE, bool B_KC>
static bool bf16_mfma_ok(const GemmPlan &p, const void *A, const void *B, int M, int N, int K, int64_t lda,
                         int64_t ldb, int c_planes, int b_wrap)
{
    constexpr bool a_k_fast = (AMODE == hch::A_ROWS || AMODE == hch::A_GATHER);
    if (c_planes > 0 || lda % 8 != 0 || ldb % 8 != 0 || !aligned16(A) || !aligned16(B)) return false;
    if (p.splits > 1 && p.k_per_split % hch::BF16_BK != 0) return false;
    if (b_wrap % hch::BF16_BK != 0) return false;
    if (a_k_fast ? (K % 8 != 0) : (M % 8 != 0 || p.bm != 128)) return false;
    if (B_KC ? (K % 8 != 0) : (N % 8 != 0)) return false;
    return true;
}

template <int AMODE, bool B_KC>
static hch_status launch_gemm_bf16(const GemmPlan &p, const void *A, const void *B, float *C,
                                   const int32_t *nbr, int M, int N, int K, int64_t lda, int64_t ldb,
                                   int64_t ldc, int64_t c_split_stride, double alg_bytes, hipStream_t s,
                                   int taps, int b_wrap, int64_t b_tap_stride, const int32_t *nbr_t, int64_t a_rows = 0)
{
    if (M <= 0 || N <= 0) return HCH_OK;
    // index rows [voxel][tap], or their tap-major copy [tap][voxel] (voxels = rows of the output
    // when gathering along the reduction axis, the reduction length when gathering along the rows)
    const int64_t idx_row_stride = nbr_t ? 1 : taps;
    const int64_t idx_tap_stride = nbr_t ? (AMODE == hch::A_GATHER_T ? K : M) : 1;
    if (nbr_t) nbr = nbr_t;
    const int c_vec_ok = (ldc % 4 == 0) && (c_split_stride % 4 == 0) && aligned16(C);
    const unsigned m_tiles = (unsigned)((M + p.bm - 1) / p.bm);
    const bool remap = (AMODE == hch::A_GATHER || AMODE == hch::A_ROWS) && m_tiles >= 256;
    const unsigned gx = remap ? (m_tiles / hch::NUM_XCD + 1) * hch::NUM_XCD : m_tiles;
    const unsigned n_tiles = (unsigned)((N + p.bn - 1) / p.bn);
    // reductions over the voxels cut into a multiple of 8 slices: one XCD per slice
    const int flat = ((AMODE == hch::A_GATHER_T || AMODE == hch::A_COLS) && p.splits % (int)hch::NUM_XCD == 0) ? p.splits : 0;
    const dim3 grid = flat ? dim3((unsigned)p.splits * m_tiles * n_tiles) : dim3(gx, n_tiles, (unsigned)p.splits);
    // the lean loop: see launch_gemm_t; rows of a multiple of 64 channels here (one tile, one tap)
    constexpr bool lean_mode = (AMODE == hch::A_GATHER || (AMODE == hch::A_GATHER_T && !B_KC));
    bool lean = false;
    if constexpr (lean_mode) {
        const int64_t lim = (int64_t)1 << 31;
        const int64_t idx_rows = AMODE == hch::A_GATHER ? M : K;
        int64_t b_bytes;
        if (AMODE == hch::A_GATHER_T) b_bytes = (int64_t)K * ldb * 2;
        else if (B_KC) b_bytes = ((int64_t)(taps - 1) * (b_tap_stride < 0 ? -b_tap_stride : b_tap_stride) + (int64_t)N * ldb) * 2;
        else b_bytes = (int64_t)taps * lda * ldb * 2;
        lean = taps == 27 && nbr && a_rows > 0 && a_rows < ((int64_t)1 << 23) && lda * 2 < ((int64_t)1 << 23) &&
               a_rows * lda * 2 < lim && idx_rows * taps * 4 < lim && b_bytes < lim &&
               (AMODE == hch::A_GATHER_T || (lda % hch::BF16_BK == 0 && (B_KC ? b_wrap == (int)lda : b_wrap == 0)));
    }
    if (!g_lean_loops.load(std::memory_order_relaxed)) lean = false;
    const bool big = lean && AMODE == hch::A_GATHER && p.bm == 128 && p.bn == 64 && p.splits == 1 && M >= 256 * 1024;
    static int ids[2][5] = {{-1, -1, -1, -1, -1}, {-1, -1, -1, -1, -1}};
    const int cfg = big ? 4 : (p.bm == 64 ? 0 : (p.bn == 16 ? 1 : (p.bn == 32 ? 2 : 3)));
    const int ln = lean ? 1 : 0;
    if (ids[ln][cfg] < 0) {
        char nm[128];
        snprintf(nm, sizeof nm, "gemm_bf16_kernel<%d, %d, %d, %d, %s, %s>", big ? 256 : p.bm, p.bm == 64 ? 64 : p.bn, p.wm,
                 (int)AMODE, B_KC ? "true" : "false", lean ? "true" : "false");
        ids[ln][cfg] = hch::Profiler::get().id_for(nm);
    }
    hch::LaunchTimer lt(ids[ln][cfg], s, alg_bytes, 2.0 * M * (double)N * K);
#define HCH_BF16_CASE(BM_, BN_, WM_)                                                                                 \
    HCH_LAUNCH((hch::gemm_bf16_kernel<BM_, BN_, WM_, AMODE, B_KC>), grid, dim3(256), 0, s,                  \
                       (const uint16_t *)A, (const uint16_t *)B, C, nbr, M, N, K, lda, ldb, ldc, p.k_per_split,     \
                       c_split_stride, c_vec_ok, m_tiles, idx_row_stride, idx_tap_stride, b_wrap, b_tap_stride, flat)
#define HCH_BF16_LEAN_CASE(BM_, BN_, WM_)                                                                            \
    HCH_LAUNCH((hch::gemm_bf16_kernel<BM_, BN_, WM_, AMODE, B_KC, true>), grid, dim3(256), 0, s,                    \
                       (const uint16_t *)A, (const uint16_t *)B, C, nbr, M, N, K, lda, ldb, ldc, p.k_per_split,     \
                       c_split_stride, c_vec_ok, m_tiles, idx_row_stride, idx_tap_stride, b_wrap, b_tap_stride, flat)
    if constexpr (lean_mode) {
        if (lean) {
            if (p.bm == 64) {
                if constexpr (AMODE == hch::A_GATHER) HCH_BF16_LEAN_CASE(64, 64, 2);
                else return fail(HCH_EINVAL, "gemm_bf16: 64-row tiles with a transposed A");
            }
            else if (p.bn == 16) HCH_BF16_LEAN_CASE(128, 16, 4);
            else if (p.bn == 32) HCH_BF16_LEAN_CASE(128, 32, 4);
            else if (big) {
                // many voxels, 64 output columns: 256-row tiles, a wavefront computes 64 x 64 outputs
                // and reads a third fewer operand bytes from LDS per matrix instruction
                if constexpr (AMODE == hch::A_GATHER) {

                    const unsigned mt = (unsigned)((M + 255) / 256);
                    const dim3 g2((mt / hch::NUM_XCD + 1) * hch::NUM_XCD, n_tiles, 1);
                    HCH_LAUNCH((hch::gemm_bf16_kernel<256, 64, 4, AMODE, B_KC, true>), g2, dim3(256), 0, s,
                       (const uint16_t *)A, (const uint16_t *)B, C, nbr, M, N, K, lda, ldb, ldc, p.k_per_split,
                       c_split_stride, c_vec_ok, mt, idx_row_stride, idx_tap_stride, b_wrap, b_tap_stride, flat);
                }
            }
            else HCH_BF16_LEAN_CASE(128, 64, 4);
            HCH_LAUNCH_CHECK("gemm_bf16_kernel");
            return HCH_OK;
        }
    }
#undef HCH_BF16_LEAN_CASE
    if (p.bm == 64) {
        if constexpr (AMODE == hch::A_ROWS || AMODE == hch::A_GATHER) HCH_BF16_CASE(64, 64, 2);
        else return fail(HCH_EINVAL, "gemm_bf16: 64-row tiles with a transposed A");
    }
    else if (p.bn == 16) HCH_BF16_CASE(128, 16, 4);
    else if (p.bn == 32) HCH_BF16_CASE(128, 32, 4);
    else HCH_BF16_CASE(128, 64, 4);
#undef HCH_BF16_CASE
    HCH_LAUNCH_CHECK("gemm_bf16_kernel");
    return HCH_OK;
}

template <int AMODE, bool B_KC>
static hch_status launch_gemm(hch_dtype dtype, const GemmPlan &p, const void *A, const void *B, float *C,
                              const int32_t *nbr, int M, int N, int K, int64_t lda, int64_t ldb,
                              int64_t ldc, int64_t c_split_stride, double alg_bytes, hipStream_t s,
                              int c_planes = 0, int taps = 27, int b_wrap = 0, int64_t b_tap_stride = 0,
                              const int32_t *nbr_t = nullptr, const int32_t *rowmap = nullptr, const uint32_t *tilemask = nullptr,
                              int64_t a_rows = 0 /* rows of the gathered matrix; 0: not known, no lean loop */,
                              const uint32_t *rowmask = nullptr /* per output row: which groups of mask_c columns to store (fp32 kernel) */,
                              int mask_c = 1)
{
    if (dtype == HCH_BF16 && bf16_mfma_ok<AMODE, B_KC>(p, A, B, M, N, K, lda, ldb, c_planes, b_wrap))
        return launch_gemm_bf16<AMODE, B_KC>(p, A, B, C, nbr, M, N, K, lda, ldb, ldc, c_split_stride, alg_bytes, s, taps, b_wrap, b_tap_stride, nbr_t, a_rows);
    if (dtype == HCH_BF16)
        return launch_gemm_t<uint16_t, AMODE, B_KC>(p, A, B, C, nbr, M, N, K, lda, ldb, ldc, c_split_stride, alg_bytes, s, c_planes, taps, b_wrap, b_tap_stride);
    return launch_gemm_t<float, AMODE, B_KC>(p, A, B, C, nbr, M, N, K, lda, ldb, ldc, c_split_stride, alg_bytes, s, c_planes, taps, b_wrap, b_tap_stride,
                                             rowmap, tilemask, a_rows, rowmask, mask_c);
}

// Register-direct gathered product (conv_direct_kernel): shape-only part of the plan, shared by
// the workspace query and the launch.  Used for products with at most 16 output columns (the
// first forward layer, data gradients into few channels): there a staged tile would be written
// to LDS and read back exactly once, and this kernel measured faster; wider outputs go to the
// LDS-tiled kernel, which measured faster there.
struct DirectPlan {
    bool ok;
    int rt, nt, S;
    bool check;
    int J, upt, step_t, step_q;
    int splits, j_per_split;
    unsigned wave_tiles, n_groups;
};

static DirectPlan plan_direct(int64_t M, int c, int N)
{
    DirectPlan d{};
    d.ok = M > 0 && c % 4 == 0 && N % 4 == 0 && N <= 16 && M * std::max(c, N) < ((int64_t)1 << 31) - 64 * std::max(c, N);
    if (!d.ok) return d;
    d.nt = 1; d.rt = 4; d.S = 4;
    d.check = (c % 16 != 0) || (N % (16 * d.nt) != 0);
    d.upt = c / 4;
    d.J = (27 * d.upt + 3) / 4;
    d.step_t = 4 / d.upt;
    d.step_q = 4 % d.upt;
    d.n_groups = (unsigned)((N + 16 * d.nt - 1) / (16 * d.nt));
    d.wave_tiles = (unsigned)((M + 16 * d.rt - 1) / (16 * d.rt));
    // small levels: slices of the reduction until every SIMD has a few waves
    const int64_t waves = (int64_t)d.wave_tiles * d.n_groups;
    int64_t want = waves >= 1536 ? 1 : std::max<int64_t>(1, std::min<int64_t>((2048 + waves - 1) / waves, d.J / (3 * d.S)));
    int jps = (int)((d.J + want - 1) / want);
    jps = (jps + d.S - 1) / d.S * d.S;
    d.j_per_split = jps;
    d.splits = (d.J + jps - 1) / jps;
    return d;
}

static hch_status launch_direct(const DirectPlan &d, const float *X, const int32_t *nbr, const float *Wm,
                                float *out, int64_t M, int c, int N, double alg_bytes, hipStream_t s, int flipped = 0,
                                const int32_t *rowmap = nullptr, const uint32_t *tilemask = nullptr)
{
    const unsigned blocks = (d.wave_tiles + 3) / 4;
    const bool skip = rowmap && tilemask;        // rows in pattern order, absent taps left out, chunks of tiles per XCD
    const dim3 grid(skip ? hch::skip_grid(blocks, hch::skip_chunk(d.wave_tiles, 4)) : (blocks / hch::NUM_XCD + 1) * hch::NUM_XCD, d.n_groups, (unsigned)d.splits);
    static int ids[2][2] = {{-1, -1}, {-1, -1}};
    const int b = d.check ? 1 : 0, k = skip ? 1 : 0;
    if (ids[k][b] < 0) {
        char nm[96];
        snprintf(nm, sizeof nm, "conv_direct_kernel<%d, %d, %d, %s, %s>", d.rt, d.nt, d.S, d.check ? "true" : "false", skip ? "true" : "false");
        ids[k][b] = hch::Profiler::get().id_for(nm);
    }
    hch::LaunchTimer lt(ids[k][b], s, alg_bytes, 2.0 * M * (double)N * 27.0 * c);
#define HCH_DIRECT_CASE(RT_, NT_, S_, CHECK_, SKIP_)                                                                \
    HCH_LAUNCH((hch::conv_direct_kernel<RT_, NT_, S_, CHECK_, SKIP_>), grid, dim3(256), 0, s, X, nbr, Wm, out,  \
                       (int)M, c, N, d.J, d.j_per_split, d.upt, d.step_t, d.step_q, d.wave_tiles, M * (int64_t)N, flipped, \
                       rowmap, tilemask)
    if (skip) { if (d.check) HCH_DIRECT_CASE(4, 1, 4, true, true); else HCH_DIRECT_CASE(4, 1, 4, false, true); }
    else { if (d.check) HCH_DIRECT_CASE(4, 1, 4, true, false); else HCH_DIRECT_CASE(4, 1, 4, false, false); }
#undef HCH_DIRECT_CASE
    HCH_LAUNCH_CHECK("conv_direct_kernel");
    return HCH_OK;
}

// gathered product into exactly 4 output columns (conv_narrow4_kernel)
static bool narrow4_ok(int64_t M, int c, int N)
{
    return N == 4 && (c == 16 || c == 32 || c == 64) && M > 0 && M * (int64_t)c < ((int64_t)1 << 31) - 64 * c;
}

static hch_status launch_narrow4(const float *X, const int32_t *nbr, const float *Wm, float *out, int64_t M, int c,
                                 double alg_bytes, hipStream_t s, int flipped = 0,
                                 const int32_t *rowmap = nullptr, const uint32_t *tilemask = nullptr)
{
    const unsigned wave_tiles = (unsigned)((M + 63) / 64);
    const unsigned blocks = (wave_tiles + 3) / 4;
    const bool skip = rowmap && tilemask;
    const dim3 grid(skip ? hch::skip_grid(blocks, hch::skip_chunk(wave_tiles, 4)) : (blocks / hch::NUM_XCD + 1) * hch::NUM_XCD);
    const int cc = c / 16;
    int kid;
    if (skip) kid = cc == 1 ? HCH_KERNEL_ID("conv_narrow4_kernel<1, true>") : (cc == 2 ? HCH_KERNEL_ID("conv_narrow4_kernel<2, true>") : HCH_KERNEL_ID("conv_narrow4_kernel<4, true>"));
    else kid = cc == 1 ? HCH_KERNEL_ID("conv_narrow4_kernel<1, false>") : (cc == 2 ? HCH_KERNEL_ID("conv_narrow4_kernel<2, false>") : HCH_KERNEL_ID("conv_narrow4_kernel<4, false>"));
    hch::LaunchTimer lt(kid, s, alg_bytes, 2.0 * M * 4.0 * 27.0 * c);
#define HCH_NARROW_CASE(CC_)                                                                                          \
    do {                                                                                                                \
        if (skip) HCH_LAUNCH((hch::conv_narrow4_kernel<CC_, true>), grid, dim3(256), 0, s, X, nbr, Wm, out, (int)M, wave_tiles, flipped, rowmap, tilemask); \
        else HCH_LAUNCH((hch::conv_narrow4_kernel<CC_, false>), grid, dim3(256), 0, s, X, nbr, Wm, out, (int)M, wave_tiles, flipped, rowmap, tilemask);     \
    } while (0)
    if (cc == 1) HCH_NARROW_CASE(1);
    else if (cc == 2) HCH_NARROW_CASE(2);
    else if (cc == 4) HCH_NARROW_CASE(4);
    else return fail(HCH_EINVAL, "conv_narrow4: channel count");
#undef HCH_NARROW_CASE
    HCH_LAUNCH_CHECK("conv_narrow4_kernel");
    return HCH_OK;
}

static hch_status launch_reduce(const float *part, float *out, int64_t n, int splits, hipStream_t s)
{
    const int kid = splits <= 16 ? HCH_KERNEL_ID("splitk_reduce_kernel<1>")
                    : (n >= 65536 || splits <= 256 ? HCH_KERNEL_ID("splitk_reduce_kernel<16>") : HCH_KERNEL_ID("splitk_reduce_kernel<64>"));
    hch::LaunchTimer lt(kid, s, 4.0 * n * (splits + 1.0), (double)n * splits);
    // few slices: a thread per output; many slices: 16 or 64 lanes per output, so that even a
    // small output (a 27 x 4 x 16 weight gradient) spreads over a few hundred workgroups
    if (splits <= 16)
        HCH_LAUNCH(hch::splitk_reduce_kernel<1>, dim3(blocks_for(n)), dim3(256), 0, s, part, out, n, splits, n);
    else if (n >= 65536 || splits <= 256)
        HCH_LAUNCH(hch::splitk_reduce_kernel<16>, dim3((unsigned)((n + 15) / 16)), dim3(256), 0, s, part, out, n, splits, n);
    else
        HCH_LAUNCH(hch::splitk_reduce_kernel<64>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, part, out, n, splits, n);
    HCH_LAUNCH_CHECK("splitk_reduce_kernel");
    return HCH_OK;
}

// One workgroup of the two weight-gradient kernels per CU; their partial sums, one tile per workgroup,
// fit the built-in array of hch_conv_bwd_weight_noalloc.
constexpr int64_t WG_RESIDENT = 256;
static_assert(WG_RESIDENT * hch::WG_UNITS * 16 * 64 * 4 <= HCH_NOALLOC_SCRATCH_BYTES, "wgrad_split_kernel: 28 MiB");
static_assert(WG_RESIDENT * hch::WGB_UNITS * 32 * 64 * 4 <= HCH_NOALLOC_SCRATCH_BYTES, "wgrad_bf16_kernel: 32 MiB");

// The weight gradient on split operands (wgrad_split_kernel): rows of `nbr` hold `taps` indices into
// the x_rows rows of X; `max_slices` partial sums fit the caller's workspace.
struct WgradSplitPlan { bool ok; int slices, m_tiles, n_tiles; };

static WgradSplitPlan plan_wgrad_split(int64_t n, int64_t x_rows, int c, int N, int taps, int64_t max_slices)
{
    WgradSplitPlan p{false, 1, 1, 1};
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit byte offsets reach everything, a negative one nothing; a workgroup's rows touch 28 taps
    if (x_rows * c * 4 >= lim || n * N * 4 >= lim || n * taps * 4 >= lim || x_rows >= (1 << 23) || c * 4 >= (1 << 23) || (c < 16 && taps > hch::WG_UNITS)) return p;
    if (N <= 16 || (int64_t)taps * c < 16) return p;
    // a workgroup needs some blocks of voxels to get going, gemm_f32_kernel is ahead on little work: 16 -> 32
    // at 32k voxels 24 us against 35, 32 -> 64 at 8k 24 against 41; 32 -> 64 at 32k 50 against 48, 64 -> 128
    // at 8k 54 against 47, 16 -> 32 at 110k 45 against 44 (its path for channel counts that are not a
    // multiple of 4 is behind everywhere: 50 -> 50 at 800 voxels 39 against 27).  Just above the line it is still
    // ahead at some shapes, 32 -> 64 at 20k 36 us against 45, with twice the error, 2.1e-7 against 1.0e-7
    if (c % 4 == 0 && N % 4 == 0 && (double)n * c * N < 40e6) return p;
    const int64_t m_tiles = ((int64_t)taps * c + hch::WG_UNITS * 16 - 1) / (hch::WG_UNITS * 16), n_tiles = N <= 32 ? 1 : (N + 63) / 64;
    // one workgroup per CU; as a multiple of 8 (whole slices per XCD) where there are that many
    int64_t s = std::max<int64_t>(1, WG_RESIDENT / (m_tiles * n_tiles));
    s = std::min({s, (n + hch::WG_VOX - 1) / hch::WG_VOX, max_slices});
    if (s >= 8) s = s / 8 * 8;
    p.ok = true; p.slices = (int)s; p.m_tiles = (int)m_tiles; p.n_tiles = (int)n_tiles;
    return p;
}

static hch_status launch_wgrad_split(const WgradSplitPlan &p, const float *X, const float *dY, float *out, float *part,
                                     const int32_t *nbr, const int32_t *order, int64_t n, int64_t x_rows, int c, int N, int taps,
                                     double bytes, hipStream_t s)
{
    const int64_t wsize = (int64_t)taps * c * N;
    {
        const bool c16 = c % 16 == 0;
        const int kid = N <= 32 ? (c16 ? HCH_KERNEL_ID("wgrad_split_kernel<2, true>") : HCH_KERNEL_ID("wgrad_split_kernel<2, false>"))
                                : (c16 ? HCH_KERNEL_ID("wgrad_split_kernel<4, true>") : HCH_KERNEL_ID("wgrad_split_kernel<4, false>"));
        hch::LaunchTimer lt(kid, s, bytes + 4.0 * wsize * p.slices, 2.0 * wsize * n);
        float *dst = p.slices == 1 ? out : part;
        const dim3 grid((unsigned)(p.slices * p.m_tiles * p.n_tiles));
#define HCH_WGRAD_CASE(NT_, C16_)                                                                                  \
        HCH_LAUNCH((hch::wgrad_split_kernel<NT_, C16_>), grid, dim3(512), 0, s, X, dY, dst, nbr, order, taps * c, N, \
                   (int)n, x_rows, c, taps, p.slices, p.m_tiles, p.n_tiles, wsize)
        if (N <= 32) { if (c16) HCH_WGRAD_CASE(2, true); else HCH_WGRAD_CASE(2, false); }
        else { if (c16) HCH_WGRAD_CASE(4, true); else HCH_WGRAD_CASE(4, false); }
#undef HCH_WGRAD_CASE
    }
    HCH_LAUNCH_CHECK("wgrad_split_kernel");
    return p.slices > 1 ? launch_reduce(part, out, wsize, p.slices, s) : HCH_OK;
}

// The weight gradient with bf16 operands in the same manner (wgrad_bf16_kernel): even channel counts.
static WgradSplitPlan plan_wgrad_bf16(int64_t n, int c, int N, int64_t max_slices)
{
    WgradSplitPlan p{false, 1, 1, 1};
    const int64_t lim = (int64_t)1 << 31, rows = hch::WGB_UNITS * 32;
    if (n * c * 2 >= lim || n * N * 2 >= lim || n * 108 >= lim || n >= (1 << 23) || c * 2 >= (1 << 23)) return p;
    if (c % 2 || N % 2 || N <= 16 || 27 * c < 32) return p;
    // gemm_bf16_kernel, where it applies (multiples of 8), is ahead on less work: 32 -> 64 at 110k voxels
    // 35 us against 38, 64 -> 64 at 32k 29 against 32; 64 -> 64 at 110k 54 against 51, 32 -> 64 at 280k 64
    // against 60, 64 -> 128 at 280k 213 against 162.  Other channel counts: 50 -> 50 at 280k 1090 against 103
    if (c % 8 == 0 && N % 8 == 0 && (double)n * c * N < 4e8) return p;
    const int64_t m_tiles = ((int64_t)27 * c + rows - 1) / rows, n_tiles = N <= 32 ? 1 : (N + 63) / 64;
    int64_t s = std::max<int64_t>(1, WG_RESIDENT / (m_tiles * n_tiles));
    s = std::min({s, (n + hch::WG_VOX - 1) / hch::WG_VOX, max_slices});
    if (s >= 8) s = s / 8 * 8;
    p.ok = true; p.slices = (int)s; p.m_tiles = (int)m_tiles; p.n_tiles = (int)n_tiles;
    return p;
}

static hch_status launch_wgrad_bf16(const WgradSplitPlan &p, const uint16_t *X, const uint16_t *dY, float *out, float *part,
                                    const int32_t *nbr, const int32_t *order, int64_t n, int c, int N, double bytes, hipStream_t s)
{
    const int64_t wsize = (int64_t)27 * c * N;
    {
        hch::LaunchTimer lt(N <= 32 ? HCH_KERNEL_ID("wgrad_bf16_kernel<2>") : HCH_KERNEL_ID("wgrad_bf16_kernel<4>"), s,
                            bytes + 4.0 * wsize * p.slices, 2.0 * wsize * n);
        float *dst = p.slices == 1 ? out : part;
        const dim3 grid((unsigned)(p.slices * p.m_tiles * p.n_tiles));
        if (N <= 32)
            HCH_LAUNCH(hch::wgrad_bf16_kernel<2>, grid, dim3(512), 0, s, X, dY, dst, nbr, order, 27 * c, N, (int)n, n, c, 27,
                       p.slices, p.m_tiles, p.n_tiles, wsize);
        else
            HCH_LAUNCH(hch::wgrad_bf16_kernel<4>, grid, dim3(512), 0, s, X, dY, dst, nbr, order, 27 * c, N, (int)n, n, c, 27,
                       p.slices, p.m_tiles, p.n_tiles, wsize);
    }
    HCH_LAUNCH_CHECK("wgrad_bf16_kernel");
    return p.slices > 1 ? launch_reduce(part, out, wsize, p.slices, s) : HCH_OK;
}

// Forward product and data gradient on split operands (conv_split_kernel); `max_splits` partial results fit
// the caller's workspace.
struct ConvSplitPlan { bool ok; int nt, wv, splits; unsigned m_tiles; };

static ConvSplitPlan plan_conv_split(int64_t n, int c, int N, int max_splits)
{
    ConvSplitPlan p{false, 4, 4, 1, 0};
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit byte offsets reach everything, a negative one nothing; 24-bit row and row-length factors
    if (n >= (1 << 23) || c * 4 >= (1 << 23) || n * c * 4 >= lim || n * 108 >= lim || (int64_t)108 * c * N >= lim) return p;
    p.nt = N <= 16 ? 1 : (N <= 32 ? 2 : 4);
    const int64_t n_tiles = (N + 16 * p.nt - 1) / (16 * p.nt);
    p.m_tiles = (unsigned)((n + 63) / 64);
    // 16 wavefronts per CU, 64 or 128 rows to a workgroup.  128 rows share the weights' splitting: 64 -> 64 at 280 000
    // voxels 198 -> 187 us, at 31 000 12 -> 64 24 -> 21; at 10 000 voxels 128 -> 256 123 -> 130 and 16 -> 32 14 -> 17.  A
    // tile of 16 columns has too few weights for 512 threads (32 -> 16 at 280 000: 53 -> 62).  Small levels
    // split the reduction to fill the chip
    if (p.nt > 1 && p.m_tiles >= 384) p.wv = 8;
    // (Rows of 4 channels, half of whose split terms are padding, and little work with more than 32 columns are
    // faster with gemm_f32_kernel, 4 -> 32 at 280k voxels 37 us against 46, 12 -> 64 at 10k 14 against 19, but
    // its results are 2.5 and 3 times as far from the exact ones, 1.2e-7 against 4.6e-8 and 2.0e-7 against 6.4e-8.)
    const int64_t blocks = p.m_tiles * n_tiles, steps = (int64_t)27 * ((c + 7) / 8) / 4;
    if (blocks < 512) p.splits = (int)std::max<int64_t>(1, std::min<int64_t>({1024 / blocks, steps / 6, max_splits}));
    p.ok = true;
    return p;
}

// transposed: W(t, k, n) = W[26 - t][n][k]
static hch_status launch_conv_split(const ConvSplitPlan &p, const Level &L, const float *X, const float *W, float *out, float *part,
                                    int64_t n, int c, int N, bool transposed, double bytes, hipStream_t s)
{
    float *dst = p.splits > 1 ? part : out;
    const unsigned n_tiles = (unsigned)((N + 16 * p.nt - 1) / (16 * p.nt));
    const bool fast = c % 32 == 0;
    static int ids[3][2][2][2];                        // [columns][wavefronts][fast][transposed]
    static const bool ids_ready = [] { memset(ids, 0xFF, sizeof ids); return true; }();
    (void)ids_ready;
    int &id = ids[p.nt / 2][p.wv / 8][fast][transposed];
    if (id < 0) {
        char nm[96];
        snprintf(nm, sizeof nm, "conv_split_kernel<%d, %d, %s, %s>", p.nt, p.wv, fast ? "true" : "false", transposed ? "true" : "false");
        id = hch::Profiler::get().id_for(nm);
    }
    {
        hch::LaunchTimer lt(id, s, bytes, 2.0 * 27 * c * (double)N * n);
        const unsigned group = (unsigned)p.wv / 4;     // 64-row tiles per workgroup
        const dim3 grid(hch::skip_grid((p.m_tiles + group - 1) / group, hch::skip_chunk(p.m_tiles, group)), n_tiles, (unsigned)p.splits);
        const int vec_out = N % 4 == 0 && aligned16(dst);
#define HCH_CONV_SPLIT(NT_, WV_, F_, T_)                                                                       \
        HCH_LAUNCH((hch::conv_split_kernel<NT_, WV_, F_, T_>), grid, dim3(64 * WV_), 0, s, X, W, dst, L.dnbr, L.rows(),  \
                   (const uint32_t *)L.row_taps(), (int)n, N, c, p.m_tiles, n * N, vec_out)
#define HCH_CONV_SPLIT_FT(NT_, WV_)                                                                            \
        do {                                                                                                   \
            if (fast) { if (transposed) HCH_CONV_SPLIT(NT_, WV_, true, true); else HCH_CONV_SPLIT(NT_, WV_, true, false); } \
            else { if (transposed) HCH_CONV_SPLIT(NT_, WV_, false, true); else HCH_CONV_SPLIT(NT_, WV_, false, false); } \
        } while (0)
        if (p.nt == 1) HCH_CONV_SPLIT_FT(1, 4);
        else if (p.nt == 2) { if (p.wv == 8) HCH_CONV_SPLIT_FT(2, 8); else HCH_CONV_SPLIT_FT(2, 4); }
        else { if (p.wv == 8) HCH_CONV_SPLIT_FT(4, 8); else HCH_CONV_SPLIT_FT(4, 4); }
#undef HCH_CONV_SPLIT_FT
#undef HCH_CONV_SPLIT
    }
    HCH_LAUNCH_CHECK("conv_split_kernel");
    return p.splits > 1 ? launch_reduce(part, out, n * N, p.splits, s) : HCH_OK;
}

// The forward product of the columns algorithm with the column matrix on the way (columns_split_kernel)
static hch_status launch_columns_split(const ConvSplitPlan &p, const Level &L, const float *X, const float *W, float *out, float *part, float *col,
                                       int64_t n, int c, int N, double bytes, hipStream_t s)
{
    float *dst = p.splits > 1 ? part : out;
    const unsigned n_tiles = (unsigned)((N + 16 * p.nt - 1) / (16 * p.nt));
    const bool fast = c % 32 == 0;
    const bool stream = c % 16 == 0 && n * 108 * c > (int64_t)(c == 16 ? 256 : 288) << 20;
    static int ids[3][2][2][2];                        // [columns][wavefronts][fast][stream]
    static const bool ids_ready = [] { memset(ids, 0xFF, sizeof ids); return true; }();
    (void)ids_ready;
    int &id = ids[p.nt / 2][p.wv / 8][fast][stream];
    if (id < 0) {
        char nm[96];
        snprintf(nm, sizeof nm, "columns_split_kernel<%d, %d, %s, %s>", p.nt, p.wv, fast ? "true" : "false", stream ? "true" : "false");
        id = hch::Profiler::get().id_for(nm);
    }
    {
        hch::LaunchTimer lt(id, s, bytes, 2.0 * 27 * c * (double)N * n);
        const unsigned group = (unsigned)p.wv / 4, groups = (p.m_tiles + group - 1) / group;
        const dim3 grid((groups + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD, n_tiles, (unsigned)p.splits);
        const int vec_out = N % 4 == 0 && aligned16(dst);
#define HCH_COLUMNS_SPLIT_F(NT_, WV_, FAST_)                                                                                                     \
        do {                                                                                                                                     \
            if (stream) HCH_LAUNCH((hch::columns_split_kernel<NT_, WV_, FAST_, true>), grid, dim3(64 * WV_), 0, s, X, W, dst, L.dnbr, col, (int)n, N, c, p.m_tiles, n * N, vec_out); \
            else HCH_LAUNCH((hch::columns_split_kernel<NT_, WV_, FAST_, false>), grid, dim3(64 * WV_), 0, s, X, W, dst, L.dnbr, col, (int)n, N, c, p.m_tiles, n * N, vec_out); \
        } while (0)
#define HCH_COLUMNS_SPLIT(NT_, WV_) do { if (fast) HCH_COLUMNS_SPLIT_F(NT_, WV_, true); else HCH_COLUMNS_SPLIT_F(NT_, WV_, false); } while (0)
        if (p.nt == 1) HCH_COLUMNS_SPLIT(1, 4);
        else if (p.nt == 2) { if (p.wv == 8) HCH_COLUMNS_SPLIT(2, 8); else HCH_COLUMNS_SPLIT(2, 4); }
        else { if (p.wv == 8) HCH_COLUMNS_SPLIT(4, 8); else HCH_COLUMNS_SPLIT(4, 4); }
#undef HCH_COLUMNS_SPLIT
#undef HCH_COLUMNS_SPLIT_F
    }
    HCH_LAUNCH_CHECK("columns_split_kernel");
    return p.splits > 1 ? launch_reduce(part, out, n * N, p.splits, s) : HCH_OK;
}

// The gradient of the column matrix on split operands (dcol_split_kernel): rows of 32, 64 or 128 gradients, which the wavefronts keep in
// registers and whose weights share out evenly over 512 threads (not 96 or 160), 32-bit byte offsets.  256 take twice the registers, two workgroups to
// a CU: 64 -> 256 at 800 voxels 19 us on the fp32 instruction and 29, at 5400 57 and 64.5, at 23 000 195 and 164, and levels with so many channels
// have few voxels.  Few rows of 128 are cut for too few columns each: with the gather that follows, 128 -> 128 at 800
// voxels 17 us on the fp32 instruction, 20 here, 64 -> 128 at 2700 23 and 25, at 5400 37 and 32, 128 -> 128 65 and 47.5
static bool dcol_split_ok(int64_t n, int c_in, int c_out)
{
    const int64_t lim = (int64_t)1 << 31;
    if (c_out == 128 && n < 4096) return false;
    return (c_out == 32 || c_out == 64 || c_out == 128) && c_in % 4 == 0 && (n + 128) * c_out * 4 < lim && (int64_t)(27 * c_in + 256) * c_out * 4 < lim;
}

static hch_status launch_dcol_split(const float *dY, const float *W, float *dcol, int64_t n, int c_in, int c_out, double bytes, hipStream_t s)
{
    const int N = 27 * c_in, bn = 4096 / c_out, chunks = (N + bn - 1) / bn;
    const unsigned tiles = (unsigned)((n + 127) / 128);
    // four workgroups per CU
    const int per = (int)std::max<int64_t>(1, std::min<int64_t>(chunks, (int64_t)chunks * tiles / 1024));
    const dim3 grid((tiles + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD, (unsigned)((chunks + per - 1) / per));
    const int kid = c_out == 32 ? HCH_KERNEL_ID("dcol_split_kernel<1>") : (c_out == 64 ? HCH_KERNEL_ID("dcol_split_kernel<2>") : HCH_KERNEL_ID("dcol_split_kernel<4>"));
    {
        hch::LaunchTimer lt(kid, s, bytes, 2.0 * N * (double)c_out * n);
        if (c_out == 32) HCH_LAUNCH(hch::dcol_split_kernel<1>, grid, dim3(512), 0, s, dY, W, dcol, (int)n, N, tiles, per);
        else if (c_out == 64) HCH_LAUNCH(hch::dcol_split_kernel<2>, grid, dim3(512), 0, s, dY, W, dcol, (int)n, N, tiles, per);
        else HCH_LAUNCH(hch::dcol_split_kernel<4>, grid, dim3(512), 0, s, dY, W, dcol, (int)n, N, tiles, per);
    }
    HCH_LAUNCH_CHECK("dcol_split_kernel");
    return HCH_OK;
}

// The same products for few voxels (conv_small_kernel).  It reads all weights of its taps once per 16 rows, so the line lies at little work, and for
// the data gradient, whose weights it reads in pieces of 16 bytes, or one by one where rows are no multiple of 8 channels, lower.  Calls one after
// the other (10 us: what the host takes for one) against conv_split_kernel with the launch that adds its parts: forward 16 -> 32 at 12 000 voxels 9.8
// us and 11.1, 32 -> 64 at 3200 10 and 16, at 6000 12.5 and 16.6, 64 -> 64 at 1500 10.5 and 16, 64 -> 128 at 800 10.5 and 16; data gradient 32 -> 16
// at 12 000 10 and 12.5, 64 -> 32 at 2200 11 and 15.  (Tiles of 64 columns 10.2 and 16 with 32 -> 64 and 64 -> 64 at 3200, 16 wavefronts 11.5 and
// 18.) The lines keep every call that was behind (of 25 by 16 pairs of channels at 23 level sets from 60 to 40 000 voxels, both directions) with
// conv_split_kernel, which splits long reductions over workgroups: 256 -> 32 at 800 voxels 14 us, 31 here, 128 -> 32 14.5 and 17.5, 96 -> 20 13.4 and
// 14.9; 16 -> 32 at 24 000 14 and 16, 12 -> 5 at 30 000 11.3 and 14.1, 32 -> 5 at 18 000 14.3 and 15.9, 80 -> 40 at 2200 17 and 20, 60 -> 40 15 and
// 16.5; data gradient of 100 channels to 32 at 800 13.5 and 26, of 60 to 32 13 and 17.5, of 128 to 32 14 and 20, of 12 to 32 at 10 000 12 and 13.7.
static bool conv_small_faster(int64_t n, int c, int N, bool transposed)
{
    if (n * c * 4 >= ((int64_t)1 << 31) || n * 108 >= ((int64_t)1 << 31)) return false;        // 32-bit byte offsets
    const double work = (double)n * ((c + 15) / 16 * 16) * ((N + 15) / 16 * 16);               // as tiles and loads are padded
    if ((int64_t)c * N > (transposed ? 4096 : 8192)) return false;
    if (transposed) return c <= (N <= 16 ? 112 : c % 8 ? 40 : 88) && work <= (c % 8 && (c <= 32 || c > 40) ? 4.2e6 : 6.5e6);
    if (c > (N > 16 && N <= 32 ? 88 : 112)) return false;
    if (c <= 16 || c > 64) return work <= 6.2e6;
    return work <= (c % 16 ? (c <= 56 ? 8e6 : 6.2e6) : (N <= 16 ? 8e6 : 12.5e6));
}

static hch_status launch_conv_small(const Level &L, const float *X, const float *W, float *out, int64_t n, int c, int N, bool transposed,
                                    double bytes, hipStream_t s)
{
    const int nt = N <= 16 ? 1 : 2;
    const int id = nt == 1 ? (transposed ? HCH_KERNEL_ID("conv_small_kernel<1, true>") : HCH_KERNEL_ID("conv_small_kernel<1, false>"))
                           : (transposed ? HCH_KERNEL_ID("conv_small_kernel<2, true>") : HCH_KERNEL_ID("conv_small_kernel<2, false>"));
    hch::LaunchTimer lt(id, s, bytes, 2.0 * 27 * c * (double)N * n);
    const dim3 grid((unsigned)((n + 15) / 16), (unsigned)((N + 16 * nt - 1) / (16 * nt)));
    const int vec_out = N % 4 == 0 && aligned16(out);
#define HCH_CONV_SMALL(NT_, T_) HCH_LAUNCH((hch::conv_small_kernel<NT_, T_>), grid, dim3(64 * hch::SMALL_WAVES), 0, s, X, W, out, (const int32_t *)L.dnbr, (int)n, N, c, vec_out)
    if (nt == 1) { if (transposed) HCH_CONV_SMALL(1, true); else HCH_CONV_SMALL(1, false); }
    else { if (transposed) HCH_CONV_SMALL(2, true); else HCH_CONV_SMALL(2, false); }
#undef HCH_CONV_SMALL
    HCH_LAUNCH_CHECK("conv_small_kernel");
    return HCH_OK;
}

// Forward product and data gradient (transposed) with bf16 operands over the row order (conv_bf16_kernel).  Its lines are by direction: of 170 pairs of
// channels at 9 to 24 sizes each, 800 to 609 000 rows, what takes longer with it than without stays with the kernel named.
static bool conv_bf16_ok(const Level &L, const void *X, const void *W, int64_t n, int c, int N, bool transposed)
{
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit byte offsets reach everything, a negative one nothing; 24-bit row and row-length factors; pairs of columns
    if (!L.rows() || n >= (1 << 23) || c * 2 >= (1 << 23) || n * c * 2 >= lim || n * 108 >= lim || (int64_t)54 * c * N >= lim) return false;
    if (c % 2 || N % 2 || ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 3u)) return false;
    const bool full = c % 32 == 0 && aligned16(X) && aligned16(W);
    const double neighbours = (double)L.nbr_valid / (double)n;
    if (c % 8 || N % 8 || !aligned16(X) || !aligned16(W)) {
        // Without gemm_bf16_kernel the products go to the fp32 instruction: 50 -> 50 at 800 rows 62 us and 27, at 16 500 101 and 29, at 127 000 606
        // and 51; rows of 2 channels are mostly padding here: 2 -> 16 at 800 rows 13 and 16, at 80 000 17.5 and 19, at 98 400 27 and 20.5, 2 -> 64 at
        // 64 000 25 and 25
        if (c % 4 || N % 4 || !aligned16(X) || !aligned16(W)) return c > 2 || n >= (N > 32 ? 65536 : 98304);
        // Where that has its vector path it is ahead on few rows, the longer with little to multiply: 12 -> 20 at 44 000 0.89 of its time, 20 -> 4 0.94,
        // 12 -> 16 1.22, at 80 000 0.98, 8 -> 20 1.23 and 1.00, 8 -> 12 1.62, 1.38, at 160 000 1.22; rows of 4 channels, 4 -> 16 at 280 000 30 us and 37
        if (!full) return c >= 20 || (c >= 12 && N > 16) ? n >= 40960 : c >= 8 && (c > 8 || N > 16) && n >= 81920;
        // It splits the reduction of few rows, here 27 * c terms follow one another: 64 -> 12 at 7000 rows 1.06 of its time, at 12 000 0.92, 96 -> 12
        // 1.72 and 1.23, at 16 500 1.01, 64 -> 20 at 3200 1.12, at 7000 0.78, 96 -> 36 1.36 and 0.86, 128 -> 20 1.43 and 0.99.  With transposed
        // weights it has its better loop for rows of a multiple of 64: to 12 channels 1.16 to 1.29 up to 64 000, 0.90 to 1.06 beyond, with 17
        // neighbours a voxel 1.18; to 20 1.11, 0.84 to 0.98, 1.10; to 36 and 60 1.28, 0.99, 0.95
        if (c == 32) return true;
        if (transposed && c % 64 == 0) return n >= 98304 && (N > 32 || (N > 16 && neighbours <= 11));
        return n >= (N < 20 ? 192 : 96) * (int64_t)c;
    }
    // 16 columns: 32 -> 16 at 800 to 44 000 rows 0.89 to 0.99 of gemm_bf16_kernel's time, at 64 000 1.11 (32 -> 8 1.03 and 1.14), at 80 000 0.94, at
    // 280 000 0.75; data gradient 0.71 to 0.90 at all sizes.  Longer rows to 16 columns, half of a tile, 64 -> 16, 96 -> 16, 128 -> 16: at 64 000
    // 1.21, 1.08, 1.23, at 127 000 1.03, 0.80, 1.05, with 17 neighbours a voxel 1.15, 1.13, 1.39; at 280 000 0.86, 0.69, 0.84
    if (N <= 16) return full && c == 32 && (transposed || n >= 81920);
    // Against gemm_bf16_kernel, which splits the reduction of few rows: 32 -> 64 at 16 500 to 32 000 rows 0.76 to 0.87, data gradient 0.64 to 0.74,
    // 64 -> 64 0.88 to 0.97 and 0.89 to 1.02, 32 -> 24 and 64 -> 24 at 16 500 1.02 to 1.10, at 24 000 0.85 and 0.94; longer rows: 96 -> 32 at 32 000
    // 26 us and 30, from 66 000 on 0.61 to 0.84, 128 -> 128 0.86 to 1.00.  Rows that fill a step in part: from 98 000 on 0.71 to 0.95 with 24, 56, 80
    // channels, 0.90 to 1.03 with 72; with 40, 3 of 8 padding, 0.96 to 1.15 at 98 000 and 127 000, 0.89 to 0.99 at 160 000; with 17 neighbours a
    // voxel 48 -> 64 1.09 to 1.15, 24 -> 128 1.04 to 1.08
    if (!full) {
        if (c < 24 || neighbours > 11 || n < (c * 4 >= (c + 31) / 32 * 96 ? 98304 : 160000)) return false;
    } else if (n < (c > 64 ? 65536 : N <= 32 && !transposed ? 20480 : 16384)) return false;
    // Where that kernel's tiles just fill a round of workgroups without splitting: to 32 columns, 52 000 to 64 000 rows, 32 -> 32 1.04 to 1.08, 64 ->
    // 32 0.99 to 1.08 and the same back (48 000 0.72 to 0.78, 72 000 0.90); to 64, 33 000 to 48 000, 32 -> 64 1.03 to 1.09, 64 -> 64 1.06 to 1.13,
    // back 1.02 to 1.11 (32 000 0.88, 52 000 0.95); to 128, 16 500 to 32 000, 32 -> 128 1.03 to 1.19, 64 -> 128 1.08 to 1.26, back 1.13 to 1.31 (36
    // 000 0.95 to 1.01).  Data gradients of 32 channels have no such stretch
    if (full && c <= 64 && (!transposed || c == 64)) {
        const int64_t tiles = N <= 32 ? (n + 127) / 128 : (n + 63) / 64 * ((N + 63) / 64);
        if (N <= 32 ? tiles > 384 && tiles <= 540 : tiles > 512 && tiles <= (N <= 64 ? 768 : 1024)) return false;
    }
    // It lives on the taps that a tile's rows leave out: of 27, 256 rows of thin shells (9 neighbours a voxel) have 10 to 16, of
    // thick ones (17) 18 to 20.  Times over those of gemm_bf16_kernel, index lists also tap-major (which that kernel is faster with) or
    // not, at 0.25 to 1.3 million rows: 9 to 10.6 neighbours 0.53 to 0.96 and 0.51 to 0.91 (64 -> 32 at 10.6 1.02); spheres' shells, 14
    // neighbours, 64 -> 64 0.96 to 1.06 and 0.93 to 0.98, 64 -> 32 1.07 to 1.19 and 0.92 to 1.04; 17 to 18, 64 -> 64 0.92 to 1.15 and 0.90
    // to 1.07, 128 -> 128 1.02 to 1.23 and 0.84 to 1.10, 64 -> 32 0.95 to 1.37 and 0.85 to 1.16; 21, 64 -> 64 1.10 to 1.15.  Rows that are no
    // multiple of 64 channels, for which gemm_bf16_kernel has the slower loop, to 64 columns and more: 17 to 18, 32 -> 64 0.88
    // to 1.05, 96 -> 96 0.79 to 1.02; 19 to 21, 32 -> 64 1.00 to 1.08, 26 1.13.
    if (neighbours > (N < 64 ? 11 : (c % 64 ? 18 : (L.dnbr_t ? 11 : 15)))) return false;
    // Up to the last-level cache: the order scatters the rows that a tile reads over the whole of X.  (Thin shells would gain
    // beyond it too, 1.5 million rows, 128 -> 128, 366 MB: 1469 us there, 925 here; thick ones of 64 channels 869 and 884.)
    return n * c * 2 <= (int64_t)256 << 20;
}

// transposed: W(t, k, n) = W[26 - t][n][k]
static hch_status launch_conv_bf16(const Level &L, const uint16_t *X, const uint16_t *W, float *out, int64_t n, int c, int N, bool transposed,
                                   double bytes, hipStream_t s)
{
    const unsigned m_tiles = (unsigned)((n + 63) / 64);
    // Where plan_rows splits the reduction of a level that does not fill the chip, a single chain of all terms is further from the exact sums than
    // its slices are: there tiles of 32 columns, which add up sums of 128 terms.  Errors of slices, chain, such sums: 50 -> 50 at 3200 rows 1.03e-7,
    // 1.61e-7, 0.80e-7, at 20 000 1.01e-7, 1.23e-7, 0.71e-7, 34 -> 66 at 12 000 (data gradient) 1.01e-7, 1.47e-7, 0.78e-7.  Times of tiles of 64 and
    // 32 columns there: 50 -> 50 at 800 rows 31 us and 27, at 16 500 31 and 29, 64 -> 64 23 and 20.
    const bool few = (int64_t)m_tiles * ((N + 63) / 64) < 512 && 27 * c >= 512;
    const int nt = N <= 32 || few ? 2 : 4, ks = c % 64 == 0 ? 64 : 32;
    const bool full = c % 32 == 0 && aligned16(X) && aligned16(W);
    const int wv = full && nt == 4 && ks == 64 && n >= 98304 ? 8 : 4;           // see conv_bf16_rows
    static int ids[2][3][2][2];                        // [columns][channels a step: part of 32, 32, 64][wavefronts][transposed]
    static const bool ids_ready = [] { memset(ids, 0xFF, sizeof ids); return true; }();
    (void)ids_ready;
    int &id = ids[nt / 4][full ? ks / 32 : 0][wv / 8][transposed];
    if (id < 0) {
        char nm[96];
        if (full) snprintf(nm, sizeof nm, "conv_bf16_kernel<%d, %d, %d, %s>", nt, ks, wv, transposed ? "true" : "false");
        else snprintf(nm, sizeof nm, "conv_ragged_bf16_kernel<%d, %s>", nt, transposed ? "true" : "false");
        id = hch::Profiler::get().id_for(nm);
    }
    {
        hch::LaunchTimer lt(id, s, bytes, 2.0 * 27 * c * (double)N * n);
        const unsigned group = wv / 2;
        const dim3 grid(hch::skip_grid((m_tiles + group - 1) / group, hch::skip_chunk(m_tiles, group)), (unsigned)((N + 16 * nt - 1) / (16 * nt)));
        const int vec_out = N % 4 == 0 && aligned16(out);
#define HCH_CONV_BF16(KERNEL_)                                                                                                    \
        HCH_LAUNCH(KERNEL_, grid, dim3(64 * wv), 0, s, X, W, out, (const int32_t *)L.dnbr, L.rows(), (const uint32_t *)L.row_taps(), (int)n, N, c, \
                   m_tiles, vec_out)
#define HCH_CONV_BF16_T(NT_, KS_, WV_) do { if (transposed) HCH_CONV_BF16((hch::conv_bf16_kernel<NT_, KS_, WV_, true>)); else HCH_CONV_BF16((hch::conv_bf16_kernel<NT_, KS_, WV_, false>)); } while (0)
#define HCH_CONV_RAGGED_T(NT_) do { if (transposed) HCH_CONV_BF16((hch::conv_ragged_bf16_kernel<NT_, true>)); else HCH_CONV_BF16((hch::conv_ragged_bf16_kernel<NT_, false>)); } while (0)
        if (!full) { if (nt == 2) HCH_CONV_RAGGED_T(2); else HCH_CONV_RAGGED_T(4); }
        else if (ks == 32) { if (nt == 2) HCH_CONV_BF16_T(2, 32, 4); else HCH_CONV_BF16_T(4, 32, 4); }
        else if (nt == 2) HCH_CONV_BF16_T(2, 64, 4);
        else if (wv == 8) HCH_CONV_BF16_T(4, 64, 8);
        else HCH_CONV_BF16_T(4, 64, 4);
#undef HCH_CONV_RAGGED_T
#undef HCH_CONV_BF16_T
#undef HCH_CONV_BF16
    }
    HCH_LAUNCH_CHECK("conv_bf16_kernel");
    return HCH_OK;
}

// workspace layout, all offsets 256-byte aligned:
//   columns algorithm : [ column matrix | split-K partial sums ]
//   fused algorithm   : [ flipped+transposed weights (bwd_data only) | split-K partial sums ]
struct WsLayout { size_t first_bytes, part_bytes; };

// bf16 forward product: with rows of a multiple of 64 channels the kernel takes the weights from a
// copy transposed per tap, Wt[27][c_out][c_in] at the start of the workspace, in which the
// reduction index is the fast one -- its tiles then go to LDS as they are, instead of being
// transposed in registers on every tile (vector instructions that cost matrix time)
static bool fwd_transposed_weights(hch_dtype dtype, int c_in, int c_out)
{
    return dtype == HCH_BF16 && c_in % hch::BF16_BK == 0 && c_out % 8 == 0;
}

// least: what a call needs; else what it can make use of (the query's answer)
static WsLayout ws_layout(const Level &L, int c_in, int c_out, hch_dtype dtype, hch_ws_kind kind, hch_algo algo, bool least = false)
{
    const size_t Kc = (size_t)27 * c_in, n = (size_t)L.n_total;
    WsLayout w{0, 0};
    if (kind == HCH_WS_FWD) {
        const GemmPlan p = plan_rows(L.n_total, c_out, (int)Kc, true, k_gran(dtype));
        if (algo == HCH_ALGO_COLUMNS) w.first_bytes = round_up(n * Kc * elem_size(dtype), 256);
        int splits = p.splits;
        if (algo == HCH_ALGO_FUSED) { const DirectPlan d = plan_direct(L.n_total, c_in, c_out); if (d.ok) splits = std::max(splits, d.splits); }
        if (algo == HCH_ALGO_FUSED && fwd_transposed_weights(dtype, c_in, c_out)) w.first_bytes = round_up(Kc * c_out * elem_size(dtype), 256);
        if (splits > 1) w.part_bytes = round_up((size_t)splits * n * c_out * 4, 256);
    } else if (kind == HCH_WS_BWD_DATA) {
        if (algo == HCH_ALGO_COLUMNS) w.first_bytes = round_up(n * Kc * 4, 256);
        else {
            const GemmPlan p = plan_rows(L.n_total, c_in, 27 * c_out, true, k_gran(dtype));
            w.first_bytes = round_up(Kc * c_out * elem_size(dtype), 256);
            const DirectPlan d = plan_direct(L.n_total, c_out, c_in);
            const int splits = d.ok ? std::max(p.splits, d.splits) : p.splits;
            if (splits > 1) w.part_bytes = round_up((size_t)splits * n * c_in * 4, 256);
        }
    } else if (kind == HCH_WS_BWD_WEIGHT) {
        const GemmPlan p = plan_wgrad(L.n_total, c_in, c_out, 27, k_gran(dtype));
        if (algo == HCH_ALGO_COLUMNS) w.first_bytes = round_up(n * Kc * elem_size(dtype), 256);
        int splits = p.splits;
        if (algo == HCH_ALGO_FUSED && dtype == HCH_F32 && !least) {
            const WgradSplitPlan q = plan_wgrad_split(L.n_total, L.n_total, c_in, c_out, 27, INT32_MAX);
            if (q.ok) splits = std::max(splits, q.slices);
        }
        if (algo == HCH_ALGO_FUSED && dtype == HCH_BF16 && !least) {
            const WgradSplitPlan q = plan_wgrad_bf16(L.n_total, c_in, c_out, INT32_MAX);
            if (q.ok) splits = std::max(splits, q.slices);
        }
        if (splits > 1) w.part_bytes = round_up((size_t)splits * Kc * c_out * 4, 256);
    }
    return w;
}

extern "C" size_t hch_conv_workspace_bytes(const hch_levels *levels, int32_t level, int32_t c_in,
                                           int32_t c_out, hch_dtype dtype, hch_ws_kind kind, hch_algo algo)
{
    if (!levels || level < 0 || level >= (int32_t)levels->lv.size() || c_in <= 0 || c_out <= 0) return 0;
    if (algo == HCH_ALGO_COLUMNS_RESIDENT) algo = HCH_ALGO_COLUMNS;
    if (algo == HCH_ALGO_FUSED_DENSE) algo = HCH_ALGO_FUSED;     // same workspace as the fused algorithm
    if (algo != HCH_ALGO_COLUMNS && algo != HCH_ALGO_FUSED) return 0;
    const Level &L = levels->lv[level];
    if (kind == HCH_WS_MIN) {
        // hch_conv_fwd with the columns algorithm: room for 1024 rows of the column matrix
        // next to the split-K area
        const WsLayout w = ws_layout(L, c_in, c_out, dtype, HCH_WS_FWD, algo);
        const size_t rows = std::min<size_t>((size_t)L.n_total, 1024);
        const size_t first = algo == HCH_ALGO_COLUMNS ? round_up(rows * 27 * c_in * elem_size(dtype), 256) : w.first_bytes;
        return std::max<size_t>(256, first + w.part_bytes);
    }
    if (kind != HCH_WS_FWD && kind != HCH_WS_BWD_DATA && kind != HCH_WS_BWD_WEIGHT) return 0;
    const WsLayout w = ws_layout(L, c_in, c_out, dtype, kind, algo);
    return std::max<size_t>(256, w.first_bytes + w.part_bytes);
}

// ---------------------------------------------------------------------------------------
// convolution
// ---------------------------------------------------------------------------------------

static hch_status conv_args(const hch_levels *levels, int32_t level, hch_dtype dtype, const void *a,
                            const void *b, const void *c, int32_t c_in, int32_t c_out,
                            const void *ws, hch_algo algo, const Level **L, const char *who)
{
    hch_status st = get_level(levels, level, L, who);
    if (st != HCH_OK) return st;
    if (!a || !b || !c || !ws || c_in <= 0 || c_out <= 0)
        return fail(HCH_EINVAL, std::string(who) + ": null pointer or non-positive channel count");
    if ((int64_t)27 * c_in * c_out >= ((int64_t)1 << 31))
        return fail(HCH_EINVAL, std::string(who) + ": weight tensor too large");
    if (algo != HCH_ALGO_COLUMNS && algo != HCH_ALGO_FUSED)
        return fail(HCH_EINVAL, std::string(who) + ": unknown algorithm");
    if (dtype != HCH_F32 && dtype != HCH_BF16)
        return fail(HCH_EINVAL, std::string(who) + ": unknown dtype");
    if (reinterpret_cast<uintptr_t>(ws) & 255u)
        return fail(HCH_EINVAL, std::string(who) + ": workspace must be 256-byte aligned");
    if ((*L)->n_total >= ((int64_t)1 << 31) / 64)
        return fail(HCH_EUNSUPPORTED, std::string(who) + ": too many voxels");
    // the kernels index feature rows with 32 bits: voxel * channels + channel
    if ((*L)->n_total * (int64_t)std::max(c_in, c_out) >= ((int64_t)1 << 31))
        return fail(HCH_EUNSUPPORTED, std::string(who) + ": a feature matrix of more than 2^31 elements");
    return HCH_OK;
}

extern "C" hch_status hch_conv_fwd(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                   const void *X, const void *W, float *Y, int32_t c_in,
                                   int32_t c_out, void *workspace, size_t ws_bytes, hch_algo algo,
                                   void *stream)
{
    const Level *L;
    const bool skip = algo == HCH_ALGO_FUSED;                    // absent taps may be skipped
    if (algo == HCH_ALGO_FUSED_DENSE) algo = HCH_ALGO_FUSED;
    hch_status st = conv_args(levels, level, dtype, X, W, Y, c_in, c_out, workspace, algo, &L, "hch_conv_fwd");
    if (st != HCH_OK) return st;
    if (ws_bytes < hch_conv_workspace_bytes(levels, level, c_in, c_out, dtype, HCH_WS_MIN, algo))
        return fail(HCH_EWORKSPACE, "hch_conv_fwd: workspace too small");
    hipStream_t s = (hipStream_t)stream;
    const int Kc = 27 * c_in;
    const int64_t n = L->n_total;
    const WsLayout w = ws_layout(*L, c_in, c_out, dtype, HCH_WS_FWD, algo);
    const GemmPlan p = plan_rows(n, c_out, Kc, true, k_gran(dtype));
    const double es = elem_size(dtype);               // bytes per input element
    float *part = (float *)((char *)workspace + ((ws_bytes - w.part_bytes) & ~(size_t)255));   // split-K area at the end

    if (algo == HCH_ALGO_FUSED) {
        // Y = gathered columns . W, the column matrix never leaves the chip.  Per voxel: 27
        // indices and its feature row in, one output row out; the weights once.
        if (narrow4_ok(n, c_in, c_out) && dtype == HCH_F32 && aligned16(X) && aligned16(W) && aligned16(Y)) {
            const double bytes = (double)n * (108.0 + 4.0 * c_in + 4.0 * c_out) + 4.0 * Kc * c_out;
            return launch_narrow4((const float *)X, L->dnbr, (const float *)W, Y, n, c_in, bytes, s, 0,
                                  skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr);
        }
        const DirectPlan d = plan_direct(n, c_in, c_out);
        if (d.ok && dtype == HCH_F32 && aligned16(X) && aligned16(W) && aligned16(Y)) {
            const double bytes = (double)n * (108.0 + 4.0 * c_in + 4.0 * c_out * d.splits) + 4.0 * Kc * c_out;
            st = launch_direct(d, (const float *)X, L->dnbr, (const float *)W, d.splits > 1 ? part : Y, n, c_in, c_out, bytes, s, 0,
                               skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr);
            if (st != HCH_OK) return st;
            if (d.splits > 1) st = launch_reduce(part, Y, n * c_out, d.splits, s);
            return st;
        }
        if (skip && dtype == HCH_F32 && conv_small_faster(n, c_in, c_out, false))
            return launch_conv_small(*L, (const float *)X, (const float *)W, Y, n, c_in, c_out, false,
                                     (double)n * (108.0 + 4.0 * c_in + 4.0 * c_out) + 4.0 * Kc * c_out, s);
        if (skip && dtype == HCH_F32 && L->rows()) {
            const ConvSplitPlan q = plan_conv_split(n, c_in, c_out, p.splits);
            if (q.ok)
                return launch_conv_split(q, *L, (const float *)X, (const float *)W, Y, part, n, c_in, c_out, false,
                                         (double)n * (108.0 + 4.0 * c_in + 4.0 * c_out * q.splits) + 4.0 * Kc * c_out, s);
        }
        const double bytes = (double)n * (108.0 + es * c_in + 4.0 * c_out * p.splits) + es * Kc * c_out;
        if (skip && dtype == HCH_BF16 && conv_bf16_ok(*L, X, W, n, c_in, c_out, false))
            return launch_conv_bf16(*L, (const uint16_t *)X, (const uint16_t *)W, Y, n, c_in, c_out, false,
                                    (double)n * (108.0 + es * c_in + 4.0 * c_out) + es * Kc * c_out, s);
        if (fwd_transposed_weights(dtype, c_in, c_out) && aligned16(X) && aligned16(W) && aligned16(workspace)) {
            const int64_t wn = (int64_t)Kc * c_out, per_tap = (int64_t)c_in * c_out;
            {
                hch::LaunchTimer lt(HCH_KERNEL_ID("flip_transpose_weights_kernel<unsigned short>"), s, 4.0 * wn, 0.0);
                HCH_LAUNCH(hch::flip_transpose_weights_kernel<uint16_t>, dim3(blocks_for(wn)), dim3(256), 0, s,
                           (const uint16_t *)W, (uint16_t *)workspace, c_in, c_out, 27, 0);
            }
            HCH_LAUNCH_CHECK("flip_transpose_weights_kernel");
            st = launch_gemm<hch::A_GATHER, true>(dtype, p, X, workspace, p.splits > 1 ? part : Y, L->dnbr, (int)n, c_out, Kc,
                                                  c_in, c_in, c_out, n * c_out, bytes, s, 0, 27, c_in, per_tap, L->dnbr_t,
                                                  nullptr, nullptr, n);
            if (st != HCH_OK) return st;
            if (p.splits > 1) st = launch_reduce(part, Y, n * c_out, p.splits, s);
            return st;
        }
        st = launch_gemm<hch::A_GATHER, false>(dtype, p, X, W,
                                               p.splits > 1 ? part : Y, L->dnbr, (int)n, c_out, Kc, c_in,
                                               c_out, c_out, n * c_out, bytes, s, 0, 27, 0, 0, L->dnbr_t,
                                               skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr, n);
        if (st != HCH_OK) return st;
        if (p.splits > 1) st = launch_reduce(part, Y, n * c_out, p.splits, s);
        return st;
    }

    // as many rows of the column matrix as the workspace holds, in multiples of the GEMM tile
    int64_t chunk = (int64_t)(((ws_bytes - w.part_bytes) & ~(size_t)255) / ((size_t)Kc * elem_size(dtype)));
    // room for all of the column matrix: written on the way (faster at all 90 shapes that were tried, 800 to 282 000 voxels, 1.06 to 2.2 times)
    if (chunk >= n && dtype == HCH_F32 && c_in % 4 == 0 && (int64_t)(27 * c_in + 128) * c_out * 4 < (int64_t)1 << 31) {
        const ConvSplitPlan q = plan_conv_split(n, c_in, c_out, p.splits);
        if (q.ok)
            return launch_columns_split(q, *L, (const float *)X, (const float *)W, Y, part, (float *)workspace, n, c_in, c_out,
                                        (double)n * (108.0 + 112.0 * c_in + 4.0 * c_out * q.splits) + 4.0 * Kc * c_out, s);
    }
    if (chunk < n) chunk = std::max<int64_t>(128, chunk / 128 * 128);
    for (int64_t r0 = 0; r0 < n; r0 += chunk) {
        const int64_t rows = std::min<int64_t>(chunk, n - r0);
        st = do_hash2col(*L, dtype, X, c_in, r0, rows, workspace, s);
        if (st != HCH_OK) return st;
        const double bytes = es * ((double)rows * Kc + (double)Kc * c_out) + 4.0 * (double)rows * c_out * p.splits;
        // the split plan was made for all n rows; slices of a chunk land in the same places
        st = launch_gemm<hch::A_ROWS, false>(dtype, p, workspace, W,
                                             p.splits > 1 ? part + r0 * c_out : Y + r0 * c_out, nullptr,
                                             (int)rows, c_out, Kc, Kc, c_out, c_out, n * c_out, bytes, s);
        if (st != HCH_OK) return st;
    }
    if (p.splits > 1) st = launch_reduce(part, Y, n * c_out, p.splits, s);
    return st;
}

extern "C" hch_status hch_conv_bwd_data(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                        const void *dY, const void *W, float *dX, int32_t c_in,
                                        int32_t c_out, void *workspace, size_t ws_bytes, hch_algo algo,
                                        void *stream)
{
    const Level *L;
    const bool skip = algo == HCH_ALGO_FUSED;
    if (algo == HCH_ALGO_FUSED_DENSE) algo = HCH_ALGO_FUSED;
    hch_status st = conv_args(levels, level, dtype, dY, W, dX, c_in, c_out, workspace, algo, &L, "hch_conv_bwd_data");
    if (st != HCH_OK) return st;
    if (ws_bytes < hch_conv_workspace_bytes(levels, level, c_in, c_out, dtype, HCH_WS_BWD_DATA, algo))
        return fail(HCH_EWORKSPACE, "hch_conv_bwd_data: workspace too small");
    hipStream_t s = (hipStream_t)stream;
    const int Kc = 27 * c_in;
    const int64_t n = L->n_total;
    const double es = elem_size(dtype);

    if (algo == HCH_ALGO_FUSED) {
        // dX[q] = sum_k dY[neighbour 26-k of q] . W[k]^T: a gathered product over the output
        // gradients with the flipped, transposed weights; dcol is never formed.
        const WsLayout w = ws_layout(*L, c_in, c_out, dtype, HCH_WS_BWD_DATA, algo);
        void *Wt = workspace;
        float *part = (float *)((char *)workspace + w.first_bytes);
        const int64_t wn = (int64_t)Kc * c_out;
        const int Kd = 27 * c_out;
        // narrow outputs: kernels that read the weights in place (flipped and transposed on the fly)
        if (narrow4_ok(n, c_out, c_in) && dtype == HCH_F32 && aligned16(dY) && aligned16(dX) && aligned16(W)) {
            const double bytes = (double)n * (108.0 + 4.0 * c_out + 4.0 * c_in) + 4.0 * wn;
            return launch_narrow4((const float *)dY, L->dnbr, (const float *)W, dX, n, c_out, bytes, s, 1,
                                  skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr);
        }
        const DirectPlan d = plan_direct(n, c_out, c_in);
        // (gradients whose rows hold a multiple of 32 channels are faster on split operands below: 32 -> 16
        // channels on 280k voxels 67 us against 93, on 12k 18 against 20)
        if (d.ok && c_out % 32 != 0 && dtype == HCH_F32 && aligned16(dY) && aligned16(dX) && aligned16(W)) {
            const double bytes = (double)n * (108.0 + 4.0 * c_out + 4.0 * c_in * d.splits) + 4.0 * wn;
            st = launch_direct(d, (const float *)dY, L->dnbr, (const float *)W, d.splits > 1 ? part : dX, n, c_out, c_in, bytes, s, 1,
                               skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr);
            if (st != HCH_OK) return st;
            if (d.splits > 1) st = launch_reduce(part, dX, n * c_in, d.splits, s);
            return st;
        }
        const GemmPlan p = plan_rows(n, c_in, Kd, true, k_gran(dtype));
        if (skip && dtype == HCH_F32 && conv_small_faster(n, c_out, c_in, true))
            return launch_conv_small(*L, (const float *)dY, (const float *)W, dX, n, c_out, c_in, true,
                                     (double)n * (108.0 + 4.0 * c_out + 4.0 * c_in) + 4.0 * wn, s);
        if (skip && dtype == HCH_F32 && L->rows()) {
            const ConvSplitPlan q = plan_conv_split(n, c_out, c_in, p.splits);
            if (q.ok)
                return launch_conv_split(q, *L, (const float *)dY, (const float *)W, dX, part, n, c_out, c_in, true,
                                         (double)n * (108.0 + 4.0 * c_out + 4.0 * c_in * q.splits) + 4.0 * wn, s);
        }
        if (skip && dtype == HCH_BF16 && conv_bf16_ok(*L, dY, W, n, c_out, c_in, true))
            return launch_conv_bf16(*L, (const uint16_t *)dY, (const uint16_t *)W, dX, n, c_out, c_in, true,
                                    (double)n * (108.0 + es * c_out + 4.0 * c_in) + es * wn, s);
        if (c_out % k_gran(dtype) == 0 && c_in % 4 == 0 && aligned16(dY) && aligned16(W)) {
            // the LDS-tiled kernel reads W[27][c_in][c_out] in place as the flipped, transposed
            // matrix: tap 26 - t of the weights for rows t*c_out .. (t+1)*c_out - 1
            const int64_t per_tap = (int64_t)c_in * c_out;
            const char *Wlast = (const char *)W + 26 * per_tap * elem_size(dtype);
            const double bytes = (double)n * (108.0 + es * c_out + 4.0 * c_in * p.splits) + es * wn;
            st = launch_gemm<hch::A_GATHER, true>(dtype, p, dY, Wlast, p.splits > 1 ? part : dX, L->dnbr, (int)n, c_in, Kd,
                                                  c_out, c_out, c_in, n * c_in, bytes, s, 0, 27, c_out, -per_tap, L->dnbr_t,
                                                  skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr, n);
            if (st != HCH_OK) return st;
            if (p.splits > 1) st = launch_reduce(part, dX, n * c_in, p.splits, s);
            return st;
        }
        if (dtype == HCH_F32) {
            hch::LaunchTimer lt(HCH_KERNEL_ID("flip_transpose_weights_kernel<float>"), s, 8.0 * wn, 0.0);
            HCH_LAUNCH(hch::flip_transpose_weights_kernel<float>, dim3(blocks_for(wn)), dim3(256), 0, s,
                               (const float *)W, (float *)Wt, c_in, c_out, 27, 1);
        } else {
            hch::LaunchTimer lt(HCH_KERNEL_ID("flip_transpose_weights_kernel<unsigned short>"), s, 4.0 * wn, 0.0);
            HCH_LAUNCH(hch::flip_transpose_weights_kernel<uint16_t>, dim3(blocks_for(wn)), dim3(256), 0, s,
                               (const uint16_t *)W, (uint16_t *)Wt, c_in, c_out, 27, 1);
        }
        HCH_LAUNCH_CHECK("flip_transpose_weights_kernel");
        const double bytes = (double)n * (108.0 + es * c_out + 4.0 * c_in * p.splits) + es * wn;
        st = launch_gemm<hch::A_GATHER, false>(dtype, p, dY, Wt,
                                               p.splits > 1 ? part : dX, L->dnbr, (int)n, c_in, Kd, c_out,
                                               c_in, c_in, n * c_in, bytes, s, 0, 27, 0, 0, L->dnbr_t,
                                               skip ? L->rows() : nullptr, skip ? L->row_taps() : nullptr, n);
        if (st != HCH_OK) return st;
        if (p.splits > 1) st = launch_reduce(part, dX, n * c_in, p.splits, s);
        return st;
    }

    float *dcol = (float *)workspace;
    // dcol[N x Kc] = dY[N x c_out] . W^T   (W is [Kc x c_out]: its rows are B's columns)
    const GemmPlan p = plan_rows(n, Kc, c_out, false, k_gran(dtype));
    // with few input channels dcol is stored tap-major ([27][n][c_in]) between the two kernels:
    // the gather then reads, tap by tap, 16- or 32-byte pieces of nearly consecutive rows that
    // lie next to each other, instead of one such piece out of every 27*c_in-float row.  (With
    // 16 channels or more a piece fills its own memory sectors and the row-major store of the
    // product is the cheaper one: measured.)
    const bool planes = c_in % 4 == 0 && c_in <= 8 && aligned16(dX);
    // Algorithm 2 adds dcol[i][k] to voxel nbr[i][k] and drops it where there is none: in the
    // tap-major form those pieces (two thirds of dcol at the finest level) are not stored; the
    // per-voxel bit sets of existing neighbours come with the index lists.  (Row-major, with 16 or
    // more channels, leaving pieces out of the rows made the product slower by more than the
    // gather gained: 96 -> 111 us and 45 -> 31 us at level 1, 72 -> 81 and 13 -> 13 at level 2.)
    const bool masked = planes && L->dmask27 != nullptr;
    const uint32_t *rowmask = masked ? L->dmask27 : nullptr;
    // bytes: dY and W in; all of dcol, or of it the pieces that have a destination, and 4 per row for the bit set
    const bool split = !planes && dtype == HCH_F32 && dcol_split_ok(n, c_in, c_out);
    const double bytes = es * ((double)n * c_out + (double)Kc * c_out) +
                         (masked && !split ? 4.0 * ((double)L->nbr_valid * c_in + (double)n) : 4.0 * (double)n * Kc);
    if (split) st = launch_dcol_split((const float *)dY, (const float *)W, dcol, n, c_in, c_out, bytes, s);
    else
        st = launch_gemm<hch::A_ROWS, true>(dtype, p, dY, W, dcol, nullptr,
                                            (int)n, Kc, c_out, c_out, c_out, Kc, 0, bytes, s, planes ? c_in : 0,
                                            27, 0, 0, nullptr, nullptr, nullptr, 0, rowmask, c_in);
    if (st != HCH_OK) return st;
    return do_col2hash(*L, dcol, c_in, dX, planes, s);
}

static hch_status conv_bwd_weight_impl(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                       const void *X, const void *dY, float *dW, int32_t c_in,
                                       int32_t c_out, void *workspace, size_t ws_bytes, hch_algo algo,
                                       void *stream, const char *who)
{
    const Level *L;
    const bool resident = algo == HCH_ALGO_COLUMNS_RESIDENT;     // the column matrix is in the workspace already
    if (resident) algo = HCH_ALGO_COLUMNS;
    const bool skip = algo == HCH_ALGO_FUSED;                    // absent taps may be left out
    if (algo == HCH_ALGO_FUSED_DENSE) algo = HCH_ALGO_FUSED;
    hch_status st = conv_args(levels, level, dtype, X, dY, dW, c_in, c_out, workspace, algo, &L, who);
    if (st != HCH_OK) return st;
    const WsLayout w = ws_layout(*L, c_in, c_out, dtype, HCH_WS_BWD_WEIGHT, algo, true);
    if (ws_bytes < std::max<size_t>(256, w.first_bytes + w.part_bytes))
        return fail(HCH_EWORKSPACE, std::string(who) + ": workspace too small");
    hipStream_t s = (hipStream_t)stream;
    const int Kc = 27 * c_in;
    const int64_t n = L->n_total;
    const double es = elem_size(dtype);
    const GemmPlan p = plan_wgrad(n, c_in, c_out, 27, k_gran(dtype));
    const int64_t wsize = (int64_t)Kc * c_out;
    float *part = (float *)((char *)workspace + w.first_bytes);
    float *dst = (p.splits == 1) ? dW : part;

    // dW[Kc x c_out] = col^T[Kc x N] . dY[N x c_out], reduction over the voxels split in slices
    if (algo == HCH_ALGO_FUSED) {
        if (skip && dtype == HCH_F32 && L->rows()) {
            const WgradSplitPlan q = plan_wgrad_split(n, n, c_in, c_out, 27, std::max<int64_t>(1, (int64_t)(ws_bytes / (4 * (size_t)wsize))));
            if (q.ok)
                return launch_wgrad_split(q, (const float *)X, (const float *)dY, dW, part, L->dnbr, L->rows(), n, n, c_in, c_out, 27,
                                          (double)n * (108.0 + 4.0 * c_in + 4.0 * c_out), s);
        }
        if (skip && dtype == HCH_BF16 && L->rows() && !((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(dY)) & 3u)) {
            const WgradSplitPlan q = plan_wgrad_bf16(n, c_in, c_out, std::max<int64_t>(1, (int64_t)(ws_bytes / (4 * (size_t)wsize))));
            if (q.ok)
                return launch_wgrad_bf16(q, (const uint16_t *)X, (const uint16_t *)dY, dW, part, L->dnbr, L->rows(), n, c_in, c_out,
                                         (double)n * (108.0 + 2.0 * c_in + 2.0 * c_out), s);
        }
        const double bytes = (double)n * (108.0 + es * c_in + es * c_out) + 4.0 * wsize * p.splits;
        st = launch_gemm<hch::A_GATHER_T, false>(dtype, p, X, dY, dst,
                                                 L->dnbr, Kc, c_out, (int)n, c_in, c_out, c_out, wsize, bytes, s, 0, 27, 0, 0, L->dnbr_t,
                                                 nullptr, nullptr, n);
    } else {
        void *col = workspace;
        if (!resident) {
            st = do_hash2col(*L, dtype, X, c_in, 0, n, col, s);
            if (st != HCH_OK) return st;
        }
        const double bytes = es * ((double)n * Kc + (double)n * c_out) + 4.0 * (double)wsize * p.splits;
        st = launch_gemm<hch::A_COLS, false>(dtype, p, col, dY, dst, nullptr,
                                             Kc, c_out, (int)n, Kc, c_out, c_out, wsize, bytes, s);
    }
    if (st != HCH_OK) return st;
    if (p.splits > 1) st = launch_reduce(part, dW, wsize, p.splits, s);
    return st;
}

extern "C" hch_status hch_conv_bwd_weight(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                          const void *X, const void *dY, float *dW, int32_t c_in,
                                          int32_t c_out, void *workspace, size_t ws_bytes, hch_algo algo,
                                          void *stream)
{
    return conv_bwd_weight_impl(levels, level, dtype, X, dY, dW, c_in, c_out, workspace, ws_bytes, algo, stream,
                                "hch_conv_bwd_weight");
}

// ---------------------------------------------------------------------------------------
// The weight gradient for callers that cannot allocate and bring no workspace: the partial sums of
// the split reduction live in a fixed array in device memory that every GPU the library runs on
// holds until the process ends.
// ---------------------------------------------------------------------------------------

// The array's name is only a host-side handle of the symbol; the device address is asked for
// once per device (each GPU has its own copy at its own address) and only that pointer is
// handed to kernels.
static __device__ __align__(256) unsigned char scratch[HCH_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::atomic<void *> g_scratch_ptr[MAX_DEVICES];
}

static hch_status scratch_address(void **out)
{
    int dev = -1;
    HCH_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(HCH_EUNSUPPORTED, "hch_conv_bwd_weight_noalloc: device ordinal above 63");
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        // two threads may both ask; they get the same answer
        HCH_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u))
            return fail(HCH_EHIP, "hch_conv_bwd_weight_noalloc: no usable address for the scratch array");
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return HCH_OK;
}

extern "C" hch_status hch_conv_bwd_weight_noalloc(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                                  const void *X, const void *dY, float *dW, int32_t c_in,
                                                  int32_t c_out, void *stream)
{
    if (!levels || level < 0 || level >= (int32_t)levels->lv.size() || c_in <= 0 || c_out <= 0)
        return fail(HCH_EINVAL, "hch_conv_bwd_weight_noalloc: bad level or channel count");
    if (dtype != HCH_F32 && dtype != HCH_BF16) return fail(HCH_EINVAL, "hch_conv_bwd_weight_noalloc: unknown dtype");
    if ((int64_t)27 * c_in * c_out >= ((int64_t)1 << 31))
        return fail(HCH_EINVAL, "hch_conv_bwd_weight_noalloc: weight tensor too large");
    const size_t need = hch_conv_workspace_bytes(levels, level, c_in, c_out, dtype, HCH_WS_BWD_WEIGHT, HCH_ALGO_FUSED);
    if (need == 0 || need > (size_t)HCH_NOALLOC_SCRATCH_BYTES)
        return fail(HCH_EWORKSPACE, "hch_conv_bwd_weight_noalloc: the partial sums of this product need " +
                                        std::to_string(need) + " bytes, the built-in scratch array holds " +
                                        std::to_string((size_t)HCH_NOALLOC_SCRATCH_BYTES) +
                                        "; use hch_conv_bwd_weight with a workspace");
    void *ptr = nullptr;
    hch_status st = scratch_address(&ptr);
    if (st != HCH_OK) return st;
    // every slice of the split reduction writes all of its 27*c_in*c_out partial sums (zeros where
    // its range of voxels is empty) before the reduction kernel reads them: nothing has to be
    // cleared between calls
    return conv_bwd_weight_impl(levels, level, dtype, X, dY, dW, c_in, c_out, ptr, (size_t)HCH_NOALLOC_SCRATCH_BYTES,
                                HCH_ALGO_FUSED, stream, "hch_conv_bwd_weight_noalloc");
}

// ---------------------------------------------------------------------------------------
// pooling, ReLU
// ---------------------------------------------------------------------------------------

extern "C" hch_status hch_pool_fwd(const hch_levels *levels, int32_t level_in, const float *X,
                                   float *Y, int32_t *argmax, int32_t c, void *stream)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_pool_fwd: level_in must have a coarser level");
    if (!X || !Y || !argmax || c <= 0) return fail(HCH_EINVAL, "hch_pool_fwd: bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_pool_fwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_pool_fwd: levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(X) && aligned16(Y) && aligned16(argmax);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_pool_fwd: too large");
    {
        // per coarse voxel: 8 child indices, its children's rows in; value and switch rows out
        const Level &Lf = levels->lv[level_in];
        const double bytes = (double)Lc.n_total * (32.0 + 8.0 * c) + (double)Lf.n_total * 4.0 * c;
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("pool_fwd_kernel<4>") : HCH_KERNEL_ID("pool_fwd_kernel<1>"), (hipStream_t)stream, bytes, 0.0);
        if (vec)
            HCH_LAUNCH(hch::pool_fwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               X, Lc.dchild, Y, argmax, Lc.n_total, c);
        else
            HCH_LAUNCH(hch::pool_fwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               X, Lc.dchild, Y, argmax, Lc.n_total, c);
    }
    HCH_LAUNCH_CHECK("pool_fwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_pool_bwd(const hch_levels *levels, int32_t level_in, const float *dY,
                                   const int32_t *argmax, float *dX, int32_t c, void *stream)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_pool_bwd: level_in must have a coarser level");
    if (!dY || !argmax || !dX || c <= 0) return fail(HCH_EINVAL, "hch_pool_bwd: bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_pool_bwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_pool_bwd: levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(dY) && aligned16(dX) && aligned16(argmax);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (Lc.n_total * 8 * (vec ? c / 4 : c) > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_pool_bwd: too large");
    {
        const Level &Lf = levels->lv[level_in];
        const double bytes = (double)Lc.n_total * (32.0 + 8.0 * c) + (double)Lf.n_total * 4.0 * c;
        const bool few = items < hch::POOL_BWD_FEW;
#define HCH_POOL_BWD(VEC_, KIDS_)                                                                                     \
        do {                                                                                                          \
            hch::LaunchTimer lt(HCH_KERNEL_ID("pool_bwd_kernel<" #VEC_ ", " #KIDS_ ">"), (hipStream_t)stream, bytes, 0.0); \
            HCH_LAUNCH((hch::pool_bwd_kernel<VEC_, KIDS_>), dim3(blocks_for(items * (8 / KIDS_))), dim3(256), 0,      \
                               (hipStream_t)stream, dY, argmax, Lc.dchild, dX, Lc.n_total, c);                        \
        } while (0)
        if (vec) { if (few) HCH_POOL_BWD(4, 1); else HCH_POOL_BWD(4, 8); }
        else { if (few) HCH_POOL_BWD(1, 1); else HCH_POOL_BWD(1, 8); }
#undef HCH_POOL_BWD
    }
    HCH_LAUNCH_CHECK("pool_bwd_kernel");
    return HCH_OK;
}

// ---------------------------------------------------------------------------------------
// transposed convolution and max-unpooling (paper Section 4, last paragraphs): the same
// products with the roles of input and output exchanged
// ---------------------------------------------------------------------------------------

extern "C" hch_status hch_deconv_fwd(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                     const void *X, const void *W, float *Y, int32_t c_in,
                                     int32_t c_out, void *workspace, size_t ws_bytes, hch_algo algo,
                                     void *stream)
{
    // Y = col2hash(X . W^T): the data-gradient path of the convolution c_out -> c_in
    return hch_conv_bwd_data(levels, level, dtype, X, W, Y, c_out, c_in, workspace, ws_bytes, algo, stream);
}

extern "C" hch_status hch_deconv_bwd_data(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                          const void *dY, const void *W, float *dX, int32_t c_in,
                                          int32_t c_out, void *workspace, size_t ws_bytes,
                                          hch_algo algo, void *stream)
{
    // the adjoint of the above is the forward convolution c_out -> c_in
    return hch_conv_fwd(levels, level, dtype, dY, W, dX, c_out, c_in, workspace, ws_bytes, algo, stream);
}

extern "C" hch_status hch_deconv_bwd_weight(const hch_levels *levels, int32_t level, hch_dtype dtype,
                                            const void *X, const void *dY, float *dW, int32_t c_in,
                                            int32_t c_out, void *workspace, size_t ws_bytes,
                                            hch_algo algo, void *stream)
{
    // dW[27][c_out][c_in] = hash2col(dY)^T . X: the weight gradient of the convolution c_out -> c_in
    // whose input is dY and whose output gradient is X
    return hch_conv_bwd_weight(levels, level, dtype, dY, X, dW, c_out, c_in, workspace, ws_bytes, algo, stream);
}

extern "C" hch_status hch_unpool_fwd(const hch_levels *levels, int32_t level_out, const float *Xc,
                                     const int32_t *argmax, float *Y, int32_t c, void *stream)
{
    return hch_pool_bwd(levels, level_out, Xc, argmax, Y, c, stream);
}

extern "C" hch_status hch_unpool_bwd(const hch_levels *levels, int32_t level_out, const float *dY,
                                     const int32_t *argmax, float *dXc, int32_t c, void *stream)
{
    if (!levels || level_out < 0 || level_out + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_unpool_bwd: level_out must have a coarser level");
    if (!dY || !argmax || !dXc || c <= 0) return fail(HCH_EINVAL, "hch_unpool_bwd: bad argument");
    const Level &Lc = levels->lv[level_out + 1];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_unpool_bwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_unpool_bwd: levels were built without device tables");
    const int64_t items = Lc.n_total * c;
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_unpool_bwd: too large");
    if (items == 0) return HCH_OK;
    {
        const bool vec = c % 4 == 0 && aligned16(argmax) && aligned16(dXc);
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("unpool_bwd_kernel<4>") : HCH_KERNEL_ID("unpool_bwd_kernel<1>"), (hipStream_t)stream, 12.0 * items, 0.0);
        if (vec)
            HCH_LAUNCH(hch::unpool_bwd_kernel<4>, dim3(blocks_for(items / 4)), dim3(256), 0, (hipStream_t)stream,
                               dY, argmax, dXc, Lc.n_total, c);
        else
            HCH_LAUNCH(hch::unpool_bwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               dY, argmax, dXc, Lc.n_total, c);
    }
    HCH_LAUNCH_CHECK("unpool_bwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_relu_pool_fwd(const hch_levels *levels, int32_t level_in, const float *Y,
                                        float *A, float *P, int32_t *argmax, int32_t c, void *stream)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_relu_pool_fwd: level_in must have a coarser level");
    if (!Y || !P || !argmax || c <= 0) return fail(HCH_EINVAL, "hch_relu_pool_fwd: bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    const Level &Lf = levels->lv[level_in];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_relu_pool_fwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_relu_pool_fwd: levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(Y) && (!A || aligned16(A)) && aligned16(P) && aligned16(argmax);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_relu_pool_fwd: too large");
    {
        // per fine voxel: its row in (and its rectified row out when A is given); per coarse
        // voxel: 8 indices in, value and switch rows out
        const double bytes = (double)Lf.n_total * (A ? 8.0 : 4.0) * c + (double)Lc.n_total * (32.0 + 8.0 * c);
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("relu_pool_fwd_kernel<4>") : HCH_KERNEL_ID("relu_pool_fwd_kernel<1>"),
                            (hipStream_t)stream, bytes, 0.0);
        if (vec)
            HCH_LAUNCH(hch::relu_pool_fwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               Y, Lc.dchild, A, P, argmax, Lc.n_total, c);
        else
            HCH_LAUNCH(hch::relu_pool_fwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               Y, Lc.dchild, A, P, argmax, Lc.n_total, c);
    }
    HCH_LAUNCH_CHECK("relu_pool_fwd_kernel");
    return HCH_OK;
}

// shared by the two forms of the fused backward step: `sign` holds fine rows (A or Y) or, pooled, the rows P
static hch_status pool_relu_bwd_impl(const hch_levels *levels, int32_t level_in, const float *dP,
                                     const int32_t *argmax, const float *sign, bool pooled, float *dY, int32_t c,
                                     void *stream, const char *who)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, std::string(who) + ": level_in must have a coarser level");
    if (!dP || !argmax || !sign || !dY || c <= 0) return fail(HCH_EINVAL, std::string(who) + ": bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    const Level &Lf = levels->lv[level_in];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, std::string(who) + ": these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, std::string(who) + ": levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(dP) && aligned16(argmax) && aligned16(sign) && aligned16(dY);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, std::string(who) + ": too large");
    {
        // per fine voxel: its gradient row out (and its row in, unless the pooled rows stand in);
        // per coarse voxel: 8 indices, gradient and switch rows (and the pooled row) in
        const double bytes = (double)Lf.n_total * (pooled ? 4.0 : 8.0) * c + (double)Lc.n_total * (32.0 + (pooled ? 12.0 : 8.0) * c);
        const int kid = pooled ? (vec ? HCH_KERNEL_ID("pool_relu_bwd_kernel<4, true>") : HCH_KERNEL_ID("pool_relu_bwd_kernel<1, true>"))
                               : (vec ? HCH_KERNEL_ID("pool_relu_bwd_kernel<4, false>") : HCH_KERNEL_ID("pool_relu_bwd_kernel<1, false>"));
        hch::LaunchTimer lt(kid, (hipStream_t)stream, bytes, 0.0);
#define HCH_POOL_RELU_BWD(VEC_, POOLED_)                                                                             \
    HCH_LAUNCH((hch::pool_relu_bwd_kernel<VEC_, POOLED_>), dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream, \
                       dP, argmax, Lc.dchild, sign, dY, Lc.n_total, c)
        if (pooled) { if (vec) HCH_POOL_RELU_BWD(4, true); else HCH_POOL_RELU_BWD(1, true); }
        else { if (vec) HCH_POOL_RELU_BWD(4, false); else HCH_POOL_RELU_BWD(1, false); }
#undef HCH_POOL_RELU_BWD
    }
    HCH_LAUNCH_CHECK("pool_relu_bwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_pool_relu_bwd(const hch_levels *levels, int32_t level_in, const float *dP,
                                        const int32_t *argmax, const float *A, float *dY, int32_t c,
                                        void *stream)
{
    return pool_relu_bwd_impl(levels, level_in, dP, argmax, A, false, dY, c, stream, "hch_pool_relu_bwd");
}

extern "C" hch_status hch_pool_relu_bwd_pooled(const hch_levels *levels, int32_t level_in, const float *dP,
                                               const int32_t *argmax, const float *P, float *dY, int32_t c,
                                               void *stream)
{
    return pool_relu_bwd_impl(levels, level_in, dP, argmax, P, true, dY, c, stream, "hch_pool_relu_bwd_pooled");
}

// ---------------------------------------------------------------------------------------
// general kernel side / stride / padding (Algorithm 1 and 2 as stated), average pooling
// ---------------------------------------------------------------------------------------

// level_out for a field of stride S read at level_in, or a failure
static hch_status field_levels(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride, int32_t pad,
                               const Level **Li, const Level **Lo, const char *who)
{
    if (!levels) return fail(HCH_EINVAL, std::string(who) + ": null levels");
    if (F < 1 || F > 7) return fail(HCH_EINVAL, std::string(who) + ": kernel side must be 1..7");
    if (stride < 1) return fail(HCH_EINVAL, std::string(who) + ": stride must be positive");
    if (stride == 1 && (F % 2 == 0 || pad != (F - 1) / 2))
        return fail(HCH_EINVAL, std::string(who) + ": a stride-1 field is centred: odd kernel side, padding (F-1)/2");
    if (pad < 0 || pad >= F) return fail(HCH_EINVAL, std::string(who) + ": padding must be in [0, F)");
    if (level_in < 0 || level_in >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, std::string(who) + ": level out of range");
    // the output level: the one whose side relates to level_in's by exactly `stride`
    int shift = 0;
    int64_t prod = 1;
    while (prod < stride && level_in + shift + 1 < (int32_t)levels->lv.size()) {
        ++shift;
        prod *= levels->lv[level_in + shift].ratio;
    }
    if (prod != stride)
        return fail(HCH_EINVAL, std::string(who) + ": no level of this set is `stride` times coarser than level_in");
    *Li = &levels->lv[level_in];
    *Lo = &levels->lv[level_in + shift];
    if (!(*Li)->dslot3 || !(*Lo)->dslot3) return fail(HCH_EINVAL, std::string(who) + ": levels were built without device tables");
    return HCH_OK;
}

extern "C" hch_status hch_field_build(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                      int32_t pad, int32_t *field, int32_t *field_t, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = field_levels(levels, level_in, F, stride, pad, &Li, &Lo, "hch_field_build");
    if (st != HCH_OK) return st;
    if (!field && !field_t) return fail(HCH_EINVAL, "hch_field_build: nothing to build");
    const int F3 = F * F * F;
    hipStream_t s = (hipStream_t)stream;
    auto build = [&](auto transposed, const Level &owner, const Level &probe, int32_t *out, int reversed) {
        constexpr bool T = decltype(transposed)::value;
        // planes of rows per workgroup (see field_kernel): enough workgroups for 3 per CU, and their rows
        // of 64 voxels in at most 32 KB of LDS (5 workgroups per CU) or else one plane of at most 64 KB.
        // Of 256, 512, 768 and 1024 workgroups, 768 is the best or within 0.5 us of it from 200 to 609k voxels.
        const int step = T ? std::min(stride, F) : 1, K = (F + step - 1) / step, plane = step * F * F * 4;
        const int64_t tiles = (owner.max_n + 63) / 64 * (int64_t)owner.b;
        int slabs = (int)std::max<int64_t>(1, std::min<int64_t>(K, K * tiles / 768));
        slabs = std::max(1, std::min(slabs, 32768 / (64 * plane)));
        const int tv = std::min(slabs * step, F) * F * F * 4 * 64 <= 65536 ? 64 : 32;
        const unsigned z = (unsigned)((K + slabs - 1) / slabs);
        const size_t lds = (size_t)tv * std::min(slabs * step, F) * F * F * 4;
        // fewer than 64 wavefronts per CU: twice as many (5^3, 40k voxels 38 -> 31 us, 3^3 12.2 -> 11.1)
        const unsigned threads = tiles * z < 4096 ? 512 : 256;
        hch::LaunchTimer lt(T ? HCH_KERNEL_ID("field_kernel<true>") : HCH_KERNEL_ID("field_kernel<false>"), s,
                            (double)owner.n_total * (12.0 + 4.0 * F3), 0.0);
        HCH_LAUNCH(hch::field_kernel<T>, dim3((unsigned)((owner.max_n + tv - 1) / tv), (unsigned)owner.b, z), dim3(threads), lds, s,
                   probe.view(), owner.dcoords, owner.dN(), out, F, stride, pad, tv, slabs, reversed);
    };
    if (field) build(std::false_type{}, *Lo, *Li, field, 0);
    if (field_t && stride == 1) build(std::false_type{}, *Li, *Lo, field_t, 1);
    else if (field_t) build(std::true_type{}, *Li, *Lo, field_t, 0);
    HCH_LAUNCH_CHECK("field_kernel");
    return HCH_OK;
}

// Products over general index rows on split operands (field_split_kernel): `M` index rows of `taps` entries into the
// x_rows rows of X, c channels to N; the cut weights take field_weights_bytes of workspace.
static size_t field_weights_bytes(int taps, int c, int N)
{
    return (size_t)taps * (size_t)((c + 7) / 8) * (size_t)((N + 15) / 16) * 768;
}

enum FieldUse { FIELD_FWD, FIELD_BWD, FIELD_BWD_STRIDED };

// Forward and the data gradient within a level against gemm_f32_kernel on its vector path.  Both take a time that goes with the
// rows per CU in whole rounds of workgroups, of 64 or 128 rows there and of 256 here: 20 -> 64 at 66 000, 75 000 and 127 000
// rows (258, 293 and 496 workgroups) 57, 58 and 86 us there, 69, 78 and 80 here.  A row and term of a tile of 16, 32 or 64 columns
// takes 1.0, 1.5 or 2.66e-4 us there; here that times the factors below (the taps that 16 rows leave out), with channels
// padded to 8.  Fitted to 4680 shapes (3^3 and 2^3, 8 to 128 channels, 50 000 to 420 000 rows): without this 533 of them were
// slower here by more than 2 %, up to 38 %; with it 79, by 10 % at most, and 103 go there that would be faster here.
static bool field_split_faster(int64_t M, int64_t x_rows, int taps, int c, int N)
{
    // one tap: nothing to leave out (279 722 rows, 256 -> 64 110 us there, 164 here; 64 -> 256 137 and 146)
    if (taps == 1) return false;
    // 2^3 fields of stride 2 read every row once, there in order: beyond the last-level cache that is what counts (609 000 rows
    // of 128 channels, 312 MB, to 32: 149 us there, 180 here; 500 000, 256 MB: 112 and 125; 400 000, 205 MB: 89 and 77)
    if (taps < 27 && x_rows * c * 4 > (int64_t)224 << 20) return false;
    const GemmPlan p = plan_rows(M, N, taps * c, true);
    const int64_t n_tiles = (N + p.bn - 1) / p.bn, tiles = (M + p.bm - 1) / p.bm * n_tiles;
    const int64_t groups = (M + hch::FIELD_ROWS - 1) / hch::FIELD_ROWS * n_tiles, rest = groups % 256;
    const double there = (double)((tiles + 255) / 256) * p.bm * taps * c;
    // up to 5 workgroups more than a whole round are less than one
    const double rounds = (double)(groups / 256) + (rest ? std::min(1.0, 0.5 + (double)rest / 10) : 0.0);
    const double factor = taps < 27 ? 0.74 : (p.bn == 64 ? 0.66 : (p.bn == 32 ? 0.68 : 0.74));
    const double here = rounds * hch::FIELD_ROWS * taps * ((c + 7) / 8 * 8) * factor;
    const double unit = p.bn == 16 ? 1.0e-4 : (p.bn == 32 ? 1.5e-4 : 2.66e-4);
    return 4.0 + unit * here < unit * there;          // 4 us: the weights are cut in a launch of their own
}

// Whether that is the faster way, and within its limits.  Its results are closer to the exact ones than those of the
// fp32 instruction, as everywhere on split operands.  gemm_vec: gemm_f32_kernel has its vector path for these operands, else it
// takes 1.3 to 5 times as long.
static bool field_split_ok(FieldUse use, bool gemm_vec, int64_t M, int64_t x_rows, int taps, int c, int N, size_t ws_bytes)
{
    const int64_t lim = (int64_t)1 << 31;
    // 32-bit byte offsets reach everything, a negative one nothing; 24-bit row and row-length factors; a bit per tap
    if (taps > 32 || x_rows >= (1 << 23) || c * 4 >= (1 << 23) || x_rows * c * 4 >= lim || M * taps >= lim || (int64_t)N * c * taps * 6 >= lim / 4 ||
        field_weights_bytes(taps, c, N) > ws_bytes)
        return false;
    // 256 rows to a workgroup, and some 10 us until the first sums: with fewer rows the chip stands empty (16 000 rows, 32 ->
    // 64, 3^3: forward 15 us on the fp32 instruction, 51 here; data gradient of stride 2 19 and 33)
    if (M < 49152) return false;
    const double work = (double)M * taps * c * N;
    // Forward: 3^3, 64 000 rows 24 -> 40 (1.7e9) 60 -> 50 us, 16 -> 32 (0.9e9) 26.5 and 27.6; 197 000 rows 16 -> 32 (2.7e9) 77 ->
    // 71, 32 -> 64 229 -> 175; 82 000 rows 32 -> 32 (2.3e9) 62 and 63; 2^3, 82 000 rows 32 -> 64 (1.3e9) 39 and 44.  Rows of 4
    // channels are half padding.
    if (use == FIELD_FWD) return c >= 16 && work >= 1.6e9 && (N > 32 || M >= 98304) && (!gemm_vec || field_split_faster(M, x_rows, taps, c, N));
    if (taps * c < 256) return false;                  // 2^3, 16 -> 4 at 609 000 rows: 30 us, 37 here
    // Data gradient within a level: 64 000 rows 32 -> 16 (0.9e9) 33 and 35 us, 40 -> 24 (1.7e9) 57 -> 49; 280 000 rows 16 -> 4 67 -> 58,
    // 32 -> 16 115 -> 91, 64 -> 32 305 -> 231
    if (use == FIELD_BWD) return (work >= 1.6e9 || M >= 262144) && (!gemm_vec || field_split_faster(M, x_rows, taps, c, N));
    // Between levels, against the gradient of the column matrix through memory: 609 000 rows, stride 2, 32 -> 16 208 -> 84 us, 64 -> 32
    // 438 -> 176, 16 -> 4 84 -> 64; where that matrix is small (3^3, stride 4, 64 000 rows, 32 -> 16: 2.3 M elements) 14.6 and
    // 15.6, with 3.5 M 25 -> 19.  Few columns leave most of the matrix tile empty: 280 000 rows, 64 -> 4 52 and 70, 50 -> 7 96 -> 66;
    // of whole 16 bytes, 207 000 rows, 28 -> 4 35 and 38, 24 -> 4 35 and 36, 40 -> 8 55 -> 45, and 2^3, 32 -> 8 20 and 22 (400 000 27
    // and 32), 32 -> 12 26 -> 22
    if (N < 16 && (gemm_vec ? c > 6 * N || taps * N < 96 : c >= 8 * N)) return false;
    return (double)x_rows * taps * N >= 3e6;
}

static hch_status launch_field_split(const float *X, const float *W, float *out, const int32_t *field, void *ws, int64_t M, int64_t x_rows,
                                     int taps, int c, int N, bool transposed, double bytes, hipStream_t s)
{
    hch::u32x4 *wp = (hch::u32x4 *)ws;
    const size_t wbytes = field_weights_bytes(taps, c, N);
    {
        hch::LaunchTimer lt(transposed ? HCH_KERNEL_ID("split_weights_kernel<true>") : HCH_KERNEL_ID("split_weights_kernel<false>"), s,
                            4.0 * taps * c * N + (double)wbytes, 0.0);
        const dim3 grid(blocks_for((int64_t)(wbytes / 48)));
        if (transposed) HCH_LAUNCH(hch::split_weights_kernel<true>, grid, dim3(256), 0, s, W, wp, taps, c, N);
        else HCH_LAUNCH(hch::split_weights_kernel<false>, grid, dim3(256), 0, s, W, wp, taps, c, N);
    }
    HCH_LAUNCH_CHECK("split_weights_kernel");
    const int nt = N <= 16 ? 1 : (N <= 32 ? 2 : 4);
    const unsigned tiles = (unsigned)((M + hch::FIELD_ROWS - 1) / hch::FIELD_ROWS);
    const dim3 grid((tiles + hch::NUM_XCD - 1) / hch::NUM_XCD * hch::NUM_XCD, (unsigned)((N + 16 * nt - 1) / (16 * nt)));
    const int vec_out = N % 4 == 0 && aligned16(out);
    const size_t lds = (size_t)hch::FieldLds::bytes(taps);
    {
        static int ids[3][2];
        static const bool ids_ready = [] { memset(ids, 0xFF, sizeof ids); return true; }();
        (void)ids_ready;
        int &id = ids[nt / 2][transposed];
        if (id < 0) {
            char nm[96];
            snprintf(nm, sizeof nm, "field_split_kernel<%d, %s>", nt, transposed ? "true" : "false");
            id = hch::Profiler::get().id_for(nm);
        }
        hch::LaunchTimer lt(id, s, bytes, 2.0 * taps * c * (double)N * M);
#define HCH_FIELD_CASE(NT_, T_)                                                                                          \
        HCH_LAUNCH((hch::field_split_kernel<NT_, T_>), grid, dim3(64 * hch::FIELD_WAVES), lds, s, X, W, (const hch::u32x4 *)wp, out, \
                   field, (int)M, N, c, taps, x_rows, tiles, vec_out)
        if (transposed) { if (nt == 1) HCH_FIELD_CASE(1, true); else if (nt == 2) HCH_FIELD_CASE(2, true); else HCH_FIELD_CASE(4, true); }
        else { if (nt == 1) HCH_FIELD_CASE(1, false); else if (nt == 2) HCH_FIELD_CASE(2, false); else HCH_FIELD_CASE(4, false); }
#undef HCH_FIELD_CASE
    }
    HCH_LAUNCH_CHECK("field_split_kernel");
    return HCH_OK;
}

// workspace of the three products of a general convolution: [ transposed weights (bwd_data on one
// level) or the column-matrix gradient (bwd_data between two levels) | split partial sums ];
// least: as in ws_layout
static WsLayout sconv_layout(const Level &Li, const Level &Lo, int taps, int c_in, int c_out, hch_dtype dtype, hch_ws_kind kind,
                             bool least = false)
{
    WsLayout w{0, 0};
    if (kind == HCH_WS_FWD) {
        const GemmPlan p = plan_rows(Lo.n_total, c_out, taps * c_in, true, k_gran(dtype));
        if (p.splits > 1) w.part_bytes = round_up((size_t)p.splits * Lo.n_total * c_out * 4, 256);
        if (dtype == HCH_F32 && !least) w.part_bytes = std::max(w.part_bytes, field_weights_bytes(taps, c_in, c_out));
    } else if (kind == HCH_WS_BWD_DATA && &Li != &Lo) {
        // between two levels: the gradient of the column matrix, [N_out][taps*c_in] floats, unless the product goes without it
        // (what does so on the vector path of gemm_f32_kernel does so without it too)
        const size_t cut = field_weights_bytes(taps, c_out, c_in);
        if (dtype == HCH_F32 && field_split_ok(FIELD_BWD_STRIDED, true, Li.n_total, Lo.n_total, taps, c_out, c_in, cut)) w.first_bytes = round_up(cut, 256);
        else w.first_bytes = round_up((size_t)Lo.n_total * taps * c_in * 4, 256);
    } else if (kind == HCH_WS_BWD_DATA) {
        const GemmPlan p = plan_rows(Li.n_total, c_in, taps * c_out, true, k_gran(dtype));
        w.first_bytes = round_up((size_t)taps * c_in * c_out * elem_size(dtype), 256);
        if (p.splits > 1) w.part_bytes = round_up((size_t)p.splits * Li.n_total * c_in * 4, 256);
        if (dtype == HCH_F32 && !least) w.part_bytes = std::max(w.part_bytes, field_weights_bytes(taps, c_out, c_in));
    } else {
        int splits = plan_wgrad(Lo.n_total, c_in, c_out, taps, k_gran(dtype)).splits;
        if (dtype == HCH_F32 && !least) {
            const WgradSplitPlan q = plan_wgrad_split(Lo.n_total, Li.n_total, c_in, c_out, taps, INT32_MAX);
            if (q.ok) splits = std::max(splits, q.slices);
        }
        if (splits > 1) w.part_bytes = round_up((size_t)splits * taps * c_in * c_out * 4, 256);
    }
    return w;
}

extern "C" size_t hch_sconv_workspace_bytes(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                            int32_t c_in, int32_t c_out, hch_dtype dtype, hch_ws_kind kind)
{
    const Level *Li, *Lo;
    if (c_in <= 0 || c_out <= 0 || (kind != HCH_WS_FWD && kind != HCH_WS_BWD_DATA && kind != HCH_WS_BWD_WEIGHT)) return 0;
    if (field_levels(levels, level_in, F, stride, stride == 1 ? (F - 1) / 2 : 0, &Li, &Lo, "hch_sconv_workspace_bytes") != HCH_OK) return 0;
    const WsLayout w = sconv_layout(*Li, *Lo, F * F * F, c_in, c_out, dtype, kind);
    return std::max<size_t>(256, w.first_bytes + w.part_bytes);
}

static hch_status sconv_args(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride, hch_dtype dtype,
                             const void *a, const void *b, const void *c, const void *idx, int32_t c_in, int32_t c_out,
                             const void *ws, size_t ws_bytes, hch_ws_kind kind, const Level **Li, const Level **Lo,
                             const char *who)
{
    hch_status st = field_levels(levels, level_in, F, stride, stride == 1 ? (F - 1) / 2 : 0, Li, Lo, who);
    if (st != HCH_OK) return st;
    if (!a || !b || !c || !idx || !ws || c_in <= 0 || c_out <= 0)
        return fail(HCH_EINVAL, std::string(who) + ": null pointer or non-positive channel count");
    if ((int64_t)F * F * F * c_in * c_out >= ((int64_t)1 << 31)) return fail(HCH_EINVAL, std::string(who) + ": weight tensor too large");
    if (dtype != HCH_F32 && dtype != HCH_BF16) return fail(HCH_EINVAL, std::string(who) + ": unknown dtype");
    if (reinterpret_cast<uintptr_t>(ws) & 255u) return fail(HCH_EINVAL, std::string(who) + ": workspace must be 256-byte aligned");
    if (std::max((*Li)->n_total, (*Lo)->n_total) >= ((int64_t)1 << 31) / 512)
        return fail(HCH_EUNSUPPORTED, std::string(who) + ": too many voxels");
    if (std::max((*Li)->n_total, (*Lo)->n_total) * (int64_t)std::max(c_in, c_out) >= ((int64_t)1 << 31))
        return fail(HCH_EUNSUPPORTED, std::string(who) + ": a feature matrix of more than 2^31 elements");
    const WsLayout w = sconv_layout(**Li, **Lo, F * F * F, c_in, c_out, dtype, kind, true);
    if (ws_bytes < std::max<size_t>(256, w.first_bytes + w.part_bytes))
        return fail(HCH_EWORKSPACE, std::string(who) + ": workspace too small");
    return HCH_OK;
}

extern "C" hch_status hch_sconv_fwd(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                    hch_dtype dtype, const void *X, const void *W, float *Y, const int32_t *field,
                                    int32_t c_in, int32_t c_out, void *workspace, size_t ws_bytes, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = sconv_args(levels, level_in, F, stride, dtype, X, W, Y, field, c_in, c_out, workspace, ws_bytes,
                               HCH_WS_FWD, &Li, &Lo, "hch_sconv_fwd");
    if (st != HCH_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const int taps = F * F * F, K = taps * c_in;
    const int64_t n = Lo->n_total;
    const double es = elem_size(dtype);
    const GemmPlan p = plan_rows(n, c_out, K, true, k_gran(dtype));
    float *part = (float *)workspace;
    const double bytes = (double)n * (4.0 * taps + 4.0 * c_out * p.splits) + es * (double)Li->n_total * c_in + es * K * c_out;
    const bool gemm_vec = c_in % 4 == 0 && c_out % 4 == 0 && aligned16(X) && aligned16(W);
    if (dtype == HCH_F32 && field_split_ok(FIELD_FWD, gemm_vec, n, Li->n_total, taps, c_in, c_out, ws_bytes))
        return launch_field_split((const float *)X, (const float *)W, Y, field, workspace, n, Li->n_total, taps, c_in, c_out, false,
                                  (double)n * (4.0 * taps + 4.0 * c_out) + 4.0 * ((double)Li->n_total * c_in + (double)K * c_out), s);
    st = launch_gemm<hch::A_GATHER, false>(dtype, p, X, W, p.splits > 1 ? part : Y, field, (int)n, c_out, K, c_in,
                                           c_out, c_out, n * c_out, bytes, s, 0, taps);
    if (st != HCH_OK) return st;
    if (p.splits > 1) st = launch_reduce(part, Y, n * c_out, p.splits, s);
    return st;
}

extern "C" hch_status hch_sconv_bwd_weight(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                           hch_dtype dtype, const void *X, const void *dY, float *dW,
                                           const int32_t *field, int32_t c_in, int32_t c_out, void *workspace,
                                           size_t ws_bytes, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = sconv_args(levels, level_in, F, stride, dtype, X, dY, dW, field, c_in, c_out, workspace, ws_bytes,
                               HCH_WS_BWD_WEIGHT, &Li, &Lo, "hch_sconv_bwd_weight");
    if (st != HCH_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const int taps = F * F * F, K = taps * c_in;
    const int64_t n = Lo->n_total, wsize = (int64_t)K * c_out;
    const double es = elem_size(dtype);
    const GemmPlan p = plan_wgrad(n, c_in, c_out, taps, k_gran(dtype));
    if (dtype == HCH_F32) {
        const WgradSplitPlan q = plan_wgrad_split(n, Li->n_total, c_in, c_out, taps, std::max<int64_t>(1, (int64_t)(ws_bytes / (4 * (size_t)wsize))));
        if (q.ok)
            return launch_wgrad_split(q, (const float *)X, (const float *)dY, dW, (float *)workspace, field, nullptr, n, Li->n_total,
                                      c_in, c_out, taps, (double)n * (4.0 * taps + 4.0 * c_out) + 4.0 * (double)Li->n_total * c_in, s);
    }
    float *part = (float *)workspace;
    const double bytes = (double)n * (4.0 * taps + es * c_out) + es * (double)Li->n_total * c_in + 4.0 * wsize * p.splits;
    st = launch_gemm<hch::A_GATHER_T, false>(dtype, p, X, dY, p.splits == 1 ? dW : part, field, K, c_out, (int)n, c_in,
                                             c_out, c_out, wsize, bytes, s, 0, taps);
    if (st != HCH_OK) return st;
    if (p.splits > 1) st = launch_reduce(part, dW, wsize, p.splits, s);
    return st;
}

extern "C" hch_status hch_sconv_bwd_data(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                         hch_dtype dtype, const void *dY, const void *W, float *dX,
                                         const int32_t *field_t, int32_t c_in, int32_t c_out, void *workspace,
                                         size_t ws_bytes, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = sconv_args(levels, level_in, F, stride, dtype, dY, W, dX, field_t, c_in, c_out, workspace, ws_bytes,
                               HCH_WS_BWD_DATA, &Li, &Lo, "hch_sconv_bwd_data");
    if (st != HCH_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    const int taps = F * F * F, Kd = taps * c_out;
    const int64_t n = Li->n_total, wn = (int64_t)taps * c_in * c_out;
    const double es = elem_size(dtype);
    const WsLayout w = sconv_layout(*Li, *Lo, taps, c_in, c_out, dtype, HCH_WS_BWD_DATA, true);
    // (within a level the weights are transposed into the workspace first; between two, rows of c_in enter only the gather)
    const bool gemm_vec = c_out % 4 == 0 && aligned16(dY) && (Li == Lo ? c_in % 4 == 0 : aligned16(W));
    if (dtype == HCH_F32 && field_split_ok(Li == Lo ? FIELD_BWD : FIELD_BWD_STRIDED, gemm_vec, n, Lo->n_total, taps, c_out, c_in, ws_bytes))
        return launch_field_split((const float *)dY, (const float *)W, dX, field_t, workspace, n, Lo->n_total, taps, c_out, c_in, true,
                                  (double)n * (4.0 * taps + 4.0 * c_in) + 4.0 * ((double)Lo->n_total * c_out + (double)wn), s);
    if (Li != Lo) {
        // Between two levels only about one field row in stride^3 of an input voxel has an owner,
        // so the gathered product below would multiply mostly zeros.  Here the paper's own order
        // is the cheaper one: dcol[N_out][taps*c_in] = dY . W^T (Eq.8), then col2hash (Algorithm
        // 2) as a gather through field_t.
        float *dcol = (float *)workspace;
        const int Kc = taps * c_in;
        const int64_t no = Lo->n_total;
        const GemmPlan pc = plan_rows(no, Kc, c_out, false, k_gran(dtype));
        const double gbytes = es * ((double)no * c_out + (double)wn) + 4.0 * (double)no * Kc;
        st = launch_gemm<hch::A_ROWS, true>(dtype, pc, dY, W, dcol, nullptr, (int)no, Kc, c_out, c_out, c_out, Kc, 0, gbytes, s);
        if (st != HCH_OK) return st;
        const bool vec = c_in % 4 == 0 && aligned16(dX);
        const int64_t items = n * (vec ? c_in / 4 : c_in);
        if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_sconv_bwd_data: too large");
        // per input voxel: its index row, one piece of dcol per owner (about taps / stride^3), its row out
        const double cbytes = (double)n * (4.0 * taps + 4.0 * c_in + 4.0 * c_in * taps / ((double)stride * stride * stride));
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("field_col2hash_kernel<4>") : HCH_KERNEL_ID("field_col2hash_kernel<1>"), s, cbytes, 0.0);
        if (vec)
            HCH_LAUNCH(hch::field_col2hash_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, s, dcol, field_t, dX, n, taps, c_in);
        else
            HCH_LAUNCH(hch::field_col2hash_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, s, dcol, field_t, dX, n, taps, c_in);
        HCH_LAUNCH_CHECK("field_col2hash_kernel");
        return HCH_OK;
    }
    void *Wt = workspace;
    float *part = (float *)((char *)workspace + w.first_bytes);
    // dX[i] = sum over rows of dY[field_t[i][row]] . W[row]^T: a gathered product over the output
    // gradients through the transposed index rows, weights transposed per tap (not flipped)
    if (dtype == HCH_F32) {
        hch::LaunchTimer lt(HCH_KERNEL_ID("flip_transpose_weights_kernel<float>"), s, 8.0 * wn, 0.0);
        HCH_LAUNCH(hch::flip_transpose_weights_kernel<float>, dim3(blocks_for(wn)), dim3(256), 0, s,
                           (const float *)W, (float *)Wt, c_in, c_out, taps, 0);
    } else {
        hch::LaunchTimer lt(HCH_KERNEL_ID("flip_transpose_weights_kernel<unsigned short>"), s, 4.0 * wn, 0.0);
        HCH_LAUNCH(hch::flip_transpose_weights_kernel<uint16_t>, dim3(blocks_for(wn)), dim3(256), 0, s,
                           (const uint16_t *)W, (uint16_t *)Wt, c_in, c_out, taps, 0);
    }
    HCH_LAUNCH_CHECK("flip_transpose_weights_kernel");
    const GemmPlan p = plan_rows(n, c_in, Kd, true, k_gran(dtype));
    const double bytes = (double)n * (4.0 * taps + 4.0 * c_in * p.splits) + es * (double)Lo->n_total * c_out + es * wn;
    st = launch_gemm<hch::A_GATHER, false>(dtype, p, dY, Wt, p.splits > 1 ? part : dX, field_t, (int)n, c_in, Kd, c_out,
                                           c_in, c_in, n * c_in, bytes, s, 0, taps);
    if (st != HCH_OK) return st;
    if (p.splits > 1) st = launch_reduce(part, dX, n * c_in, p.splits, s);
    return st;
}

// pooling over general receptive fields between level_in and the level `stride` times coarser
static hch_status spool_args(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride, const void *a,
                             const void *b, const void *idx, int32_t c, const Level **Li, const Level **Lo, const char *who)
{
    hch_status st = field_levels(levels, level_in, F, stride, stride == 1 ? (F - 1) / 2 : 0, Li, Lo, who);
    if (st != HCH_OK) return st;
    if (!a || !b || !idx || c <= 0) return fail(HCH_EINVAL, std::string(who) + ": null pointer or non-positive channel count");
    if (std::max((*Li)->n_total, (*Lo)->n_total) * (int64_t)c > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, std::string(who) + ": too large");
    return HCH_OK;
}

extern "C" hch_status hch_spool_max_fwd(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                        const float *X, const int32_t *field, float *Y, int32_t *argmax,
                                        int32_t c, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = spool_args(levels, level_in, F, stride, X, Y, field, c, &Li, &Lo, "hch_spool_max_fwd");
    if (st != HCH_OK) return st;
    if (!argmax) return fail(HCH_EINVAL, "hch_spool_max_fwd: null argmax");
    const int taps = F * F * F;
    const bool vec = c % 4 == 0 && aligned16(X) && aligned16(Y) && aligned16(argmax);
    const int64_t items = Lo->n_total * (vec ? c / 4 : c);
    const double bytes = (double)Lo->n_total * (4.0 * taps + 8.0 * c) + (double)Li->n_total * 4.0 * c;
    hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("field_pool_fwd_kernel<4>") : HCH_KERNEL_ID("field_pool_fwd_kernel<1>"),
                        (hipStream_t)stream, bytes, 0.0);
    if (vec)
        HCH_LAUNCH(hch::field_pool_fwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                           X, field, Y, argmax, Lo->n_total, taps, c);
    else
        HCH_LAUNCH(hch::field_pool_fwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                           X, field, Y, argmax, Lo->n_total, taps, c);
    HCH_LAUNCH_CHECK("field_pool_fwd_kernel");
    return HCH_OK;
}

// backward of pooling where the fields partition the input level (F = stride): through the forward rows
template <bool MAXPOOL>
static hch_status launch_field_unpool(const float *dY, const int32_t *argmax, const int32_t *field, float *dX,
                                      int64_t n_out, int64_t n_in, int taps, int c, hipStream_t s)
{
    const bool vec = c % 4 == 0 && aligned16(dY) && aligned16(dX) && (!MAXPOOL || aligned16(argmax));
    const int64_t items = n_out * taps * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "field pooling backward: too large");
    const double bytes = (double)n_out * (4.0 * taps + (MAXPOOL ? 8.0 : 4.0) * c) + (double)n_in * 4.0 * c;
    const int kid = MAXPOOL ? (vec ? HCH_KERNEL_ID("field_unpool_kernel<4, true>") : HCH_KERNEL_ID("field_unpool_kernel<1, true>"))
                            : (vec ? HCH_KERNEL_ID("field_unpool_kernel<4, false>") : HCH_KERNEL_ID("field_unpool_kernel<1, false>"));
    hch::LaunchTimer lt(kid, s, bytes, 0.0);
    if (vec)
        HCH_LAUNCH((hch::field_unpool_kernel<4, MAXPOOL>), dim3(blocks_for(items)), dim3(256), 0, s,
                           dY, argmax, field, dX, n_out, taps, c, 1.0f / taps);
    else
        HCH_LAUNCH((hch::field_unpool_kernel<1, MAXPOOL>), dim3(blocks_for(items)), dim3(256), 0, s,
                           dY, argmax, field, dX, n_out, taps, c, 1.0f / taps);
    HCH_LAUNCH_CHECK("field_unpool_kernel");
    return HCH_OK;
}

// The fields of a pooling with F = stride > 1 and NO padding partition the input level, and every
// input voxel lies in the field of an occupied output voxel (its parent): only then may the
// backward pass write dX through the forward rows.  With padding an input voxel can fall into the
// field of a position that is not occupied on the output level, and no forward row reaches it.
static inline bool fields_partition(int32_t F, int32_t stride, int32_t pad) { return F == stride && stride > 1 && pad == 0; }

extern "C" hch_status hch_spool_max_bwd(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                        int32_t pad, const float *dY, const int32_t *argmax, const int32_t *field,
                                        const int32_t *field_t, float *dX, int32_t c, void *stream)
{
    const Level *Li, *Lo;
    const bool partition = field && fields_partition(F, stride, pad);
    if (pad < 0 || pad >= F) return fail(HCH_EINVAL, "hch_spool_max_bwd: padding must be in [0, F)");
    if (!partition && !field_t)
        return fail(HCH_EINVAL, "hch_spool_max_bwd: field_t is needed unless F = stride > 1, pad = 0 and field is given");
    hch_status st = spool_args(levels, level_in, F, stride, dY, dX, partition ? field : field_t, c, &Li, &Lo, "hch_spool_max_bwd");
    if (st != HCH_OK) return st;
    if (!argmax) return fail(HCH_EINVAL, "hch_spool_max_bwd: null argmax");
    const int taps = F * F * F;
    if (partition) return launch_field_unpool<true>(dY, argmax, field, dX, Lo->n_total, Li->n_total, taps, c, (hipStream_t)stream);
    const bool vec = c % 4 == 0 && aligned16(dY) && aligned16(dX) && aligned16(argmax);
    const int64_t items = Li->n_total * (vec ? c / 4 : c);
    const double bytes = (double)Li->n_total * (4.0 * taps + 4.0 * c) + (double)Lo->n_total * 8.0 * c;
    hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("field_pool_bwd_kernel<4>") : HCH_KERNEL_ID("field_pool_bwd_kernel<1>"),
                        (hipStream_t)stream, bytes, 0.0);
    if (vec)
        HCH_LAUNCH(hch::field_pool_bwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                           dY, argmax, field_t, dX, Li->n_total, taps, c);
    else
        HCH_LAUNCH(hch::field_pool_bwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                           dY, argmax, field_t, dX, Li->n_total, taps, c);
    HCH_LAUNCH_CHECK("field_pool_bwd_kernel");
    return HCH_OK;
}

static hch_status launch_field_avg(const float *src, const int32_t *idx, float *dst, int64_t n_dst, int64_t n_src,
                                   int taps, int c, hipStream_t s)
{
    const bool vec = c % 4 == 0 && aligned16(src) && aligned16(dst);
    const int64_t items = n_dst * (vec ? c / 4 : c);
    const double bytes = (double)n_dst * (4.0 * taps + 4.0 * c) + (double)n_src * 4.0 * c;
    hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("field_avg_kernel<4>") : HCH_KERNEL_ID("field_avg_kernel<1>"), s, bytes, 0.0);
    if (vec)
        HCH_LAUNCH(hch::field_avg_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, s, src, idx, dst, n_dst, taps, c, 1.0f / taps);
    else
        HCH_LAUNCH(hch::field_avg_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, s, src, idx, dst, n_dst, taps, c, 1.0f / taps);
    HCH_LAUNCH_CHECK("field_avg_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_spool_avg_fwd(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                        const float *X, const int32_t *field, float *Y, int32_t c, void *stream)
{
    const Level *Li, *Lo;
    hch_status st = spool_args(levels, level_in, F, stride, X, Y, field, c, &Li, &Lo, "hch_spool_avg_fwd");
    if (st != HCH_OK) return st;
    return launch_field_avg(X, field, Y, Lo->n_total, Li->n_total, F * F * F, c, (hipStream_t)stream);
}

extern "C" hch_status hch_spool_avg_bwd(const hch_levels *levels, int32_t level_in, int32_t F, int32_t stride,
                                        int32_t pad, const float *dY, const int32_t *field, const int32_t *field_t,
                                        float *dX, int32_t c, void *stream)
{
    const Level *Li, *Lo;
    const bool partition = field && fields_partition(F, stride, pad);
    if (pad < 0 || pad >= F) return fail(HCH_EINVAL, "hch_spool_avg_bwd: padding must be in [0, F)");
    if (!partition && !field_t)
        return fail(HCH_EINVAL, "hch_spool_avg_bwd: field_t is needed unless F = stride > 1, pad = 0 and field is given");
    hch_status st = spool_args(levels, level_in, F, stride, dY, dX, partition ? field : field_t, c, &Li, &Lo, "hch_spool_avg_bwd");
    if (st != HCH_OK) return st;
    if (partition) return launch_field_unpool<false>(dY, nullptr, field, dX, Lo->n_total, Li->n_total, F * F * F, c, (hipStream_t)stream);
    return launch_field_avg(dY, field_t, dX, Li->n_total, Lo->n_total, F * F * F, c, (hipStream_t)stream);
}

extern "C" hch_status hch_avgpool_fwd(const hch_levels *levels, int32_t level_in, const float *X, float *Y,
                                      int32_t c, void *stream)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_avgpool_fwd: level_in must have a coarser level");
    if (!X || !Y || c <= 0) return fail(HCH_EINVAL, "hch_avgpool_fwd: bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    const Level &Lf = levels->lv[level_in];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_avgpool_fwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_avgpool_fwd: levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(X) && aligned16(Y);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_avgpool_fwd: too large");
    {
        const double bytes = (double)Lf.n_total * 4.0 * c + (double)Lc.n_total * (32.0 + 4.0 * c);
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("avgpool_fwd_kernel<4>") : HCH_KERNEL_ID("avgpool_fwd_kernel<1>"),
                            (hipStream_t)stream, bytes, 8.0 * Lc.n_total * c);
        if (vec)
            HCH_LAUNCH(hch::avgpool_fwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               X, Lc.dchild, Y, Lc.n_total, c);
        else
            HCH_LAUNCH(hch::avgpool_fwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               X, Lc.dchild, Y, Lc.n_total, c);
    }
    HCH_LAUNCH_CHECK("avgpool_fwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_avgpool_bwd(const hch_levels *levels, int32_t level_in, const float *dY, float *dX,
                                      int32_t c, void *stream)
{
    if (!levels || level_in < 0 || level_in + 1 >= (int32_t)levels->lv.size())
        return fail(HCH_EINVAL, "hch_avgpool_bwd: level_in must have a coarser level");
    if (!dY || !dX || c <= 0) return fail(HCH_EINVAL, "hch_avgpool_bwd: bad argument");
    const Level &Lc = levels->lv[level_in + 1];
    const Level &Lf = levels->lv[level_in];
    if (Lc.ratio != 2) return fail(HCH_EUNSUPPORTED, "hch_avgpool_bwd: these two levels are not in ratio 2; use hch_field_build with hch_spool_* / hch_sconv_*");
    if (!Lc.dchild) return fail(HCH_EINVAL, "hch_avgpool_bwd: levels were built without device tables");
    const bool vec = c % 4 == 0 && aligned16(dY) && aligned16(dX);
    const int64_t items = Lc.n_total * (vec ? c / 4 : c);
    if (items > MAX_GRID_ITEMS) return fail(HCH_EUNSUPPORTED, "hch_avgpool_bwd: too large");
    {
        const double bytes = (double)Lf.n_total * 4.0 * c + (double)Lc.n_total * (32.0 + 4.0 * c);
        hch::LaunchTimer lt(vec ? HCH_KERNEL_ID("avgpool_bwd_kernel<4>") : HCH_KERNEL_ID("avgpool_bwd_kernel<1>"),
                            (hipStream_t)stream, bytes, 0.0);
        if (vec)
            HCH_LAUNCH(hch::avgpool_bwd_kernel<4>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               dY, Lc.dchild, dX, Lc.n_total, c);
        else
            HCH_LAUNCH(hch::avgpool_bwd_kernel<1>, dim3(blocks_for(items)), dim3(256), 0, (hipStream_t)stream,
                               dY, Lc.dchild, dX, Lc.n_total, c);
    }
    HCH_LAUNCH_CHECK("avgpool_bwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_relu_fwd(const float *x, float *y, int64_t n, void *stream)
{
    if (!x || !y || n < 0) return fail(HCH_EINVAL, "hch_relu_fwd: bad argument");
    if (n == 0) return HCH_OK;
    {
        hch::LaunchTimer lt(HCH_KERNEL_ID("relu_fwd_kernel"), (hipStream_t)stream, 8.0 * n, 0.0);
        const int64_t n4 = (aligned16(x) && aligned16(y)) ? n / 4 : 0;
        HCH_LAUNCH(hch::relu_fwd_kernel, dim3(blocks_for(std::max(n4, n - 4 * n4))), dim3(256), 0,
                           (hipStream_t)stream, x, y, n, n4);
    }
    HCH_LAUNCH_CHECK("relu_fwd_kernel");
    return HCH_OK;
}

extern "C" hch_status hch_relu_bwd(const float *y, const float *dy, float *dx, int64_t n, void *stream)
{
    if (!y || !dy || !dx || n < 0) return fail(HCH_EINVAL, "hch_relu_bwd: bad argument");
    if (n == 0) return HCH_OK;
    {
        hch::LaunchTimer lt(HCH_KERNEL_ID("relu_bwd_kernel"), (hipStream_t)stream, 12.0 * n, 0.0);
        const int64_t n4 = (aligned16(y) && aligned16(dy) && aligned16(dx)) ? n / 4 : 0;
        HCH_LAUNCH(hch::relu_bwd_kernel, dim3(blocks_for(std::max(n4, n - 4 * n4))), dim3(256), 0,
                           (hipStream_t)stream, y, dy, dx, n, n4);
    }
    HCH_LAUNCH_CHECK("relu_bwd_kernel");
    return HCH_OK;
}

// ---------------------------------------------------------------------------------------
// per-kernel timing
// ---------------------------------------------------------------------------------------

extern "C" int32_t hch_set_lean_loops(int32_t enabled)
{
    return g_lean_loops.exchange(enabled ? 1 : 0);
}

extern "C" hch_status hch_probe_mfma(hch_dtype dtype, int32_t iters, int32_t workgroups, float *sink, void *stream)
{
    if (!sink || iters <= 0 || workgroups <= 0 || (dtype != HCH_F32 && dtype != HCH_BF16))
        return fail(HCH_EINVAL, "hch_probe_mfma: bad argument");
    hipStream_t s = (hipStream_t)stream;
    const double waves = 4.0 * workgroups, per = dtype == HCH_BF16 ? 16384.0 : 2048.0;
    hch::LaunchTimer lt(dtype == HCH_BF16 ? HCH_KERNEL_ID("mfma_probe_kernel<true>") : HCH_KERNEL_ID("mfma_probe_kernel<false>"),
                        s, 0.0, waves * iters * 8.0 * per);
    if (dtype == HCH_BF16) HCH_LAUNCH(hch::mfma_probe_kernel<true>, dim3((unsigned)workgroups), dim3(256), 0, s, sink, iters);
    else HCH_LAUNCH(hch::mfma_probe_kernel<false>, dim3((unsigned)workgroups), dim3(256), 0, s, sink, iters);
    HCH_LAUNCH_CHECK("mfma_probe_kernel");
    return HCH_OK;
}

extern "C" int32_t hch_kernel_count(void) { return hch::Profiler::get().count(); }

extern "C" const char *hch_kernel_name(int32_t id)
{
    thread_local std::string buf;
    buf = hch::Profiler::get().name(id);
    return buf.c_str();
}

extern "C" hch_status hch_profile_enable(int32_t kernel_id, int32_t on)
{
    if (kernel_id >= hch::Profiler::get().count()) return fail(HCH_EINVAL, "hch_profile_enable: unknown kernel id");
    hch::Profiler::get().enable(kernel_id, on != 0);
    return HCH_OK;
}

extern "C" hch_status hch_profile_read(int32_t kernel_id, hch_kernel_stats *out)
{
    if (!out || kernel_id < 0 || kernel_id >= hch::Profiler::get().count())
        return fail(HCH_EINVAL, "hch_profile_read: bad argument");
    hch::Profiler::get().collect();
    const hch::KernelStats st = hch::Profiler::get().read(kernel_id);
    out->launches = st.launches; out->ms = st.ms; out->bytes = st.bytes; out->flops = st.flops;
    return HCH_OK;
}

extern "C" hch_status hch_profile_reset(void)
{
    hch::Profiler::get().collect();
    hch::Profiler::get().reset();
    return HCH_OK;
}
