// libmfs host side: argument checking, plans, the preconditioned operator
// and GMRES drivers.  Every arithmetic step of the solve runs in the HIP
// kernels of this library; this file only plans and sequences them.
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <numeric>

#include "mfs_internal.h"

namespace mfs {

// kernels declared here to keep the internal header short
int launch_make_factor(int rows, int cols, const double *src, int64_t ld, bool transposed, const double *rs,
                       const double *cs, double *d64, float *d32, hipStream_t s);

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string g_last_error;

void set_error(const std::string &msg) { g_last_error = msg; }

int fail(int status, const std::string &msg) {
    g_last_error = msg;
    return status;
}

int DevBuf::reserve(size_t n) {
    if (n <= bytes && ptr) return MFS_OK;
    release();
    if (n == 0) return MFS_OK;
    hipError_t e = hipMalloc(&ptr, n);
    if (e != hipSuccess) {
        ptr = nullptr;
        return fail(e == hipErrorOutOfMemory ? MFS_ENOMEM : MFS_EHIP,
                    std::string("hipMalloc(") + std::to_string(n) + "): " + hipGetErrorString(e));
    }
    bytes = n;
    return MFS_OK;
}

int DevBuf::upload(const void *host, size_t n, hipStream_t s) {
    MFS_TRY(reserve(n));
    if (n) MFS_HIP_TRY(hipMemcpyAsync(ptr, host, n, hipMemcpyHostToDevice, s));
    return MFS_OK;
}

template <class T>
static int upload_vec(DevBuf &b, const std::vector<T> &v, hipStream_t s) {
    return b.upload(v.data(), v.size() * sizeof(T), s);
}

// ---------------------------------------------------------------------------
// pair-sum work items
// ---------------------------------------------------------------------------
// Targets of one item: 64 lanes x tpl, the waves sharing the sources; 64 per wave for the Laplace
// items of a launch with far tiles (laplace_far_item).
int64_t item_targets(int kind, int tpl, bool far) { return far && kind == MFS_LAPLACE ? 256 : 64 * tpl; }

// Shape of a pair-sum launch: bodies per source chunk (the largest chunk, so the
// fewest split slices, that still gives at least min_items items), the number of
// split slices and the number of items.
void p2p_item_count(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                    const int32_t *kind_of_body, int kind_all, int tpl, bool far, int min_items, int64_t *chunk_out,
                    int *n_split_out, int64_t *n_items_out) {
    auto blocks = [&](int64_t sy) {  // target blocks of a system
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        if (b1 == b0) return int64_t(0);
        const int64_t blk = item_targets(kind_of_body ? kind_of_body[b0] : kind_all, tpl, far);
        return (body_trg_ptr[b1] - body_trg_ptr[b0] + blk - 1) / blk;
    };
    auto count_items = [&](int64_t chunk) {
        int64_t n = 0;
        for (int64_t sy = 0; sy < n_sys; ++sy)
            n += blocks(sy) * ((sys_body_ptr[sy + 1] - sys_body_ptr[sy] + chunk - 1) / chunk);
        return n;
    };
    int64_t max_bodies = 1;
    for (int64_t sy = 0; sy < n_sys; ++sy) max_bodies = std::max(max_bodies, sys_body_ptr[sy + 1] - sys_body_ptr[sy]);
    int64_t chunk = max_bodies;
    while (chunk > 1 && count_items(chunk) < min_items) chunk = (chunk + 1) / 2;
    int n_split = 1;
    for (int64_t sy = 0; sy < n_sys; ++sy)
        n_split = std::max(n_split, (int)((sys_body_ptr[sy + 1] - sys_body_ptr[sy] + chunk - 1) / chunk));
    // every system writes all n_split slices
    int64_t n = 0;
    for (int64_t sy = 0; sy < n_sys; ++sy) n += blocks(sy) * n_split;
    *chunk_out = chunk;
    *n_split_out = n_split;
    *n_items_out = n;
}

int generate_p2p_items(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                       const int64_t *body_src_ptr, const int64_t *out_ptr, int out_dim,
                       const int32_t *kind_of_body, int kind_all, double mu, int tpl, int min_items, P2PItem *items,
                       double *work, int32_t *order, P2PItem *sorted, int64_t cap, int64_t *n_items, int *n_split_out,
                       bool far) {
    int64_t chunk = 1, n = 0;
    int n_split = 1;
    p2p_item_count(n_sys, sys_body_ptr, body_trg_ptr, kind_of_body, kind_all, tpl, far, min_items, &chunk, &n_split,
                   &n);

    if (n > cap) return fail(MFS_EINVAL, "pair sum needs " + std::to_string(n) + " work items, more than " +
                                             std::to_string(cap));
    n = 0;
    for (int64_t sy = 0; sy < n_sys; ++sy) {
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        if (b1 == b0) continue;
        const int64_t T0 = body_trg_ptr[b0], T1 = body_trg_ptr[b1];
        const int kind = kind_of_body ? kind_of_body[b0] : kind_all;
        const double scale = kind == MFS_STOKES ? 1.0 / (8.0 * PI * mu) : 1.0 / (4.0 * PI);
        const int dim = kind == MFS_STOKES ? 3 : 1;
        const int64_t blk = item_targets(kind, tpl, far);
        const int64_t base = out_ptr ? out_ptr[b0] : (int64_t)out_dim * body_trg_ptr[b0];
        for (int64_t t0 = T0; t0 < T1; t0 += blk) {
            const int64_t t1 = std::min(t0 + blk, T1);
            // every system writes all n_split slices (splits past its last body get an
            // empty body range and write zeros), so the slice reduction reads no stale data
            for (int sp = 0; sp < n_split; ++sp) {
                const int64_t c0 = std::min(b1, b0 + (int64_t)sp * chunk), c1 = std::min(b1, c0 + chunk);
                P2PItem it{};
                it.out0 = base + dim * (t0 - T0);
                it.scale = scale;
                it.t0 = (int32_t)t0;
                it.t1 = (int32_t)t1;
                it.b0 = (int32_t)c0;
                it.b1 = (int32_t)c1;
                it.sys = (int32_t)sy;
                it.split = sp;
                it.kind = kind;
                const double nsrc = (double)(body_src_ptr[c1] - body_src_ptr[c0]);
                items[n] = it;
                work[n] = nsrc * (double)(t1 - t0) * (kind == MFS_STOKES ? 2.5 : 1.0);
                ++n;
            }
        }
    }
    *n_items = n;
    *n_split_out = n_split;
    // largest work first (ties in generation order), so the dispatcher schedules greedily.  Most launches
    // have a handful of amounts of work (whole and cut blocks and chunks of each system), so the items are
    // counted by amount: 45000 items of 300 bodies 0.4 ms, 2.3 ms sorted
    constexpr int kAmounts = 256;
    double amount[kAmounts];
    int64_t at[kAmounts] = {};
    int n_amount = 0;
    bool few = true;
    for (int64_t i = 0; i < n && few; ++i) {
        int k = i > 0 && work[i] == work[i - 1] ? order[i - 1] : n_amount - 1;
        while (k >= 0 && amount[k] != work[i]) --k;
        if (k < 0) {
            few = n_amount < kAmounts;
            if (!few) break;
            k = n_amount++;
            amount[k] = work[i];
        }
        order[i] = k;
        ++at[k];
    }
    if (few) {
        int rank[kAmounts];
        std::iota(rank, rank + n_amount, 0);
        std::sort(rank, rank + n_amount, [&](int a, int b) { return amount[a] > amount[b]; });
        int64_t next = 0;
        for (int r = 0; r < n_amount; ++r) {
            const int64_t count = at[rank[r]];
            at[rank[r]] = next;
            next += count;
        }
        for (int64_t i = 0; i < n; ++i) sorted[at[order[i]]++] = items[i];
        return MFS_OK;
    }
    std::iota(order, order + n, 0);
    std::sort(order, order + n, [&](int32_t a, int32_t b) { return work[a] > work[b] || (work[a] == work[b] && a < b); });
    for (int64_t i = 0; i < n; ++i) sorted[i] = items[order[i]];
    return MFS_OK;
}

// The least number of work items of a pair-sum launch that takes us microseconds.  A launch holds
// about 2048 workgroups at a time, so with n items the last round idles about 2048 / 2n of the chip's
// time T, and an item costs about 8 us of a workgroup's beside its pairs (set-up, the sum over
// its waves, its part of the slice sums); the sum of both is least at n = 2048 sqrt(T / 16 us).
// Measured (matvec, us, at 2048 / 4096 / 8192 / 16384 / 32768 items): 50 bodies (T = 0.16 ms)
// 206 / 197 / 203 / 214 / 212, 80 bodies (0.4 ms) 471 / 452 / 443 / 449 / 481, 400 bodies
// (18 ms) 18700 / 18760 / 17830 / 17220 / 17020.
int min_items_for(double us, int most) {
    return (int)std::min((double)most, std::max(2048.0, 2048.0 * std::sqrt(us / 16.0)));
}

// Plans: T from 2.8e12 Stokes or twice as many Laplace pairs per second, and of the largest system
// alone: the items of a batch differ in size and are handed out largest first, so the small systems
// fill the last round (12 systems of 17 to 62 bodies: 529 us at 5500 items, 565 at 10000).
int default_min_items(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                      const int64_t *body_src_ptr, const int32_t *kind_of_body, int kind_all, int most) {
    double us = 0.0;
    for (int64_t sy = 0; sy < n_sys; ++sy) {
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        if (b1 == b0) continue;
        const int kind = kind_of_body ? kind_of_body[b0] : kind_all;
        us = std::max(us, (double)(body_trg_ptr[b1] - body_trg_ptr[b0]) * (double)(body_src_ptr[b1] - body_src_ptr[b0]) /
                              (kind == MFS_STOKES ? 2.8e6 : 5.6e6));
    }
    return min_items_for(us, most);
}

// Standalone calls: the same for one system (also in FP64, where twice as many items are up to 3%
// slower: 60 bodies of 331 x 667 607 us, 622).  A batch takes T of all its systems, with the rates of
// FP64 sums (1.3e12 and 2.3e12) unless it is a mixed sum (fields and gradients share their tables
// between the precisions), and half the T for mixed sums.  With T of the largest system batches took
// too few, us: 11 Stokes systems of 25 to 94 bodies of 160 x 367 1045, now 974, in FP64 2246 and 1968;
// 12 of 8 to 31 bodies of 300 x 600 in FP64 854 and 777; and with the whole T of mixed sums too many:
// 8 Laplace systems of 12 to 45 bodies of 400 x 800 317, now 297.  Launches with far tiles keep the
// plans' rule: their items are few and long, and cutting one large system in a batch gives every small
// one as many empty items (32 bodies beside 500 systems of two: 187 us, 326 with this rule).
int standalone_min_items(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                         const int64_t *body_src_ptr, int kind, bool mixed, bool far, int most) {
    double pairs = 0.0;
    int systems = 0;
    for (int64_t sy = 0; sy < n_sys; ++sy) {
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        pairs += (double)(body_trg_ptr[b1] - body_trg_ptr[b0]) * (double)(body_src_ptr[b1] - body_src_ptr[b0]);
        systems += b1 > b0;
    }
    if (far || systems <= 1)
        return default_min_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nullptr, kind, most);
    const bool stokes = kind == MFS_STOKES;
    return min_items_for(mixed ? pairs / (stokes ? 5.6e6 : 11.2e6) : pairs / (stokes ? 1.3e6 : 2.3e6), most);
}

// Whether the sums of this orientation use far tiles: Laplace bodies only (beside them the Stokes
// items of a launch would run with the far walk's registers, 4 waves per SIMD: 585 us instead of
// 532 for a batch of both), a system of at least 32 bodies (below, most are near some of an item's
// targets: 28 of 389 x 777 take 52.2 us with far tiles, 53.7 without, 36 73.9 and 82.5) and 2.5e8 pairs
// (below, 256 targets to an item leave the chip too few: 48 bodies of 200 x 400, 1.8e8 pairs, 48.0 us
// and 45.7; 56, 2.5e8, 58.1 and 59.3; 120 of 100 x 200, 2.9e8, 70.0 and 70.2), whole tiles but for a
// quarter, and bodies of at most 1024 sources (their strengths stay in LDS, 4 KB a wave).
bool use_far_tiles(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                   const int64_t *body_src_ptr, const int32_t *kind_of_body, std::vector<int32_t> &tile_ptr) {
    int64_t most = 0, sources = 0, tiles = 0;
    double pairs = 0.0;
    tile_ptr.assign(std::max<int64_t>(1, sys_body_ptr[n_sys]), 0);
    for (int64_t sy = 0; sy < n_sys; ++sy) {
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        if (b1 == b0) continue;
        if (kind_of_body && kind_of_body[b0] != MFS_LAPLACE) return false;
        most = std::max(most, b1 - b0);
        pairs += (double)(body_trg_ptr[b1] - body_trg_ptr[b0]) * (double)(body_src_ptr[b1] - body_src_ptr[b0]);
        for (int64_t b = b0; b < b1; ++b) {
            const int64_t n = body_src_ptr[b + 1] - body_src_ptr[b];
            if (n > 1024) return false;  // far_body holds that many strengths
            tile_ptr[b] = (int32_t)tiles;
            sources += n;
            tiles += (n + 15) / 16;
            if (tiles > INT32_MAX / 2) return false;
        }
    }
    tile_ptr.push_back((int32_t)tiles);  // the total
    return most >= 32 && pairs >= 2.5e8 && 16.0 * (double)tiles <= 1.25 * (double)sources;
}

// Whether a standalone mixed sum takes wide items (p2p_wide_kernel: 16 waves on 64 targets and every
// source of their system, one launch): when that many workgroups fit the chip at once and the longest
// of them, S sources on one CU (its waves share the LDS that they read the sources from: 7.7 ns a
// Stokes source, 3.5 Laplace), takes no more than the sum on all CUs plus the launches saved.  Both
// sides, us: Stokes 4 bodies of 300 x 600 19.1 general, 13.7 wide; 6 of 400 x 800 18.3, 20.9; 10 of
// 300 x 600 18.4, 25.7; Laplace 20 of 400 x 800 35.2, 31.5; 6 of 200 x 400 in 6 systems 18.1, 13.3.
bool use_wide_items(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                    const int64_t *body_src_ptr, int kind) {
    constexpr double saved_us = 11.0;
    const bool stokes = kind == MFS_STOKES;
    int64_t blocks = 0;
    double longest = 0.0, all = 0.0;  // us
    for (int64_t sy = 0; sy < n_sys; ++sy) {
        const int64_t b0 = sys_body_ptr[sy], b1 = sys_body_ptr[sy + 1];
        const int64_t nt = body_trg_ptr[b1] - body_trg_ptr[b0], ns = body_src_ptr[b1] - body_src_ptr[b0];
        if (nt == 0) continue;
        blocks += (nt + 63) / 64;
        longest = std::max(longest, (double)ns * (stokes ? 7.7e-3 : 3.5e-3));
        all += (double)nt * (double)ns / (stokes ? 2.9e6 : 5.7e6);
    }
    return blocks <= 256 && longest <= all + saved_us;
}

int build_p2p_items(P2PPlan &pp, int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                    const int64_t *body_src_ptr, const int64_t *out_ptr, const int32_t *kind_of_body, double mu,
                    int tpl, int min_items, hipStream_t s, bool far) {
    pp.tpl = tpl;
    pp.far = far;
    int64_t chunk = 1, cap = 0;
    int n_split = 1;
    p2p_item_count(n_sys, sys_body_ptr, body_trg_ptr, kind_of_body, 0, tpl, far, min_items, &chunk, &n_split, &cap);
    std::vector<P2PItem> tmp(std::max<int64_t>(1, cap));
    std::vector<double> work(std::max<int64_t>(1, cap));
    std::vector<int32_t> order(std::max<int64_t>(1, cap));
    pp.items.assign(std::max<int64_t>(1, cap), P2PItem{});
    int64_t n = 0;
    MFS_TRY(generate_p2p_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, out_ptr, 1, kind_of_body, 0, mu, tpl,
                               min_items, tmp.data(), work.data(), order.data(), pp.items.data(), cap, &n,
                               &pp.n_split, far));
    pp.items.resize(n);
    if (!pp.items.empty()) MFS_TRY(upload_vec(pp.d_items, pp.items, s));
    MFS_TRY(pp.d_counter.reserve(sizeof(int)));
    return MFS_OK;
}

// The same items once more (one workgroup per item), without making them again.
static int copy_p2p_items(P2PPlan &to, const P2PPlan &from, hipStream_t s) {
    to.items = from.items;
    to.n_split = from.n_split;
    to.tpl = from.tpl;
    to.far = from.far;
    to.wide = from.wide;
    const size_t bytes = from.items.size() * sizeof(P2PItem);
    if (bytes) {
        MFS_TRY(to.d_items.reserve(bytes));
        MFS_HIP_TRY(hipMemcpyAsync(to.d_items.ptr, from.d_items.ptr, bytes, hipMemcpyDeviceToDevice, s));
    }
    return to.d_counter.reserve(sizeof(int));
}

}  // namespace mfs

using namespace mfs;

// ---------------------------------------------------------------------------
// library-owned workspace for the standalone entry points
// ---------------------------------------------------------------------------
namespace {

// The structure-dependent part of a standalone call: device copies of the body
// pointers, per-point body ids and the pair-sum work items.  Built on the first
// call with a given structure and reused by later calls with the same one.
struct Layout {
    int variant = 0;  // which entry point family and kernel (see layout())
    uint64_t mu_bits = 0;
    std::vector<int64_t> sys, trg, src;  // host copies of the structure arrays (the cache key)
    std::vector<int32_t> trg32, src32, tiles_h;
    DevBuf trg_ptr, src_ptr, trg_body, src_body;
    P2PPlan pp;
    bool mixed = false, far = false;  // a mixed pair sum; far tiles used
    int64_t n_tiles = 0;
    DevBuf tile_ptr;
    uint64_t last_use = 0;
};

// launch shape of the standalone pair sums: one target per lane, standalone_min_items up to this
// many (the allocation-free call holds the items and slices of that many)
constexpr int kStandaloneMinItems = 16384;
// and of the plans' pair sums until they are tuned or set
constexpr int kPlanMinItems = 65536;

struct Workspace {
    DevBuf centre, trg_off, src_ops, partial, far_tiles, far_centre, far_rho;
    std::vector<std::unique_ptr<Layout>> layouts;
    uint64_t clock = 0;
};
constexpr size_t kMaxLayouts = 16;  // 8 structures, each with mixed pair sums and with everything else

// one workspace per host thread and device
Workspace &workspace() {
    static thread_local std::vector<std::unique_ptr<Workspace>> per_device;
    int dev = 0;
    (void)hipGetDevice(&dev);
    if ((int)per_device.size() <= dev) per_device.resize(dev + 1);
    if (!per_device[dev]) per_device[dev] = std::make_unique<Workspace>();
    return *per_device[dev];
}

// Standalone calls are asynchronous, so a workspace buffer may still be read by
// work enqueued earlier: wait for the device before a buffer is replaced.
int grow(DevBuf &b, size_t n) {
    if (n <= b.bytes && b.ptr) return MFS_OK;
    if (b.ptr) MFS_HIP_TRY(hipDeviceSynchronize());
    return b.reserve(n);
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

int check_structure(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                    const int64_t *body_src_ptr, int64_t *n_body, int64_t *n_trg, int64_t *n_src) {
    if (n_sys < 1) return fail(MFS_EINVAL, "n_sys must be >= 1");
    if (!sys_body_ptr || !body_trg_ptr || !body_src_ptr) return fail(MFS_EINVAL, "NULL structure array");
    if (sys_body_ptr[0] != 0) return fail(MFS_EINVAL, "sys_body_ptr[0] must be 0");
    for (int64_t s = 0; s < n_sys; ++s)
        if (sys_body_ptr[s + 1] < sys_body_ptr[s]) return fail(MFS_EINVAL, "sys_body_ptr not non-decreasing");
    const int64_t nb = sys_body_ptr[n_sys];
    if (body_trg_ptr[0] != 0 || body_src_ptr[0] != 0) return fail(MFS_EINVAL, "body pointers must start at 0");
    for (int64_t b = 0; b < nb; ++b)
        if (body_trg_ptr[b + 1] < body_trg_ptr[b] || body_src_ptr[b + 1] < body_src_ptr[b])
            return fail(MFS_EINVAL, "body pointers not non-decreasing");
    if (body_trg_ptr[nb] > INT32_MAX || body_src_ptr[nb] > INT32_MAX)
        return fail(MFS_EINVAL, "point counts must fit in int32");
    *n_body = nb;
    *n_trg = body_trg_ptr[nb];
    *n_src = body_src_ptr[nb];
    return MFS_OK;
}

int check_prec(int prec) {
    if (prec != MFS_MIXED && prec != MFS_FP64) return fail(MFS_EINVAL, "unknown precision");
    return MFS_OK;
}

// The cached layout of (variant, mu, structure), built if missing.  kind sets
// the items' kernel and scale; dim the output values per target of the items.
// mixed: a mixed pair sum that can take far tiles or wide items.
int layout(Workspace &ws, int variant, int kind, int dim, double mu, int64_t n_sys, const int64_t *sys_body_ptr,
           const int64_t *body_trg_ptr, const int64_t *body_src_ptr, int64_t nb, hipStream_t s, Layout **out,
           bool mixed = false) {
    uint64_t bits;
    std::memcpy(&bits, &mu, sizeof bits);
    auto same = [&](const Layout &l) {
        return l.variant == variant && l.mixed == mixed && l.mu_bits == bits && (int64_t)l.sys.size() == n_sys + 1 &&
               (int64_t)l.trg.size() == nb + 1 && (int64_t)l.src.size() == nb + 1 &&
               std::equal(l.sys.begin(), l.sys.end(), sys_body_ptr) &&
               std::equal(l.trg.begin(), l.trg.end(), body_trg_ptr) &&
               std::equal(l.src.begin(), l.src.end(), body_src_ptr);
    };
    for (auto &l : ws.layouts)
        if (same(*l)) {
            l->last_use = ++ws.clock;
            *out = l.get();
            return MFS_OK;
        }
    if (ws.layouts.size() >= kMaxLayouts) {
        // the evicted layout's items may still be read by enqueued work
        MFS_HIP_TRY(hipDeviceSynchronize());
        auto lru = std::min_element(ws.layouts.begin(), ws.layouts.end(),
                                    [](const std::unique_ptr<Layout> &a, const std::unique_ptr<Layout> &b) {
                                        return a->last_use < b->last_use;
                                    });
        ws.layouts.erase(lru);
    }
    auto l = std::make_unique<Layout>();
    l->variant = variant;
    l->mixed = mixed;
    l->mu_bits = bits;
    l->sys.assign(sys_body_ptr, sys_body_ptr + n_sys + 1);
    l->trg.assign(body_trg_ptr, body_trg_ptr + nb + 1);
    l->src.assign(body_src_ptr, body_src_ptr + nb + 1);
    l->trg32.assign(body_trg_ptr, body_trg_ptr + nb + 1);
    l->src32.assign(body_src_ptr, body_src_ptr + nb + 1);
    MFS_TRY(upload_vec(l->trg_ptr, l->trg32, s));
    MFS_TRY(upload_vec(l->src_ptr, l->src32, s));
    MFS_TRY(l->trg_body.reserve(std::max<int64_t>(1, body_trg_ptr[nb]) * sizeof(int32_t)));
    MFS_TRY(l->src_body.reserve(std::max<int64_t>(1, body_src_ptr[nb]) * sizeof(int32_t)));
    MFS_TRY(launch_fill_body_ids(nb, l->trg_ptr.as<int32_t>(), l->trg_body.as<int32_t>(), s));
    MFS_TRY(launch_fill_body_ids(nb, l->src_ptr.as<int32_t>(), l->src_body.as<int32_t>(), s));
    std::vector<int64_t> out_ptr(nb + 1);
    for (int64_t b = 0; b <= nb; ++b) out_ptr[b] = dim * body_trg_ptr[b];
    std::vector<int32_t> kob(std::max<int64_t>(1, nb), kind);
    // One walk or the other: their items differ (64 and 256 targets).  Where both rules hold, the two take the
    // same time (us, wide and far: 32 bodies of 500 x 512 58 and 56, 199 of 84 x 82 72 and 73, 2 x 40 of
    // 400 x 204 55 and 59; without either 72, 114, 75), so the one that needs no operands is taken.
    const bool wide = variant == kind && mixed && use_wide_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, kind);
    std::vector<int32_t> tiles;
    l->far = !wide && mixed && kind == MFS_LAPLACE &&
             use_far_tiles(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nullptr, tiles);
    if (l->far) {
        l->tiles_h.swap(tiles);
        l->n_tiles = l->tiles_h.back();
        MFS_TRY(upload_vec(l->tile_ptr, l->tiles_h, s));
    }
    const int min_items = wide ? 1
                               : standalone_min_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, kind, mixed,
                                                      l->far, kStandaloneMinItems);
    MFS_TRY(build_p2p_items(l->pp, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, out_ptr.data(), kob.data(), mu, 1,
                            min_items, s, l->far));
    l->pp.wide = wide;
    l->last_use = ++ws.clock;
    *out = l.get();
    ws.layouts.push_back(std::move(l));
    return MFS_OK;
}

// Per call: the body reference points (the first proxy of each body), the
// targets' offsets from them and the source records with their strengths.
int standalone_operands(Workspace &ws, const Layout &lay, int kind, int64_t n_body, int64_t n_trg, int64_t n_src,
                        const double *trg_xyz, const double *src_xyz, const double *str, int prec, hipStream_t s,
                        P2PLaunch &L) {
    MFS_TRY(grow(ws.centre, std::max<int64_t>(1, n_body) * 3 * sizeof(double)));
    MFS_TRY(grow(ws.trg_off, std::max<int64_t>(1, n_trg) * (prec == MFS_MIXED ? 16 : 32)));
    const size_t rec = kind == MFS_STOKES ? (prec == MFS_MIXED ? sizeof(SrcS32) : sizeof(SrcS64))
                                          : (prec == MFS_MIXED ? sizeof(SrcL32) : sizeof(SrcL64));
    MFS_TRY(grow(ws.src_ops, std::max<int64_t>(1, n_src) * rec));
    StandaloneOperands o;
    o.n_body = n_body;
    o.n_trg = n_trg;
    o.n_src = n_src;
    o.trg_ptr = lay.trg_ptr.as<int32_t>();
    o.src_ptr = lay.src_ptr.as<int32_t>();
    o.trg_body = lay.trg_body.as<int32_t>();
    o.src_body = lay.src_body.as<int32_t>();
    o.trg_xyz = trg_xyz;
    o.src_xyz = src_xyz;
    o.str = str;
    o.centre = ws.centre.as<double>();
    o.trg_off = ws.trg_off.ptr;
    o.src_ops = ws.src_ops.ptr;
    MFS_TRY(launch_operands(o, kind, prec, s));
    if (lay.far) {
        MFS_TRY(grow(ws.far_tiles, std::max<int64_t>(1, lay.n_tiles) * 1024));
        MFS_TRY(grow(ws.far_centre, std::max<int64_t>(1, n_body) * 3 * sizeof(double)));
        MFS_TRY(grow(ws.far_rho, std::max<int64_t>(1, n_body) * sizeof(float)));
        L.far.tiles = ws.far_tiles.ptr;
        L.far.tile_ptr = lay.tile_ptr.as<int32_t>();
        L.far.centre = ws.far_centre.as<double>();
        L.far.rho = ws.far_rho.as<float>();
        MFS_TRY(launch_far_pack(n_body, o.src_ptr, src_xyz, 3, nullptr, L.far, s));
    }
    L.prec = prec;
    L.centre = ws.centre.as<double>();
    L.trg_body = lay.trg_body.as<int32_t>();
    L.src_ptr = lay.src_ptr.as<int32_t>();
    L.trg_off = ws.trg_off.ptr;
    (kind == MFS_STOKES ? L.srcS : L.srcL) = ws.src_ops.ptr;
    return MFS_OK;
}

int standalone_partial(Workspace &ws, const Layout &lay, P2PLaunch &L) {
    if (lay.pp.n_split > 1) {
        MFS_TRY(grow(ws.partial, (size_t)lay.pp.n_split * L.n_val * sizeof(double)));
        L.partial = ws.partial.as<double>();
    }
    return MFS_OK;
}

// Whether the output shares memory with an input, which wide items would read while it is written.
bool overlaps_inputs(const double *out, int64_t n_out, const double *trg, const double *src, const double *str,
                     int64_t n_trg, int64_t n_src, int dim) {
    auto meets = [&](const double *p, int64_t n) {
        const std::less<const double *> before;
        return n > 0 && n_out > 0 && before(p, out + n_out) && before(out, p + n);
    };
    return meets(trg, 3 * n_trg) || meets(src, 3 * n_src) || meets(str, dim * n_src);
}

int p2p_standalone(int kind, int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                   const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz, const double *str,
                   double *out, double mu, int flags, int prec, void *stream) {
    int64_t nb, nt, ns;
    MFS_TRY(check_structure(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, &nb, &nt, &ns));
    MFS_TRY(check_prec(prec));
    if (flags & ~(MFS_SKIP_SAME_BODY | MFS_ACCUMULATE)) return fail(MFS_EINVAL, "unknown flags");
    if (kind == MFS_STOKES && !finite_pos(mu)) return fail(MFS_EINVAL, "mu must be finite and > 0");
    if ((nt > 0 && (!trg_xyz || !out)) || (ns > 0 && (!src_xyz || !str)))
        return fail(MFS_EINVAL, "NULL data pointer");
    if (nt == 0) return MFS_OK;
    hipStream_t s = (hipStream_t)stream;
    Workspace &ws = workspace();
    const int dim = kind == MFS_STOKES ? 3 : 1;
    Layout *lay = nullptr;
    MFS_TRY(layout(ws, kind, kind, dim, mu, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nb, s, &lay,
                   prec == MFS_MIXED && !overlaps_inputs(out, dim * nt, trg_xyz, src_xyz, str, nt, ns, dim)));
    P2PLaunch L;
    if (lay->pp.wide) {
        L.prec = prec;
        L.trg_body = lay->trg_body.as<int32_t>();
        L.src_ptr = lay->src_ptr.as<int32_t>();
        L.raw_trg = trg_xyz;
        L.raw_src = src_xyz;
        L.raw_str = str;
    } else {
        MFS_TRY(standalone_operands(ws, *lay, kind, nb, nt, ns, trg_xyz, src_xyz, str, prec, s, L));
    }
    L.skip_same = (flags & MFS_SKIP_SAME_BODY) != 0;
    L.accumulate = (flags & MFS_ACCUMULATE) != 0;
    L.out = out;
    L.n_val = dim * nt;
    MFS_TRY(standalone_partial(ws, *lay, L));
    return launch_p2p(lay->pp, L, s);
}

// Derived fields (pressure, traction, Laplace gradient) of standalone inputs.
int field_standalone(int field, int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                     const int64_t *body_src_ptr, const double *trg_xyz, const double *trg_normal,
                     const double *src_xyz, const double *str, double *out, int flags, int prec, void *stream) {
    int64_t nb, nt, ns;
    MFS_TRY(check_structure(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, &nb, &nt, &ns));
    MFS_TRY(check_prec(prec));
    if (flags & ~(MFS_SKIP_SAME_BODY | MFS_ACCUMULATE)) return fail(MFS_EINVAL, "unknown flags");
    if ((nt > 0 && (!trg_xyz || !out)) || (ns > 0 && (!src_xyz || !str)))
        return fail(MFS_EINVAL, "NULL data pointer");
    if (field == MFS_FIELD_TRACTION && nt > 0 && !trg_normal) return fail(MFS_EINVAL, "NULL target normals");
    if (nt == 0) return MFS_OK;
    hipStream_t s = (hipStream_t)stream;
    const int kind = field == MFS_FIELD_LAPLACE_GRADIENT ? MFS_LAPLACE : MFS_STOKES;
    const int dim = field == MFS_FIELD_PRESSURE ? 1 : 3;
    Workspace &ws = workspace();
    Layout *lay = nullptr;
    MFS_TRY(layout(ws, 4 + field, kind, dim, 1.0, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nb, s, &lay));
    P2PLaunch L;
    MFS_TRY(standalone_operands(ws, *lay, kind, nb, nt, ns, trg_xyz, src_xyz, str, prec, s, L));
    L.skip_same = (flags & MFS_SKIP_SAME_BODY) != 0;
    L.accumulate = (flags & MFS_ACCUMULATE) != 0;
    L.out = out;
    L.n_val = dim * nt;
    MFS_TRY(standalone_partial(ws, *lay, L));
    return launch_field(field, lay->pp, L, trg_normal, nt, s);
}

// Position gradient of the pairing over one orientation: lanes carry lane_vec
// ([n_lane][dim]), sources carry src_str; out_grad [n_lane][3].  out_sum (or null): the sum of the
// sources at the lanes as well, [n_lane][dim].
int p2p_grad_standalone(int kind, int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *lane_ptr,
                        const int64_t *src_ptr, const double *lane_xyz, const double *src_xyz, const double *lane_vec,
                        const double *src_str, double *out_grad, double *out_sum, double mu, int flags, int prec,
                        hipStream_t s) {
    const int64_t nb = sys_body_ptr[n_sys], nl = lane_ptr[nb], ns = src_ptr[nb];
    if (nl == 0) return MFS_OK;
    Workspace &ws = workspace();
    const int dim = kind == MFS_STOKES ? 3 : 1;
    Layout *lay = nullptr;
    MFS_TRY(layout(ws, 8 + kind, kind, dim, mu, n_sys, sys_body_ptr, lane_ptr, src_ptr, nb, s, &lay));
    P2PLaunch L;
    MFS_TRY(standalone_operands(ws, *lay, kind, nb, nl, ns, lane_xyz, src_xyz, src_str, prec, s, L));
    L.skip_same = (flags & MFS_SKIP_SAME_BODY) != 0;
    L.accumulate = (flags & MFS_ACCUMULATE) != 0;
    L.out = out_grad;
    L.n_val = 3 * nl + (out_sum ? dim * nl : 0);  // values of a split slice
    MFS_TRY(standalone_partial(ws, *lay, L));
    return launch_p2p_grad(lay->pp, L, lane_vec, nl, s, out_sum, dim * nl);
}

int p2p_backward_standalone(int kind, int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                            const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                            const double *src_s, const double *trg_w, double *grad_src, double *grad_trg_xyz,
                            double *grad_src_xyz, double mu, int flags, int prec, void *stream) {
    int64_t nb, nt, ns;
    MFS_TRY(check_structure(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, &nb, &nt, &ns));
    MFS_TRY(check_prec(prec));
    if (flags & ~(MFS_SKIP_SAME_BODY | MFS_ACCUMULATE)) return fail(MFS_EINVAL, "unknown flags");
    if (kind == MFS_STOKES && !finite_pos(mu)) return fail(MFS_EINVAL, "mu must be finite and > 0");
    if ((nt > 0 && (!trg_xyz || !trg_w)) || (ns > 0 && (!src_xyz || !src_s)))
        return fail(MFS_EINVAL, "NULL data pointer");
    hipStream_t s = (hipStream_t)stream;
    if (grad_src && !grad_src_xyz)  // dPhi/ds_j = sum_i G(y_j - x_i) w_i: the sum with the roles swapped
        MFS_TRY(p2p_standalone(kind, n_sys, sys_body_ptr, body_src_ptr, body_trg_ptr, src_xyz, trg_xyz, trg_w, grad_src,
                               mu, flags, prec, stream));
    if (grad_trg_xyz)
        MFS_TRY(p2p_grad_standalone(kind, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, trg_w,
                                    src_s, grad_trg_xyz, nullptr, mu, flags, prec, s));
    if (grad_src_xyz)  // odd, symmetric pair term: the same kernel on the swapped orientation, dPhi/ds_j on the way
        MFS_TRY(p2p_grad_standalone(kind, n_sys, sys_body_ptr, body_src_ptr, body_trg_ptr, src_xyz, trg_xyz, src_s,
                                    trg_w, grad_src_xyz, grad_src, mu, flags, prec, s));
    return MFS_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
struct Factor {
    int kind, shape, dN, dM;
    int64_t ut_off, w_off, u_off, wt_off;
    double ratio;
};

struct mfs_plan_s {
    int prec = MFS_MIXED;
    int formulation = MFS_MOBILITY;
    int factorization = MFS_FACTOR_SVD;
    double mu = 1.0;
    int64_t n_sys = 0, n_body = 0;
    std::vector<int64_t> sys_body_ptr;
    std::vector<int32_t> sys_kind;
    std::vector<int32_t> kind, n_src, n_trg, factor_of_body, shape_of_body;
    std::vector<double> rot_h;  // [n_body][9]
    int64_t n_shape = 0;
    // shape point sets (shape frame) and per-shape proxy Gram inverses, kept so bodies can move
    std::vector<double> shape_src_h, shape_trg_h, G0i_h;
    std::vector<int64_t> sso, sto;
    std::vector<char> G0_ok;
    std::vector<int64_t> gam_off, lam_off, net_off;  // n_body + 1 entries
    std::vector<int64_t> src_row, trg_row;           // n_body + 1 entries
    int64_t n_gamma = 0, n_lambda = 0, n_net = 0, n_srcp = 0, n_trgp = 0;
    double min_ratio = 1.0;

    // device per-body arrays
    DevBuf d_kind, d_nsrc, d_ntrg, d_gam_off, d_lam_off, d_net_off, d_src_row32, d_trg_row32, d_rot, d_gram_inv,
        d_centre, d_src_row64, d_trg_row64;
    DevBuf d_src_off64, d_trg_off64, d_src_off32, d_trg_off32;  // [n][4] double / float4
    DevBuf d_src_body, d_trg_body;
    // pair operands: forward (sources = proxies), transposed (sources = collocation points)
    DevBuf fS32, fL32, fS64, fL64, tS32, tL32, tS64, tL64;
    // far tiles (mixed sums of Laplace plans), forward and transposed sources, and their work items
    struct Far {
        bool use = false;
        P2PPlan items;
        DevBuf tiles, tile_ptr, centre, rho;
        FarTiles view() const {
            FarTiles f;
            if (use) {
                f.tiles = tiles.ptr;
                f.tile_ptr = tile_ptr.as<int32_t>();
                f.centre = centre.as<double>();
                f.rho = rho.as<float>();
            }
            return f;
        }
    } far_fwd, far_tr;
    // factors
    DevBuf A64;        // FP64 factors, then the FP32 ones (one allocation: a large free takes 0.3 ms)
    int64_t pool = 0;  // values of each
    float *a32() const { return reinterpret_cast<float *>(A64.as<double>() + pool); }
    std::vector<Factor> factors;
    DevBuf d_col_gam, d_col_lam, d_col_of_body;
    // grouped GEMMs: forward U^T then W; transposed W^T then U
    struct GemmTables {
        DevBuf groups, tiles, col_group;
        GemmLaunch L;
    } gm[4];
    DevBuf gpart32, gpart64;
    // pair plans
    P2PPlan p2p_fwd, p2p_tr, p2p_fwd1, p2p_tr1;  // *1: one target per lane (gradient kernels)
    // workspace
    DevBuf ws_g32, ws_l32a, ws_l32b, ws_g64, ws_l64a, ws_l64b, ws_l64c, partial, sys_active;
    // GMRES
    int gm_cap = 0;
    DevBuf V, Wv, R, X, dots_partial, dots, nrm, coef, chunks, sys_chunk_ptr, flag;
    // least-squares state on the device (GivensState)
    DevBuf gvR, gvCS, gvSN, gvG, gvK, gvScale, gvInit, gvEst;
    // pinned host staging of the GMRES transfers (true asynchronous copies)
    double *h_dots = nullptr;  // [n_sys] per-system norms
    double *h_init = nullptr;  // [2 n_sys] residual targets, initial residual norms
    int32_t *h_act = nullptr;  // [n_sys]
    // [STAT_SLOTS][stat_bytes()] status blocks of recent iterations, written by the device
    // (fine-grained, mapped: d_stat is its device address)
    char *h_stat = nullptr, *d_stat = nullptr;
    static constexpr int STAT_SLOTS = 3;
    hipEvent_t stat_ev[STAT_SLOTS] = {nullptr, nullptr, nullptr};
    // est doubles, then flag int32, padded so every ring slot starts 16-byte aligned
    size_t stat_bytes() const { return ((size_t)n_sys * 12 + 15) & ~(size_t)15; }
    // backward
    DevBuf bw_sigma, bw_glam, bw_g, bw_w, bw_gt, bw_gs;
    // optional timing of the matvec pair-sum kernel (per precision)
    struct Timer {
        std::vector<hipEvent_t> ev;  // start/stop pairs
        int used = 0;
        int64_t launches = 0;
        double total_ms = 0.0;
    } timer[2];
    bool timing = false;
    double offbody_pairs = 0.0;
    // hipGraph replay of the GMRES matvec: captured once per (precision, direction)
    bool use_graph = false;
    double stop_factor = 0.1;  // GMRES iterates until its estimate is below stop_factor * tol
    hipStream_t capture_stream = nullptr;
    hipGraphExec_t graph[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
    DevBuf stage;  // fixed input buffer of the captured matvec
    // autotuned pair-sum launch shape
    int tuned_tpl = 1, tuned_min_items = 2048;
    bool tuned_persistent = false;
    // matvecs per system of the last GMRES solve, by precision
    std::vector<int32_t> last_mixed, last_fp64;
    // progress callback of long solves
    mfs_progress_fn progress = nullptr;
    void *progress_user = nullptr;
    bool stop_requested = false;
    std::vector<double> prog_bnorm;  // ||b|| per system of the running solve

    ~mfs_plan_s() {
        for (auto &t : timer)
            for (auto e : t.ev) (void)hipEventDestroy(e);
        for (auto &row : graph)
            for (auto &g : row)
                if (g) (void)hipGraphExecDestroy(g);
        if (capture_stream) (void)hipStreamDestroy(capture_stream);
        for (auto &e : stat_ev)
            if (e) (void)hipEventDestroy(e);
        free_pinned();
    }
    void free_pinned() {
        if (h_dots) (void)hipHostFree(h_dots);
        if (h_init) (void)hipHostFree(h_init);
        if (h_act) (void)hipHostFree(h_act);
        if (h_stat) (void)hipHostFree(h_stat);
        h_dots = h_init = nullptr;
        h_act = nullptr;
        h_stat = d_stat = nullptr;
    }
    GivensState givens() const {
        GivensState st;
        st.n_sys = (int)n_sys;
        st.cap = gm_cap;
        st.ldh = gm_cap + 2;
        st.dots = dots.as<double>();
        st.nrm2 = nrm.as<double>();
        st.target = gvInit.as<double>();
        st.beta = gvInit.as<double>() + n_sys;
        st.R = gvR.as<double>();
        st.cs = gvCS.as<double>();
        st.sn = gvSN.as<double>();
        st.g = gvG.as<double>();
        st.k = gvK.as<int32_t>();
        st.live = sys_active.as<int32_t>();
        st.scale = gvScale.as<double>();
        st.est = gvEst.as<double>();
        return st;
    }
    std::vector<VecChunk> h_chunks;
    std::vector<int32_t> h_sys_chunk_ptr;

    BodyView view() const {
        BodyView v;
        v.n_body = n_body;
        v.kind = d_kind.as<int32_t>();
        v.n_src = d_nsrc.as<int32_t>();
        v.n_trg = d_ntrg.as<int32_t>();
        v.gam_off = d_gam_off.as<int64_t>();
        v.lam_off = d_lam_off.as<int64_t>();
        v.net_off = d_net_off.as<int64_t>();
        v.src_row = d_src_row32.as<int32_t>();
        v.trg_row = d_trg_row32.as<int32_t>();
        v.rot = d_rot.as<double>();
        v.gram_inv = d_gram_inv.as<double>();
        v.src_off64 = d_src_off64.as<double>();
        v.trg_off64 = d_trg_off64.as<double>();
        v.dirichlet = formulation == MFS_RESISTANCE ? 1 : 0;
        return v;
    }
};

namespace {

// 6x6 inverse by Gauss-Jordan with partial pivoting (FP64, host).
bool inv6(const double *A, double *Ai) {
    double M[6][12];
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 12; ++c) M[r][c] = c < 6 ? A[6 * r + c] : (c - 6 == r ? 1.0 : 0.0);
    for (int c = 0; c < 6; ++c) {
        int p = c;
        for (int r = c + 1; r < 6; ++r)
            if (std::fabs(M[r][c]) > std::fabs(M[p][c])) p = r;
        if (!(std::fabs(M[p][c]) > 0.0)) return false;
        if (p != c)
            for (int k = 0; k < 12; ++k) std::swap(M[p][k], M[c][k]);
        const double d = M[c][c];
        for (int k = 0; k < 12; ++k) M[c][k] /= d;
        for (int r = 0; r < 6; ++r)
            if (r != c) {
                const double f = M[r][c];
                if (f != 0.0)
                    for (int k = 0; k < 12; ++k) M[r][k] -= f * M[c][k];
            }
    }
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c) Ai[6 * r + c] = M[r][c + 6];
    return true;
}

// Gram matrix K^T K of rigid-body rows [I, (p)_x] over points p (relative to the centre).
void gram6(const double *pts, int n, double *G) {
    std::fill(G, G + 36, 0.0);
    for (int j = 0; j < n; ++j) {
        const double *p = pts + 3 * j;
        const double X[3][3] = {{0.0, p[2], -p[1]}, {-p[2], 0.0, p[0]}, {p[1], -p[0], 0.0}};
        double K[3][6];
        for (int a = 0; a < 3; ++a)
            for (int q = 0; q < 6; ++q) K[a][q] = q < 3 ? (a == q ? 1.0 : 0.0) : X[a][q - 3];
        for (int r = 0; r < 6; ++r)
            for (int c = 0; c < 6; ++c) {
                double s = 0.0;
                for (int a = 0; a < 3; ++a) s += K[a][r] * K[a][c];
                G[6 * r + c] += s;
            }
    }
}

// world-frame Gram inverse: R2 G0^{-1} R2^T with R2 = diag(R, R)
void rotate_gram(const double *G0i, const double *R, double *Gi) {
    double R2[6][6] = {};
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) R2[a][b] = R2[a + 3][b + 3] = R[3 * a + b];
    double T[6][6];
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c) {
            double s = 0.0;
            for (int k = 0; k < 6; ++k) s += R2[r][k] * G0i[6 * k + c];
            T[r][c] = s;
        }
    for (int r = 0; r < 6; ++r)
        for (int c = 0; c < 6; ++c) {
            double s = 0.0;
            for (int k = 0; k < 6; ++k) s += T[r][k] * R2[c][k];
            Gi[6 * r + c] = s;
        }
}

// Work tables of one grouped GEMM: tiles of 32 x 32 outputs (one workgroup of
// four waves each), K split into n_split ranges of at least 512 when there are
// fewer than 1024 tiles (the fastest of the settings timed at 100 and 1000
// bodies).  A group's last column tile is narrow (VALU) when it holds at most
// GEMM_NARROW columns, so that no matrix-core work goes to padding columns there.
int build_gemm_launch(mfs_plan_s::GemmTables &T, const std::vector<GemmGroup> &groups,
                      const std::vector<int32_t> &col_group, const std::vector<int64_t> &b_col_off, hipStream_t s) {
    int64_t tiles32 = 0, kmax = 0, mmax = 0;
    for (auto &g : groups) {
        tiles32 += (int64_t)((g.M + 31) / 32) * ((g.ncol + 31) / 32);
        kmax = std::max<int64_t>(kmax, g.K);
        mmax = std::max<int64_t>(mmax, g.M);
    }
    const int64_t target = 1024, kmin = 512;
    int n_split = (int)std::max<int64_t>(1, std::min<int64_t>((target + tiles32 - 1) / tiles32, (kmax + kmin - 1) / kmin));
    std::vector<GemmTile> tiles;
    for (size_t gi = 0; gi < groups.size(); ++gi) {
        const GemmGroup &g = groups[gi];
        const int kchunk = (int)(((g.K + n_split - 1) / n_split + 63) / 64 * 64);
        // column tiles innermost: consecutive tiles, which the kernel places on one XCD,
        // then read the same rows and K range of A
        for (int m0 = 0; m0 < g.M; m0 += 32)
            for (int sp = 0; sp < n_split; ++sp)
                for (int n0 = 0; n0 < g.ncol; n0 += 32) {
                    const int k0 = std::min(g.K, sp * kchunk), k1 = std::min(g.K, k0 + kchunk);
                    const int32_t narrow = g.ncol - n0 <= GEMM_NARROW ? 1 : 0;
                    tiles.push_back(GemmTile{(int32_t)gi, m0, n0, k0, k1, sp, narrow});
                }
    }
    MFS_TRY(upload_vec(T.groups, groups, s));
    MFS_TRY(upload_vec(T.tiles, tiles, s));
    MFS_TRY(upload_vec(T.col_group, col_group, s));
    T.L.n_tiles = (int)tiles.size();
    T.L.n_split = n_split;
    T.L.n_cols = (int)col_group.size();
    T.L.tiles = T.tiles.as<GemmTile>();
    T.L.groups = T.groups.as<GemmGroup>();
    T.L.col_group = T.col_group.as<int32_t>();
    T.L.part_col_stride = mmax;
    T.L.part_split_stride = mmax * (int64_t)col_group.size();
    // 16-byte alignment of every A row and B column start (float offsets % 4; doubles only need % 2)
    bool al = true;
    for (auto &g : groups) al = al && g.a_off % 4 == 0 && g.K % 4 == 0;
    for (int64_t o : b_col_off) al = al && o % 4 == 0;
    T.L.vec4 = al ? 1 : 0;
    return MFS_OK;
}

int build_gemm_tables(mfs_plan p, hipStream_t s) {
    // groups: per factor, the list of its bodies as columns
    std::vector<std::vector<int32_t>> cols(p->factors.size());
    for (int64_t b = 0; b < p->n_body; ++b) cols[p->factor_of_body[b]].push_back((int32_t)b);
    std::vector<int64_t> col_gam, col_lam;
    std::vector<int32_t> col_group;
    std::vector<GemmGroup> g1, g2, t1, t2;
    for (size_t f = 0; f < p->factors.size(); ++f) {
        const Factor &F = p->factors[f];
        const int32_t cb = (int32_t)col_gam.size(), nc = (int32_t)cols[f].size();
        for (int32_t b : cols[f]) {
            col_gam.push_back(p->gam_off[b]);
            col_lam.push_back(p->lam_off[b]);
            col_group.push_back((int32_t)f);
        }
        g1.push_back(GemmGroup{F.dN, F.dM, cb, nc, F.ut_off});
        g2.push_back(GemmGroup{F.dN, F.dN, cb, nc, F.w_off});
        t1.push_back(GemmGroup{F.dN, F.dN, cb, nc, F.wt_off});
        t2.push_back(GemmGroup{F.dM, F.dN, cb, nc, F.u_off});
    }
    std::vector<int32_t> col_of_body(std::max<int64_t>(1, p->n_body), 0);
    {
        int32_t c = 0;
        for (auto &cf : cols)
            for (int32_t b : cf) col_of_body[b] = c++;
    }
    MFS_TRY(upload_vec(p->d_col_gam, col_gam, s));
    MFS_TRY(upload_vec(p->d_col_lam, col_lam, s));
    MFS_TRY(upload_vec(p->d_col_of_body, col_of_body, s));
    MFS_TRY(build_gemm_launch(p->gm[0], g1, col_group, col_gam, s));
    MFS_TRY(build_gemm_launch(p->gm[1], g2, col_group, col_lam, s));
    MFS_TRY(build_gemm_launch(p->gm[2], t1, col_group, col_lam, s));
    MFS_TRY(build_gemm_launch(p->gm[3], t2, col_group, col_lam, s));
    int64_t part = 1;
    for (auto &T : p->gm)
        if (T.L.n_split > 1) part = std::max<int64_t>(part, T.L.n_split * T.L.part_split_stride);
    MFS_TRY(p->gpart32.reserve(part * sizeof(float)));
    MFS_TRY(p->gpart64.reserve(part * sizeof(double)));
    return MFS_OK;
}

// FP64 SVD of every (shape, kind) S_L on the device; fills the factor pools.
// Factors of equal size are assembled side by side and factored by one
// strided-batched SVD (in chunks that keep the scratch under ~4 GB).
int factor_shapes(mfs_plan p, const mfs_plan_desc *d, const std::vector<int64_t> &shape_src_off,
                  const std::vector<int64_t> &shape_trg_off, hipStream_t s) {
    const bool qr = p->factorization == MFS_FACTOR_QR;
    rocblas_handle h = nullptr;  // for the SVD; its workspace takes 0.8 ms to allocate and free
    if (!qr && rocblas_create_handle(&h) != rocblas_status_success) return fail(MFS_EHIP, "rocblas_create_handle failed");
    std::unique_ptr<rocblas_handle, void (*)(rocblas_handle *)> guard(&h, [](rocblas_handle *hh) {
        if (*hh) rocblas_destroy_handle(*hh);
    });
    if (h) rocblas_set_stream(h, s);
    // pool layout
    int64_t pool = 0;
    for (auto &F : p->factors) {
        F.ut_off = pool;
        pool += (int64_t)F.dN * F.dM;
        F.w_off = pool;
        pool += (int64_t)F.dN * F.dN;
        F.wt_off = pool;
        pool += (int64_t)F.dN * F.dN;
        F.u_off = pool;
        pool += (int64_t)F.dM * F.dN;
    }
    pool = std::max<int64_t>(32, (pool + 31) / 32 * 32);  // the FP32 part on a 256-byte boundary
    MFS_TRY(p->A64.reserve(pool * (sizeof(double) + sizeof(float))));
    p->pool = pool;
    // batches of equal (m, n)
    std::vector<std::vector<int>> batches;
    {
        std::vector<std::pair<std::pair<int, int>, int>> keyed;
        for (int f = 0; f < (int)p->factors.size(); ++f)
            keyed.push_back({{p->factors[f].dM, p->factors[f].dN}, f});
        std::stable_sort(keyed.begin(), keyed.end(),
                         [](const auto &a, const auto &b) { return a.first < b.first; });
        const double cap = 4e9;
        for (size_t i = 0; i < keyed.size(); ++i) {
            const int m = keyed[i].first.first, n = keyed[i].first.second;
            const double bytes = 8.0 * ((double)2 * m * n + (double)n * n);
            const size_t per = (size_t)std::max(1.0, cap / bytes);
            if (batches.empty() || p->factors[batches.back()[0]].dM != m || p->factors[batches.back()[0]].dN != n ||
                batches.back().size() >= per)
                batches.push_back({});
            batches.back().push_back(keyed[i].second);
        }
    }
    DevBuf mats, Sv, E, info, work, pts, gi, inv, tau;
    for (auto &bt : batches) {
        const int B = (int)bt.size();
        const int m = p->factors[bt[0]].dM, n = p->factors[bt[0]].dN;
        const int64_t smn = (int64_t)m * n, snn = (int64_t)n * n;
        MFS_TRY(mats.reserve((size_t)B * (2 * smn + snn) * sizeof(double)));  // a large free takes 0.3 ms
        double *SL = mats.as<double>(), *Ub = SL + B * smn, *Vb = Ub + B * smn;
        MFS_TRY(Sv.reserve((size_t)B * n * sizeof(double)));
        MFS_TRY(E.reserve((size_t)B * n * sizeof(double)));
        MFS_TRY(info.reserve((size_t)B * sizeof(rocblas_int)));
        // geometry of every factor of the batch, then assembly of each S_L
        int maxM = 0;
        std::vector<double> hp, hg;
        std::vector<int64_t> pts_off;
        for (int f : bt) {
            const Factor &F = p->factors[f];
            const int N = d->shape_n_src[F.shape], M = d->shape_n_trg[F.shape];
            maxM = std::max(maxM, M);
            pts_off.push_back((int64_t)hp.size());
            hp.insert(hp.end(), d->shape_trg + 3 * shape_trg_off[F.shape],
                      d->shape_trg + 3 * (shape_trg_off[F.shape] + M));
            hp.insert(hp.end(), d->shape_src + 3 * shape_src_off[F.shape],
                      d->shape_src + 3 * (shape_src_off[F.shape] + N));
            double G[36], Gi[36];
            gram6(d->shape_src + 3 * shape_src_off[F.shape], N, G);
            if (F.kind == MFS_STOKES && !inv6(G, Gi)) return fail(MFS_ENUMERIC, "singular proxy Gram matrix");
            if (F.kind != MFS_STOKES) std::fill(Gi, Gi + 36, 0.0);
            hg.insert(hg.end(), Gi, Gi + 36);
        }
        MFS_TRY(upload_vec(pts, hp, s));
        MFS_TRY(upload_vec(gi, hg, s));
        MFS_TRY(work.reserve((size_t)3 * maxM * 6 * sizeof(double)));
        for (int q = 0; q < B; ++q) {
            const Factor &F = p->factors[bt[q]];
            const int N = d->shape_n_src[F.shape], M = d->shape_n_trg[F.shape];
            const double *P = pts.as<double>() + pts_off[q];
            MFS_TRY(launch_assemble_SL(F.kind, M, N, P, P + 3 * (size_t)M, gi.as<double>() + 36 * q, p->mu,
                                       p->formulation == MFS_RESISTANCE, SL + q * smn,
                                       work.as<double>(), s));
        }
        if (qr) {
            // S_L = Q R (library QR): U^T <- Q^T, U <- Q, W <- R^-1, W^T <- R^-T
            MFS_TRY(tau.reserve(qr_scratch_doubles(B, n) * sizeof(double)));
            MFS_TRY(qr_inverse_batched(B, SL, m, n, smn, Ub, smn, Vb, snn,
                                       tau.as<double>(), Sv.as<double>(), s));
            std::vector<double> rat(B);
            MFS_HIP_TRY(hipMemcpyAsync(rat.data(), Sv.ptr, B * sizeof(double), hipMemcpyDeviceToHost, s));
            MFS_HIP_TRY(hipStreamSynchronize(s));
            double *A64 = p->A64.as<double>();
            float *A32 = p->a32();
            for (int q = 0; q < B; ++q) {
                Factor &F = p->factors[bt[q]];
                F.ratio = std::isfinite(rat[q]) ? rat[q] : 0.0;
                p->min_ratio = std::min(p->min_ratio, F.ratio);
                if (!(F.ratio > 1e-14))
                    return fail(MFS_ENUMERIC, "QR: 1/(|R|_F |R^-1|_F) = " + std::to_string(F.ratio) + " <= 1e-14");
                const double *Q = Ub + q * smn, *X = Vb + q * snn;
                MFS_TRY(launch_make_factor(n, m, Q, m, false, nullptr, nullptr, A64 + F.ut_off, A32 + F.ut_off, s));
                MFS_TRY(launch_make_factor(m, n, Q, m, true, nullptr, nullptr, A64 + F.u_off, A32 + F.u_off, s));
                // X column-major (ld n): W[r][c] = X[c n + r], W^T[r][c] = X[r n + c]
                MFS_TRY(launch_make_factor(n, n, X, n, true, nullptr, nullptr, A64 + F.w_off, A32 + F.w_off, s));
                MFS_TRY(launch_make_factor(n, n, X, n, false, nullptr, nullptr, A64 + F.wt_off, A32 + F.wt_off, s));
            }
            MFS_HIP_TRY(hipStreamSynchronize(s));
            continue;
        }
        rocblas_status st = rocsolver_dgesvd_strided_batched(
            h, rocblas_svect_singular, rocblas_svect_singular, m, n, SL, m, smn, Sv.as<double>(), n,
            Ub, m, smn, Vb, n, snn, E.as<double>(), n, rocblas_outofplace,
            info.as<rocblas_int>(), B);
        if (st != rocblas_status_success) return fail(MFS_EHIP, "rocsolver_dgesvd_strided_batched failed");
        std::vector<double> sv((size_t)B * n);
        std::vector<rocblas_int> hinfo(B);
        MFS_HIP_TRY(hipMemcpyAsync(sv.data(), Sv.ptr, sv.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        MFS_HIP_TRY(hipMemcpyAsync(hinfo.data(), info.ptr, B * sizeof(rocblas_int), hipMemcpyDeviceToHost, s));
        MFS_HIP_TRY(hipStreamSynchronize(s));
        std::vector<double> hinv((size_t)B * n);
        for (int q = 0; q < B; ++q) {
            Factor &F = p->factors[bt[q]];
            if (hinfo[q] != 0) return fail(MFS_ENUMERIC, "SVD did not converge");
            const double *svq = sv.data() + (size_t)q * n;
            F.ratio = svq[n - 1] / svq[0];
            p->min_ratio = std::min(p->min_ratio, F.ratio);
            if (!(F.ratio > 1e-14))
                return fail(MFS_ENUMERIC, "sigma_min/sigma_max = " + std::to_string(F.ratio) + " <= 1e-14");
            for (int i = 0; i < n; ++i) hinv[(size_t)q * n + i] = 1.0 / svq[i];
        }
        MFS_TRY(upload_vec(inv, hinv, s));
        double *A64 = p->A64.as<double>();
        float *A32 = p->a32();
        for (int q = 0; q < B; ++q) {
            const Factor &F = p->factors[bt[q]];
            const double *U = Ub + q * smn, *V = Vb + q * snn;
            const double *iv = inv.as<double>() + (size_t)q * n;
            // U^T (n x m): row r = column r of U (column-major, ld m)
            MFS_TRY(launch_make_factor(n, m, U, m, false, nullptr, nullptr, A64 + F.ut_off, A32 + F.ut_off, s));
            // U (m x n) row-major: U[r][c] = Ucm[c*m + r]
            MFS_TRY(launch_make_factor(m, n, U, m, true, nullptr, nullptr, A64 + F.u_off, A32 + F.u_off, s));
            // W = V Sigma^{-1}: the V^T output (column-major, ld n) read row-major is V
            MFS_TRY(launch_make_factor(n, n, V, n, false, nullptr, iv, A64 + F.w_off, A32 + F.w_off, s));
            // W^T = Sigma^{-1} V^T
            MFS_TRY(launch_make_factor(n, n, V, n, true, iv, nullptr, A64 + F.wt_off, A32 + F.wt_off, s));
        }
        MFS_HIP_TRY(hipStreamSynchronize(s));
    }
    return MFS_OK;
}

}  // namespace

// The work items of the far walks, in the shape of the plan's other pair sums.
static int build_far_items(mfs_plan_s *p, int min_items, bool persistent, hipStream_t s) {
    const std::vector<int64_t> &src_row = p->src_row, &trg_row = p->trg_row;
    if (p->far_fwd.use)
        MFS_TRY(build_p2p_items(p->far_fwd.items, p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                                p->gam_off.data(), p->kind.data(), p->mu, 1, min_items, s, true));
    if (p->far_tr.use)
        MFS_TRY(build_p2p_items(p->far_tr.items, p->n_sys, p->sys_body_ptr.data(), src_row.data(), trg_row.data(),
                                p->lam_off.data(), p->kind.data(), p->mu, 1, min_items, s, true));
    p->far_fwd.items.persistent = p->far_tr.items.persistent = persistent;
    return MFS_OK;
}

// Everything of a plan that depends on where the bodies are: centres, rotations,
// world-axis offsets of every point (FP64 and FP32), per-body Gram inverses
// G^-1 = R G0^-1 R^T, and the positions in the pair-operand records (strengths
// are written per call).  The per-shape factors live in the shape frame and do
// not depend on it (congruent bodies share one factorisation, Sec. 3.3).
// Buffer sizes never change, so device pointers (and captured graphs) stay valid.
static int upload_geometry(mfs_plan_s *p, const double *centre, const double *rot, hipStream_t s) {
    const int64_t nb = p->n_body;
    std::vector<double> so64(4 * p->n_srcp), to64(4 * p->n_trgp);
    std::vector<float> so32(4 * p->n_srcp), to32(4 * p->n_trgp);
    std::vector<double> gram(36 * nb, 0.0);
    for (int64_t b = 0; b < nb; ++b) {
        const int sh = p->shape_of_body[b];
        const double *R = rot + 9 * b;
        auto emit = [&](const double *loc, int n, int64_t row0, std::vector<double> &o64, std::vector<float> &o32) {
            for (int i = 0; i < n; ++i) {
                const double *q = loc + 3 * i;
                for (int a = 0; a < 3; ++a) {
                    const double v = R[3 * a] * q[0] + R[3 * a + 1] * q[1] + R[3 * a + 2] * q[2];
                    o64[4 * (row0 + i) + a] = v;
                    o32[4 * (row0 + i) + a] = (float)v;
                }
                o64[4 * (row0 + i) + 3] = 0.0;
                o32[4 * (row0 + i) + 3] = 0.f;
            }
        };
        emit(p->shape_src_h.data() + 3 * p->sso[sh], p->n_src[b], p->src_row[b], so64, so32);
        emit(p->shape_trg_h.data() + 3 * p->sto[sh], p->n_trg[b], p->trg_row[b], to64, to32);
        if (p->kind[b] == MFS_STOKES) {
            if (!p->G0_ok[sh]) {
                double G[36];
                gram6(p->shape_src_h.data() + 3 * p->sso[sh], p->n_src[b], G);
                if (!inv6(G, &p->G0i_h[36 * sh])) return fail(MFS_ENUMERIC, "singular proxy Gram matrix");
                p->G0_ok[sh] = 1;
            }
            rotate_gram(&p->G0i_h[36 * sh], R, &gram[36 * b]);
        }
    }
    p->rot_h.assign(rot, rot + 9 * nb);
    std::vector<double> cen(centre, centre + 3 * nb), rotv(rot, rot + 9 * nb);
    MFS_TRY(upload_vec(p->d_rot, rotv, s));
    MFS_TRY(upload_vec(p->d_gram_inv, gram, s));
    MFS_TRY(upload_vec(p->d_centre, cen, s));
    MFS_TRY(upload_vec(p->d_src_off64, so64, s));
    MFS_TRY(upload_vec(p->d_trg_off64, to64, s));
    MFS_TRY(upload_vec(p->d_src_off32, so32, s));
    MFS_TRY(upload_vec(p->d_trg_off32, to32, s));
    // pair operand records: positions now, strengths written per call
    auto records = [&](int64_t n, const std::vector<double> &o64, const std::vector<float> &o32, DevBuf &S32,
                       DevBuf &L32, DevBuf &S64, DevBuf &L64) -> int {
        std::vector<SrcS32> s32(n);
        std::vector<SrcL32> l32(n);
        std::vector<SrcS64> s64(n);
        std::vector<SrcL64> l64(n);
        for (int64_t j = 0; j < n; ++j) {
            s32[j].pos = make_float4(o32[4 * j], o32[4 * j + 1], o32[4 * j + 2], 0.f);
            s32[j].str = make_float4(0.f, 0.f, 0.f, 0.f);
            l32[j] = make_float4(o32[4 * j], o32[4 * j + 1], o32[4 * j + 2], 0.f);
            s64[j] = SrcS64{{o64[4 * j], o64[4 * j + 1], o64[4 * j + 2], 0.0}, {0.0, 0.0, 0.0, 0.0}};
            l64[j] = SrcL64{{o64[4 * j], o64[4 * j + 1], o64[4 * j + 2], 0.0}};
        }
        MFS_TRY(upload_vec(S32, s32, s));
        MFS_TRY(upload_vec(L32, l32, s));
        MFS_TRY(upload_vec(S64, s64, s));
        MFS_TRY(upload_vec(L64, l64, s));
        // the staging vectors are pageable and local: finish the copies before they go
        MFS_HIP_TRY(hipStreamSynchronize(s));
        return MFS_OK;
    };
    MFS_TRY(records(p->n_srcp, so64, so32, p->fS32, p->fL32, p->fS64, p->fL64));
    MFS_TRY(records(p->n_trgp, to64, to32, p->tS32, p->tL32, p->tS64, p->tL64));
    if (p->far_fwd.use)
        MFS_TRY(launch_far_pack(nb, p->d_src_row32.as<int32_t>(), p->d_src_off64.as<double>(), 4,
                                p->d_centre.as<double>(), p->far_fwd.view(), s));
    if (p->far_tr.use)
        MFS_TRY(launch_far_pack(nb, p->d_trg_row32.as<int32_t>(), p->d_trg_off64.as<double>(), 4,
                                p->d_centre.as<double>(), p->far_tr.view(), s));
    return MFS_OK;
}

// ---------------------------------------------------------------------------
// The allocation-free Stokes pair sum (mfs_p2p_stokes_noalloc).  Its device
// scratch is one file-scope array: every GPU the library runs on holds a copy of
// kScratchBytes from module load until the process ends.  In host code the name
// `scratch` is only a host-side stand-in; its device address on the current
// device comes from hipGetSymbolAddress (taken once per device, on the first
// call there) and only that address is handed to kernels.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr int64_t kNoAllocMaxBodies = int64_t(1) << 16;
constexpr int64_t kNoAllocMaxItems = int64_t(1) << 15;
constexpr int kNoAllocMaxDevices = 64;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

// Host staging of the structure and work items: static storage (no heap), used
// under g_noalloc_mutex by one call at a time.
struct NoAllocHost {
    int32_t trg32[kNoAllocMaxBodies + 1], src32[kNoAllocMaxBodies + 1];
    P2PItem items[kNoAllocMaxItems], sorted[kNoAllocMaxItems];
    double work[kNoAllocMaxItems];
    int32_t order[kNoAllocMaxItems];
};
NoAllocHost g_noalloc_host;
std::mutex g_noalloc_mutex;
void *g_scratch_ptr[kNoAllocMaxDevices];  // device address of `scratch` per device (guarded by the mutex)

int scratch_address(void **out) {
    int dev = 0;
    MFS_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kNoAllocMaxDevices) return fail(MFS_EUNSUPPORTED, "device index beyond 63");
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(MFS_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return MFS_OK;
}

size_t align256(size_t n) { return (n + 255) & ~size_t(255); }

int p2p_stokes_noalloc(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                       const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz, const double *str,
                       double *out, double mu, int flags, int prec, void *stream) {
    int64_t nb, nt, ns;
    MFS_TRY(check_structure(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, &nb, &nt, &ns));
    MFS_TRY(check_prec(prec));
    if (flags & ~(MFS_SKIP_SAME_BODY | MFS_ACCUMULATE)) return fail(MFS_EINVAL, "unknown flags");
    if (!finite_pos(mu)) return fail(MFS_EINVAL, "mu must be finite and > 0");
    if ((nt > 0 && (!trg_xyz || !out)) || (ns > 0 && (!src_xyz || !str)))
        return fail(MFS_EINVAL, "NULL data pointer");
    if (nb > kNoAllocMaxBodies)
        return fail(MFS_EINVAL, "mfs_p2p_stokes_noalloc takes at most " + std::to_string(kNoAllocMaxBodies) + " bodies");
    if (nt == 0) return MFS_OK;
    hipStream_t s = (hipStream_t)stream;
    const bool overlap = overlaps_inputs(out, 3 * nt, trg_xyz, src_xyz, str, nt, ns, 3);
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    NoAllocHost &h = g_noalloc_host;
    int64_t n_items = 0;
    int n_split = 1;
    MFS_TRY(generate_p2p_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nullptr, 3, nullptr, MFS_STOKES, mu, 1,
                               standalone_min_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, MFS_STOKES,
                                                    prec == MFS_MIXED && !overlap, false, kStandaloneMinItems),
                               h.items, h.work, h.order, h.sorted, kNoAllocMaxItems, &n_items,
                               &n_split));
    // scratch layout (256-byte aligned pieces)
    const bool f32 = prec == MFS_MIXED;
    const size_t sz_ptr = align256((nb + 1) * sizeof(int32_t));
    const size_t sz_tb = align256(nt * sizeof(int32_t)), sz_sb = align256(ns * sizeof(int32_t));
    const size_t sz_c = align256(nb * 3 * sizeof(double));
    const size_t sz_to = align256(nt * (f32 ? 16 : 32));
    const size_t sz_so = align256(ns * (f32 ? sizeof(SrcS32) : sizeof(SrcS64)));
    const size_t sz_it = align256(n_items * sizeof(P2PItem));
    const size_t sz_pa = n_split > 1 ? align256((size_t)n_split * 3 * nt * sizeof(double)) : 0;
    const size_t need = 2 * sz_ptr + sz_tb + sz_sb + sz_c + sz_to + sz_so + sz_it + sz_pa;
    if (need > kScratchBytes)
        return fail(MFS_EINVAL, "mfs_p2p_stokes_noalloc needs " + std::to_string(need) +
                                    " bytes of scratch for these sizes; it holds " + std::to_string(kScratchBytes));
    // checked above on the general items, so that what is refused does not depend on the walk
    const bool wide = f32 && use_wide_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, MFS_STOKES) && !overlap;
    if (wide)
        MFS_TRY(generate_p2p_items(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, nullptr, 3, nullptr, MFS_STOKES, mu,
                                   1, 1, h.items, h.work, h.order, h.sorted, kNoAllocMaxItems, &n_items, &n_split));
    void *base = nullptr;
    MFS_TRY(scratch_address(&base));
    unsigned char *q = static_cast<unsigned char *>(base);
    int32_t *d_trg_ptr = reinterpret_cast<int32_t *>(q);
    q += sz_ptr;
    int32_t *d_src_ptr = reinterpret_cast<int32_t *>(q);
    q += sz_ptr;
    int32_t *d_trg_body = reinterpret_cast<int32_t *>(q);
    q += sz_tb;
    int32_t *d_src_body = reinterpret_cast<int32_t *>(q);
    q += sz_sb;
    double *d_centre = reinterpret_cast<double *>(q);
    q += sz_c;
    void *d_trg_off = q;
    q += sz_to;
    void *d_src_ops = q;
    q += sz_so;
    P2PItem *d_items = reinterpret_cast<P2PItem *>(q);
    q += sz_it;
    double *d_partial = sz_pa ? reinterpret_cast<double *>(q) : nullptr;
    for (int64_t b = 0; b <= nb; ++b) {
        h.trg32[b] = (int32_t)body_trg_ptr[b];
        h.src32[b] = (int32_t)body_src_ptr[b];
    }
    MFS_HIP_TRY(hipMemcpyAsync(d_trg_ptr, h.trg32, (nb + 1) * sizeof(int32_t), hipMemcpyHostToDevice, s));
    MFS_HIP_TRY(hipMemcpyAsync(d_src_ptr, h.src32, (nb + 1) * sizeof(int32_t), hipMemcpyHostToDevice, s));
    if (n_items) MFS_HIP_TRY(hipMemcpyAsync(d_items, h.sorted, n_items * sizeof(P2PItem), hipMemcpyHostToDevice, s));
    MFS_TRY(launch_fill_body_ids(nb, d_trg_ptr, d_trg_body, s));
    MFS_TRY(launch_fill_body_ids(nb, d_src_ptr, d_src_body, s));
    StandaloneOperands o;
    o.n_body = nb;
    o.n_trg = nt;
    o.n_src = ns;
    o.trg_ptr = d_trg_ptr;
    o.src_ptr = d_src_ptr;
    o.trg_body = d_trg_body;
    o.src_body = d_src_body;
    o.trg_xyz = trg_xyz;
    o.src_xyz = src_xyz;
    o.str = str;
    o.centre = d_centre;
    o.trg_off = d_trg_off;
    o.src_ops = d_src_ops;
    if (!wide) MFS_TRY(launch_operands(o, MFS_STOKES, prec, s));
    P2PItems it;
    it.items = d_items;
    it.wide = wide;
    it.n_items = (int)n_items;
    it.n_split = n_split;
    it.tpl = 1;
    P2PLaunch L;
    L.prec = prec;
    L.skip_same = (flags & MFS_SKIP_SAME_BODY) != 0;
    L.accumulate = (flags & MFS_ACCUMULATE) != 0;
    L.centre = d_centre;
    L.trg_body = d_trg_body;
    L.src_ptr = d_src_ptr;
    L.trg_off = d_trg_off;
    L.srcS = d_src_ops;
    if (wide) {
        L.raw_trg = trg_xyz;
        L.raw_src = src_xyz;
        L.raw_str = str;
    }
    L.out = out;
    L.partial = d_partial;
    L.n_val = 3 * nt;
    MFS_TRY(launch_p2p(it, L, s));
    // the staging above and the scratch are reused by the next call
    MFS_HIP_TRY(hipStreamSynchronize(s));
    return MFS_OK;
}

}  // namespace

extern "C" {

const char *mfs_last_error(void) { return g_last_error.c_str(); }
const char *mfs_version(void) { return "libmfs 0.1 (gfx950)"; }

int mfs_p2p_laplace(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                    const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz, const double *src_q,
                    double *out_u, int flags, int prec, void *stream) {
    return p2p_standalone(MFS_LAPLACE, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, src_q, out_u,
                          1.0, flags, prec, stream);
}

int mfs_p2p_stokes(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                   const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz, const double *src_f,
                   double *out_u, double mu, int flags, int prec, void *stream) {
    return p2p_standalone(MFS_STOKES, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, src_f, out_u,
                          mu, flags, prec, stream);
}

int mfs_p2p_stokes_noalloc(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                           const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                           const double *src_f, double *out_u, double mu, int flags, int prec, void *stream) {
    return p2p_stokes_noalloc(n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, src_f, out_u, mu,
                              flags, prec, stream);
}

int mfs_p2p_laplace_backward(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                             const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                             const double *src_q, const double *trg_w, double *grad_src_q, double *grad_trg_xyz,
                             double *grad_src_xyz, int flags, int prec, void *stream) {
    return p2p_backward_standalone(MFS_LAPLACE, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, src_q,
                                   trg_w, grad_src_q, grad_trg_xyz, grad_src_xyz, 1.0, flags, prec, stream);
}

int mfs_p2p_stokes_backward(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                            const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                            const double *src_f, const double *trg_w, double *grad_src_f, double *grad_trg_xyz,
                            double *grad_src_xyz, double mu, int flags, int prec, void *stream) {
    return p2p_backward_standalone(MFS_STOKES, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, src_xyz, src_f,
                                   trg_w, grad_src_f, grad_trg_xyz, grad_src_xyz, mu, flags, prec, stream);
}

int mfs_p2p_stokes_pressure(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                            const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                            const double *src_f, double *out_p, int flags, int prec, void *stream) {
    return field_standalone(MFS_FIELD_PRESSURE, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, nullptr,
                            src_xyz, src_f, out_p, flags, prec, stream);
}

int mfs_p2p_stokes_traction(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                            const int64_t *body_src_ptr, const double *trg_xyz, const double *trg_normal,
                            const double *src_xyz, const double *src_f, double *out_t, int flags, int prec,
                            void *stream) {
    return field_standalone(MFS_FIELD_TRACTION, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz, trg_normal,
                            src_xyz, src_f, out_t, flags, prec, stream);
}

int mfs_p2p_laplace_gradient(int64_t n_sys, const int64_t *sys_body_ptr, const int64_t *body_trg_ptr,
                             const int64_t *body_src_ptr, const double *trg_xyz, const double *src_xyz,
                             const double *src_q, double *out_g, int flags, int prec, void *stream) {
    return field_standalone(MFS_FIELD_LAPLACE_GRADIENT, n_sys, sys_body_ptr, body_trg_ptr, body_src_ptr, trg_xyz,
                            nullptr, src_xyz, src_q, out_g, flags, prec, stream);
}

int mfs_plan_destroy(mfs_plan plan) {
    if (!plan) return MFS_OK;
    (void)hipDeviceSynchronize();
    delete plan;
    return MFS_OK;
}

int mfs_plan_create(mfs_plan *out, const mfs_plan_desc *d, void *stream) {
    if (!out || !d) return fail(MFS_EINVAL, "NULL plan or descriptor");
    *out = nullptr;
    if (d->precision != MFS_MIXED && d->precision != MFS_FP64) return fail(MFS_EINVAL, "unknown precision");
    if (d->formulation != MFS_MOBILITY && d->formulation != MFS_RESISTANCE)
        return fail(MFS_EINVAL, "unknown formulation");
    if (d->factorization != MFS_FACTOR_SVD && d->factorization != MFS_FACTOR_QR)
        return fail(MFS_EINVAL, "unknown factorization");
    if (d->n_sys < 1 || !d->sys_body_ptr || !d->sys_kind) return fail(MFS_EINVAL, "bad system description");
    if (d->sys_body_ptr[0] != 0) return fail(MFS_EINVAL, "sys_body_ptr[0] must be 0");
    for (int64_t sy = 0; sy < d->n_sys; ++sy) {
        if (d->sys_body_ptr[sy + 1] < d->sys_body_ptr[sy]) return fail(MFS_EINVAL, "sys_body_ptr not non-decreasing");
        if (d->sys_kind[sy] != MFS_LAPLACE && d->sys_kind[sy] != MFS_STOKES) return fail(MFS_EINVAL, "unknown kind");
    }
    const int64_t nb = d->sys_body_ptr[d->n_sys];
    if (nb < 1) return fail(MFS_EINVAL, "no bodies");
    if (d->n_sys > 65535) return fail(MFS_EINVAL, "at most 65535 systems per plan");
    if (!d->centre || !d->rot || !d->shape_of_body) return fail(MFS_EINVAL, "NULL body arrays");
    if (d->n_shape < 1 || !d->shape_n_src || !d->shape_n_trg || !d->shape_src || !d->shape_trg)
        return fail(MFS_EINVAL, "bad shape description");
    if (!finite_pos(d->mu)) return fail(MFS_EINVAL, "mu must be finite and > 0");
    std::vector<int64_t> sso(d->n_shape + 1, 0), sto(d->n_shape + 1, 0);
    for (int64_t sh = 0; sh < d->n_shape; ++sh) {
        const int N = d->shape_n_src[sh], M = d->shape_n_trg[sh];
        if (N < 1 || M < N) return fail(MFS_EINVAL, "every shape needs 1 <= N <= M");
        sso[sh + 1] = sso[sh] + N;
        sto[sh + 1] = sto[sh] + M;
    }
    for (int64_t b = 0; b < nb; ++b)
        if (d->shape_of_body[b] < 0 || d->shape_of_body[b] >= d->n_shape) return fail(MFS_EINVAL, "bad shape id");
    for (int64_t q = 0; q < 3 * nb; ++q)
        if (!std::isfinite(d->centre[q])) return fail(MFS_EINVAL, "non-finite centre");
    for (int64_t q = 0; q < 9 * nb; ++q)
        if (!std::isfinite(d->rot[q])) return fail(MFS_EINVAL, "non-finite rotation");

    hipStream_t s = (hipStream_t)stream;
    std::unique_ptr<mfs_plan_s> p(new mfs_plan_s());
    p->prec = d->precision;
    p->formulation = d->formulation;
    p->factorization = d->factorization;
    p->n_shape = d->n_shape;
    p->shape_of_body.assign(d->shape_of_body, d->shape_of_body + nb);
    p->mu = d->mu;
    p->n_sys = d->n_sys;
    p->n_body = nb;
    p->sys_body_ptr.assign(d->sys_body_ptr, d->sys_body_ptr + d->n_sys + 1);
    p->sys_kind.assign(d->sys_kind, d->sys_kind + d->n_sys);
    p->kind.resize(nb);
    p->n_src.resize(nb);
    p->n_trg.resize(nb);
    p->factor_of_body.resize(nb);
    p->gam_off.resize(nb + 1);
    p->lam_off.resize(nb + 1);
    p->net_off.resize(nb + 1);
    p->src_row.resize(nb + 1);
    p->trg_row.resize(nb + 1);
    p->gam_off[0] = p->lam_off[0] = p->net_off[0] = p->src_row[0] = p->trg_row[0] = 0;
    std::vector<std::pair<int, int>> fkeys;
    for (int64_t sy = 0; sy < d->n_sys; ++sy)
        for (int64_t b = d->sys_body_ptr[sy]; b < d->sys_body_ptr[sy + 1]; ++b) {
            const int k = d->sys_kind[sy], sh = d->shape_of_body[b];
            const int dim = k == MFS_STOKES ? 3 : 1;
            p->kind[b] = k;
            p->n_src[b] = d->shape_n_src[sh];
            p->n_trg[b] = d->shape_n_trg[sh];
            p->gam_off[b + 1] = p->gam_off[b] + dim * p->n_trg[b];
            p->lam_off[b + 1] = p->lam_off[b] + dim * p->n_src[b];
            p->net_off[b + 1] = p->net_off[b] + (k == MFS_STOKES ? 6 : 1);
            p->src_row[b + 1] = p->src_row[b] + p->n_src[b];
            p->trg_row[b + 1] = p->trg_row[b] + p->n_trg[b];
            auto key = std::make_pair(sh, k);
            auto it = std::find(fkeys.begin(), fkeys.end(), key);
            if (it == fkeys.end()) {
                fkeys.push_back(key);
                p->factor_of_body[b] = (int)fkeys.size() - 1;
            } else {
                p->factor_of_body[b] = (int)(it - fkeys.begin());
            }
        }
    p->n_gamma = p->gam_off[nb];
    p->n_lambda = p->lam_off[nb];
    p->n_net = p->net_off[nb];
    p->n_srcp = p->src_row[nb];
    p->n_trgp = p->trg_row[nb];
    if (p->n_srcp > INT32_MAX / 2 || p->n_trgp > INT32_MAX / 2) return fail(MFS_EINVAL, "too many points");
    for (auto &k : fkeys) {
        Factor F{};
        F.shape = k.first;
        F.kind = k.second;
        const int dim = F.kind == MFS_STOKES ? 3 : 1;
        F.dN = dim * d->shape_n_src[F.shape];
        F.dM = dim * d->shape_n_trg[F.shape];
        p->factors.push_back(F);
    }
    // shape point sets are kept: bodies may move later (mfs_plan_set_bodies)
    p->sso = sso;
    p->sto = sto;
    p->shape_src_h.assign(d->shape_src, d->shape_src + 3 * sso[d->n_shape]);
    p->shape_trg_h.assign(d->shape_trg, d->shape_trg + 3 * sto[d->n_shape]);
    p->G0i_h.assign(36 * d->n_shape, 0.0);
    p->G0_ok.assign(d->n_shape, 0);
    std::vector<int32_t> sbody(p->n_srcp), tbody(p->n_trgp);
    for (int64_t b = 0; b < nb; ++b) {
        std::fill(sbody.begin() + p->src_row[b], sbody.begin() + p->src_row[b + 1], (int32_t)b);
        std::fill(tbody.begin() + p->trg_row[b], tbody.begin() + p->trg_row[b + 1], (int32_t)b);
    }
    std::vector<int32_t> src_row32(p->src_row.begin(), p->src_row.end()), trg_row32(p->trg_row.begin(), p->trg_row.end());
    MFS_TRY(upload_vec(p->d_kind, p->kind, s));
    MFS_TRY(upload_vec(p->d_nsrc, p->n_src, s));
    MFS_TRY(upload_vec(p->d_ntrg, p->n_trg, s));
    MFS_TRY(upload_vec(p->d_gam_off, p->gam_off, s));
    MFS_TRY(upload_vec(p->d_lam_off, p->lam_off, s));
    MFS_TRY(upload_vec(p->d_net_off, p->net_off, s));
    MFS_TRY(upload_vec(p->d_src_row32, src_row32, s));
    MFS_TRY(upload_vec(p->d_trg_row32, trg_row32, s));
    MFS_TRY(upload_vec(p->d_src_body, sbody, s));
    MFS_TRY(upload_vec(p->d_trg_body, tbody, s));
    auto far_buffers = [&](mfs_plan_s::Far &f, const std::vector<int64_t> &trg, const std::vector<int64_t> &src) -> int {
        std::vector<int32_t> tiles;
        if (p->prec != MFS_MIXED ||
            !use_far_tiles(p->n_sys, p->sys_body_ptr.data(), trg.data(), src.data(), p->kind.data(), tiles))
            return MFS_OK;
        MFS_TRY(f.tiles.reserve((size_t)tiles.back() * 1024));
        MFS_TRY(f.centre.reserve(nb * 3 * sizeof(double)));
        MFS_TRY(f.rho.reserve(nb * sizeof(float)));
        MFS_TRY(upload_vec(f.tile_ptr, tiles, s));
        MFS_HIP_TRY(hipStreamSynchronize(s));  // `tiles` is pageable and local
        f.use = true;
        return MFS_OK;
    };
    MFS_TRY(far_buffers(p->far_fwd, p->trg_row, p->src_row));
    MFS_TRY(far_buffers(p->far_tr, p->src_row, p->trg_row));
    MFS_TRY(upload_geometry(p.get(), d->centre, d->rot, s));
    // pair-sum items, forward (targets = collocation points) and transposed (targets = proxies)
    {
        std::vector<int64_t> src_row(p->src_row), trg_row(p->trg_row);
        const int min_items = default_min_items(p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                                                p->kind.data(), 0, kPlanMinItems);
        p->tuned_min_items = min_items;
        MFS_TRY(build_p2p_items(p->p2p_fwd, p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                                p->gam_off.data(), p->kind.data(), p->mu, 1, min_items, s));
        MFS_TRY(build_p2p_items(p->p2p_tr, p->n_sys, p->sys_body_ptr.data(), src_row.data(), trg_row.data(),
                                p->lam_off.data(), p->kind.data(), p->mu, 1, min_items, s));
        MFS_TRY(copy_p2p_items(p->p2p_fwd1, p->p2p_fwd, s));
        MFS_TRY(copy_p2p_items(p->p2p_tr1, p->p2p_tr, s));
        MFS_TRY(build_far_items(p.get(), min_items, false, s));
    }
    // workspace
    {
        const int64_t ng = std::max<int64_t>(1, p->n_gamma), nl = std::max<int64_t>(1, p->n_lambda);
        MFS_TRY(p->ws_g32.reserve(ng * sizeof(float)));
        MFS_TRY(p->ws_l32a.reserve(nl * sizeof(float)));
        MFS_TRY(p->ws_l32b.reserve(nl * sizeof(float)));
        MFS_TRY(p->ws_g64.reserve(ng * sizeof(double)));
        MFS_TRY(p->ws_l64a.reserve(nl * sizeof(double)));
        MFS_TRY(p->ws_l64b.reserve(nl * sizeof(double)));
        MFS_TRY(p->ws_l64c.reserve(nl * sizeof(double)));
        const int ns = std::max({p->p2p_fwd.n_split, p->p2p_tr.n_split, p->p2p_fwd1.n_split, p->p2p_tr1.n_split,
                                 p->far_fwd.items.n_split, p->far_tr.items.n_split});
        const int64_t nv = std::max({ng, nl, 3 * p->n_srcp, 3 * p->n_trgp});
        MFS_TRY(p->partial.reserve((size_t)(ns > 1 ? ns : 1) * nv * sizeof(double)));
        MFS_TRY(p->sys_active.reserve(p->n_sys * sizeof(int32_t)));
    }
    MFS_TRY(factor_shapes(p.get(), d, sso, sto, s));
    MFS_TRY(build_gemm_tables(p.get(), s));
    for (int64_t sy = 0; sy < p->n_sys; ++sy) {
        const int64_t b0 = p->sys_body_ptr[sy], b1 = p->sys_body_ptr[sy + 1];
        const double ns = (double)(p->src_row[b1] - p->src_row[b0]);
        for (int64_t b = b0; b < b1; ++b) p->offbody_pairs += (double)p->n_trg[b] * (ns - p->n_src[b]);
    }
    // GMRES chunks (never straddle a system)
    {
        // chunks never straddle a system; about 512 of them where that leaves each thread of their
        // workgroups 1 to 4 values (50 bodies: dot products 13.1 us in 88 chunks of 1024, 6.6 in 352 of 256)
        const int64_t CH = std::min<int64_t>(1024, std::max<int64_t>(256, (p->n_gamma / 512 + 255) / 256 * 256));
        p->h_sys_chunk_ptr.assign(1, 0);
        for (int64_t sy = 0; sy < p->n_sys; ++sy) {
            const int64_t a = p->gam_off[p->sys_body_ptr[sy]], e = p->gam_off[p->sys_body_ptr[sy + 1]];
            for (int64_t c = a; c < e; c += CH) p->h_chunks.push_back(VecChunk{c, std::min(e, c + CH), (int32_t)sy, 0});
            p->h_sys_chunk_ptr.push_back((int32_t)p->h_chunks.size());
        }
        MFS_TRY(upload_vec(p->chunks, p->h_chunks, s));
        MFS_TRY(upload_vec(p->sys_chunk_ptr, p->h_sys_chunk_ptr, s));
        MFS_TRY(p->flag.reserve(sizeof(int32_t)));
    }
    MFS_HIP_TRY(hipStreamSynchronize(s));
    *out = p.release();
    return MFS_OK;
}

int mfs_plan_sizes(mfs_plan p, int64_t *n_gamma, int64_t *n_lambda, int64_t *n_net, double *min_sigma_ratio) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (n_gamma) *n_gamma = p->n_gamma;
    if (n_lambda) *n_lambda = p->n_lambda;
    if (n_net) *n_net = p->n_net;
    if (min_sigma_ratio) *min_sigma_ratio = p->min_ratio;
    return MFS_OK;
}

int mfs_plan_set_bodies(mfs_plan p, const double *centre, const double *rot, void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (!centre || !rot) return fail(MFS_EINVAL, "NULL body arrays");
    for (int64_t q = 0; q < 3 * p->n_body; ++q)
        if (!std::isfinite(centre[q])) return fail(MFS_EINVAL, "non-finite centre");
    for (int64_t q = 0; q < 9 * p->n_body; ++q)
        if (!std::isfinite(rot[q])) return fail(MFS_EINVAL, "non-finite rotation");
    hipStream_t s = (hipStream_t)stream;
    MFS_HIP_TRY(hipStreamSynchronize(s));
    MFS_TRY(upload_geometry(p, centre, rot, s));
    MFS_HIP_TRY(hipStreamSynchronize(s));
    return MFS_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// operator pieces
// ---------------------------------------------------------------------------
namespace {

// out64 = (I - L)? R S_L^+ R^T in   (gamma layout in, lambda layout out), and/or the
// strengths of the forward pair-sum records of precision src_prec (src_prec < 0: none).
// Mixed plans apply both factors in FP32, except the triangular factor R^-1 of a QR plan:
// its entries are large and cancel on smooth inputs, so an FP32 copy errs at the solution
// by about 2e-5 of the operator's output against 6e-7 for the SVD's W = V Sigma^+ (a Type
// T block, cond 5.4e6), which costs refinement rounds; it is applied in FP64 instead.
// The second GEMM's split-K slices are added by the projection kernel, the one reader
// of its output, in the order its own reduction would add them (one launch fewer).
int precond_fwd(mfs_plan p, const double *in, int prec, bool project, double *out64, int src_prec, hipStream_t s) {
    BodyView bv = p->view();
    bool f32 = prec == MFS_MIXED;
    const GemmLaunch &G2 = p->gm[1].L;
    SplitSlices sl;
    sl.n = G2.n_split;
    sl.split_stride = G2.part_split_stride;
    sl.col_stride = G2.part_col_stride;
    sl.col_of_body = p->d_col_of_body.as<int32_t>();
    if (f32) {
        MFS_TRY(launch_rotate_in(bv, in, p->ws_g32.ptr, true, false, s));
        MFS_TRY(launch_gemm_f32(p->gm[0].L, p->a32(), p->ws_g32.as<float>(), p->d_col_gam.as<int64_t>(),
                                p->ws_l32a.as<float>(), p->d_col_lam.as<int64_t>(), p->gpart32.as<float>(), s));
        if (p->factorization == MFS_FACTOR_QR) {
            MFS_TRY(launch_cast(p->n_lambda, p->ws_l32a.ptr, true, p->ws_l64a.ptr, s));
            MFS_TRY(launch_gemm_f64(G2, p->A64.as<double>(), p->ws_l64a.as<double>(), p->d_col_lam.as<int64_t>(),
                                    p->ws_l64b.as<double>(), p->d_col_lam.as<int64_t>(), p->gpart64.as<double>(), s,
                                    false));
            sl.part = p->gpart64.ptr;
            f32 = false;  // lambda in FP64
        } else {
            MFS_TRY(launch_gemm_f32(G2, p->a32(), p->ws_l32a.as<float>(), p->d_col_lam.as<int64_t>(),
                                    p->ws_l32b.as<float>(), p->d_col_lam.as<int64_t>(), p->gpart32.as<float>(), s,
                                    false));
            sl.part = p->gpart32.ptr;
        }
    } else {
        MFS_TRY(launch_rotate_in(bv, in, p->ws_g64.ptr, false, false, s));
        MFS_TRY(launch_gemm_f64(p->gm[0].L, p->A64.as<double>(), p->ws_g64.as<double>(), p->d_col_gam.as<int64_t>(),
                                p->ws_l64a.as<double>(), p->d_col_lam.as<int64_t>(), p->gpart64.as<double>(), s));
        MFS_TRY(launch_gemm_f64(G2, p->A64.as<double>(), p->ws_l64a.as<double>(), p->d_col_lam.as<int64_t>(),
                                p->ws_l64b.as<double>(), p->d_col_lam.as<int64_t>(), p->gpart64.as<double>(), s,
                                false));
        sl.part = p->gpart64.ptr;
    }
    const void *lam = f32 ? (const void *)p->ws_l32b.ptr : (const void *)p->ws_l64b.ptr;
    void *S = nullptr, *L = nullptr;
    if (src_prec >= 0) {
        S = src_prec == MFS_MIXED ? p->fS32.ptr : p->fS64.ptr;
        L = src_prec == MFS_MIXED ? p->fL32.ptr : p->fL64.ptr;
    }
    return launch_project(bv, lam, f32, true, project, out64, S, L, src_prec < 0 ? 0 : src_prec, s, &sl);
}

// out (gamma layout) = R (S_L^+)^T R^T [(I - L)] in   (in: lambda layout, world)
int precond_tr(mfs_plan p, const double *in, int prec, bool project, double *out, hipStream_t s) {
    BodyView bv = p->view();
    const double *src = in;
    if (project) {
        MFS_TRY(launch_project(bv, in, false, false, true, p->ws_l64c.as<double>(), nullptr, nullptr, 0, s));
        src = p->ws_l64c.as<double>();
    }
    if (prec == MFS_MIXED) {
        if (p->factorization == MFS_FACTOR_QR) {  // R^-T in FP64 (see precond_fwd), then Q in FP32
            MFS_TRY(launch_rotate_in(bv, src, p->ws_l64a.ptr, false, true, s));
            MFS_TRY(launch_gemm_f64(p->gm[2].L, p->A64.as<double>(), p->ws_l64a.as<double>(),
                                    p->d_col_lam.as<int64_t>(), p->ws_l64b.as<double>(), p->d_col_lam.as<int64_t>(),
                                    p->gpart64.as<double>(), s));
            MFS_TRY(launch_cast(p->n_lambda, p->ws_l64b.ptr, false, p->ws_l32b.ptr, s));
        } else {
            MFS_TRY(launch_rotate_in(bv, src, p->ws_l32a.ptr, true, true, s));
            MFS_TRY(launch_gemm_f32(p->gm[2].L, p->a32(), p->ws_l32a.as<float>(),
                                    p->d_col_lam.as<int64_t>(), p->ws_l32b.as<float>(), p->d_col_lam.as<int64_t>(),
                                    p->gpart32.as<float>(), s));
        }
        MFS_TRY(launch_gemm_f32(p->gm[3].L, p->a32(), p->ws_l32b.as<float>(), p->d_col_lam.as<int64_t>(),
                                p->ws_g32.as<float>(), p->d_col_gam.as<int64_t>(), p->gpart32.as<float>(), s));
        return launch_rotate_out(bv, p->ws_g32.ptr, true, out, false, s);
    }
    MFS_TRY(launch_rotate_in(bv, src, p->ws_l64a.ptr, false, true, s));
    MFS_TRY(launch_gemm_f64(p->gm[2].L, p->A64.as<double>(), p->ws_l64a.as<double>(), p->d_col_lam.as<int64_t>(),
                            p->ws_l64b.as<double>(), p->d_col_lam.as<int64_t>(), p->gpart64.as<double>(), s));
    MFS_TRY(launch_gemm_f64(p->gm[3].L, p->A64.as<double>(), p->ws_l64b.as<double>(), p->d_col_lam.as<int64_t>(),
                            p->ws_g64.as<double>(), p->d_col_gam.as<int64_t>(), p->gpart64.as<double>(), s));
    return launch_rotate_out(bv, p->ws_g64.ptr, false, out, false, s);
}

// The work items of a plan's pair sums
const P2PPlan &fwd_items(mfs_plan p, int prec) {
    return prec == MFS_MIXED && p->far_fwd.use && p->p2p_fwd.tpl == 1 ? p->far_fwd.items : p->p2p_fwd;
}
const P2PPlan &tr_items(mfs_plan p, int prec) {
    return prec == MFS_MIXED && p->far_tr.use && p->p2p_tr.tpl == 1 ? p->far_tr.items : p->p2p_tr;
}

P2PLaunch fwd_launch(mfs_plan p, int prec) {
    P2PLaunch L;
    L.prec = prec;
    L.centre = p->d_centre.as<double>();
    L.trg_body = p->d_trg_body.as<int32_t>();
    L.src_ptr = p->d_src_row32.as<int32_t>();
    L.trg_off = prec == MFS_MIXED ? p->d_trg_off32.ptr : p->d_trg_off64.ptr;
    L.srcS = prec == MFS_MIXED ? p->fS32.ptr : p->fS64.ptr;
    L.srcL = prec == MFS_MIXED ? p->fL32.ptr : p->fL64.ptr;
    L.far = p->far_fwd.view();
    L.partial = p->partial.as<double>();
    L.n_val = p->n_gamma;
    return L;
}

P2PLaunch tr_launch(mfs_plan p, int prec) {
    P2PLaunch L;
    L.prec = prec;
    L.centre = p->d_centre.as<double>();
    L.trg_body = p->d_src_body.as<int32_t>();
    L.src_ptr = p->d_trg_row32.as<int32_t>();
    L.trg_off = prec == MFS_MIXED ? p->d_src_off32.ptr : p->d_src_off64.ptr;
    L.srcS = prec == MFS_MIXED ? p->tS32.ptr : p->tS64.ptr;
    L.srcL = prec == MFS_MIXED ? p->tL32.ptr : p->tL64.ptr;
    L.far = p->far_tr.view();
    L.partial = p->partial.as<double>();
    L.n_val = p->n_lambda;
    return L;
}

// write strengths (gamma layout) into the transposed pair records (collocation points as sources)
int set_tr_strength(mfs_plan p, const double *w, int prec, hipStream_t s) {
    BodyView tv = p->view();
    tv.n_src = tv.n_trg;
    tv.lam_off = tv.gam_off;
    tv.src_row = tv.trg_row;
    return launch_set_src_strength(tv, w, prec == MFS_MIXED ? p->tS32.ptr : p->tS64.ptr,
                                   prec == MFS_MIXED ? p->tL32.ptr : p->tL64.ptr, prec, s);
}

// write strengths (lambda layout) into the forward pair records
int set_fwd_strength(mfs_plan p, const double *str, int prec, hipStream_t s) {
    return launch_set_src_strength(p->view(), str, prec == MFS_MIXED ? p->fS32.ptr : p->fS64.ptr,
                                   prec == MFS_MIXED ? p->fL32.ptr : p->fL64.ptr, prec, s);
}

// Collects the elapsed times of the recorded event pairs of one precision.
int harvest_timer(mfs_plan p, int prec) {
    auto &t = p->timer[prec];
    if (t.used == 0) return MFS_OK;
    MFS_HIP_TRY(hipEventSynchronize(t.ev[2 * (t.used - 1) + 1]));
    for (int i = 0; i < t.used; ++i) {
        float ms = 0.f;
        MFS_HIP_TRY(hipEventElapsedTime(&ms, t.ev[2 * i], t.ev[2 * i + 1]));
        t.total_ms += ms;
        ++t.launches;
    }
    t.used = 0;
    return MFS_OK;
}

int matvec_impl(mfs_plan p, const double *gamma, double *out, int prec, const int32_t *sys_active, hipStream_t s) {
    MFS_TRY(precond_fwd(p, gamma, prec, p->formulation == MFS_MOBILITY, nullptr, prec, s));
    P2PLaunch L = fwd_launch(p, prec);
    L.skip_same = true;
    L.addend = gamma;
    L.out = out;
    L.sys_active = sys_active;
    if (p->timing) {
        auto &t = p->timer[prec];
        if (t.ev.empty()) {
            t.ev.resize(512);
            for (auto &e : t.ev) MFS_HIP_TRY(hipEventCreate(&e));
        }
        if (2 * t.used >= (int)t.ev.size()) MFS_TRY(harvest_timer(p, prec));
        L.ev_start = t.ev[2 * t.used];
        L.ev_stop = t.ev[2 * t.used + 1];
        ++t.used;
    }
    return launch_p2p(fwd_items(p, prec), L, s);
}

// (A^T w)^(k') = w^(k') + R (S_L^+)^T R^T (I - L^(k')) sum_{k != k'} S^(kk')T w^(k)
int matvec_adjoint_impl(mfs_plan p, const double *w, double *out, int prec, const int32_t *sys_active, hipStream_t s) {
    MFS_TRY(set_tr_strength(p, w, prec, s));
    P2PLaunch L = tr_launch(p, prec);
    L.skip_same = true;
    L.out = p->ws_l64c.as<double>();
    L.sys_active = sys_active;
    MFS_TRY(launch_p2p(tr_items(p, prec), L, s));
    if (p->formulation == MFS_MOBILITY)
        MFS_TRY(launch_project(p->view(), p->ws_l64c.as<double>(), false, false, true, p->ws_l64c.as<double>(),
                               nullptr, nullptr, 0, s));
    MFS_TRY(precond_tr(p, p->ws_l64c.as<double>(), prec, false, out, s));
    return launch_add_inplace(p->n_gamma, w, out, s);
}

int check_plan_prec(mfs_plan p, int prec) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    return check_prec(prec);
}

}  // namespace

extern "C" {

int mfs_rhs(mfs_plan p, const double *net, double *b, double *strength0, int prec, void *stream) {
    MFS_TRY(check_plan_prec(p, prec));
    if (!net || !b) return fail(MFS_EINVAL, "NULL net or b");
    hipStream_t s = (hipStream_t)stream;
    if (p->formulation == MFS_RESISTANCE) {
        if (strength0) MFS_TRY(launch_fill(p->n_lambda, 0.0, strength0, s));
        return launch_dirichlet_rhs(p->view(), net, b, s);
    }
    MFS_TRY(launch_completion(p->view(), net, strength0, prec == MFS_MIXED ? p->fS32.ptr : p->fS64.ptr,
                              prec == MFS_MIXED ? p->fL32.ptr : p->fL64.ptr, prec, s));
    P2PLaunch Lr = fwd_launch(p, prec);
    Lr.skip_same = false;
    Lr.alpha = -1.0;
    Lr.out = b;
    return launch_p2p(fwd_items(p, prec), Lr, s);
}

int mfs_precond_apply(mfs_plan p, const double *in, double *out, int flags, int prec, void *stream) {
    MFS_TRY(check_plan_prec(p, prec));
    if (!in || !out) return fail(MFS_EINVAL, "NULL in or out");
    if (flags & ~(MFS_PROJECT | MFS_TRANSPOSE)) return fail(MFS_EINVAL, "unknown flags");
    if ((flags & MFS_PROJECT) && p->formulation == MFS_RESISTANCE)
        return fail(MFS_EINVAL, "no projection in the resistance formulation");
    hipStream_t s = (hipStream_t)stream;
    if (flags & MFS_TRANSPOSE) return precond_tr(p, in, prec, (flags & MFS_PROJECT) != 0, out, s);
    return precond_fwd(p, in, prec, (flags & MFS_PROJECT) != 0, out, -1, s);
}

int mfs_matvec(mfs_plan p, const double *gamma, double *out, int prec, void *stream) {
    MFS_TRY(check_plan_prec(p, prec));
    if (!gamma || !out) return fail(MFS_EINVAL, "NULL gamma or out");
    if (gamma == out) return fail(MFS_EINVAL, "gamma and out must not alias");
    return matvec_impl(p, gamma, out, prec, nullptr, (hipStream_t)stream);
}

int mfs_matvec_adjoint(mfs_plan p, const double *w, double *out, int prec, void *stream) {
    MFS_TRY(check_plan_prec(p, prec));
    if (!w || !out) return fail(MFS_EINVAL, "NULL w or out");
    if (w == out) return fail(MFS_EINVAL, "w and out must not alias");
    return matvec_adjoint_impl(p, w, out, prec, nullptr, (hipStream_t)stream);
}

int mfs_extract(mfs_plan p, const double *gamma, const double *strength0, double *out, double *sigma, void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (!gamma || (!out && !sigma)) return fail(MFS_EINVAL, "NULL gamma or outputs");
    hipStream_t s = (hipStream_t)stream;
    MFS_TRY(precond_fwd(p, gamma, MFS_FP64, false, p->ws_l64c.as<double>(), -1, s));
    return launch_extract(p->view(), p->ws_l64c.as<double>(), strength0, out, sigma, s);
}

}  // extern "C"

// ---------------------------------------------------------------------------
// GMRES over the batch of systems
// ---------------------------------------------------------------------------
namespace {

int ensure_krylov(mfs_plan p, int max_iter) {
    if (p->gm_cap >= max_iter) return MFS_OK;
    const int64_t n = std::max<int64_t>(1, p->n_gamma);
    const int nc = (int)p->h_chunks.size();
    const int S = (int)p->n_sys;
    MFS_TRY(p->V.reserve((size_t)(max_iter + 1) * n * sizeof(double)));
    MFS_TRY(p->Wv.reserve(n * sizeof(double)));
    MFS_TRY(p->R.reserve(n * sizeof(double)));
    MFS_TRY(p->X.reserve(n * sizeof(double)));
    MFS_TRY(p->dots_partial.reserve((size_t)std::max(1, nc) * (max_iter + 2) * sizeof(double)));
    MFS_TRY(p->dots.reserve((size_t)S * 2 * (max_iter + 2) * sizeof(double)));
    MFS_TRY(p->nrm.reserve((size_t)S * sizeof(double)));
    MFS_TRY(p->coef.reserve((size_t)S * (max_iter + 2) * sizeof(double)));
    MFS_TRY(p->gvR.reserve((size_t)S * ((size_t)max_iter * (max_iter + 1) / 2) * sizeof(double)));
    MFS_TRY(p->gvCS.reserve((size_t)S * max_iter * sizeof(double)));
    MFS_TRY(p->gvSN.reserve((size_t)S * max_iter * sizeof(double)));
    MFS_TRY(p->gvG.reserve((size_t)S * (max_iter + 1) * sizeof(double)));
    MFS_TRY(p->gvK.reserve((size_t)S * sizeof(int32_t)));
    MFS_TRY(p->gvScale.reserve((size_t)S * sizeof(double)));
    MFS_TRY(p->gvInit.reserve((size_t)S * 2 * sizeof(double)));
    MFS_TRY(p->gvEst.reserve((size_t)S * sizeof(double)));
    for (auto &e : p->stat_ev)
        if (!e) MFS_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    // pinned staging (callers synchronise before a solve starts, so nothing is in flight here)
    p->free_pinned();
    if (hipHostMalloc((void **)&p->h_dots, (size_t)S * sizeof(double), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&p->h_init, (size_t)S * 2 * sizeof(double), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&p->h_act, (size_t)S * sizeof(int32_t), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&p->h_stat, p->STAT_SLOTS * p->stat_bytes(),
                      hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        p->free_pinned();
        return fail(MFS_ENOMEM, "hipHostMalloc of the GMRES staging buffers failed");
    }
    if (hipHostGetDevicePointer((void **)&p->d_stat, p->h_stat, 0) != hipSuccess) {
        p->free_pinned();
        return fail(MFS_EHIP, "hipHostGetDevicePointer of the GMRES status blocks failed");
    }
    p->gm_cap = max_iter;
    return MFS_OK;
}

// per-system squared norms of x -> host
int sys_norms(mfs_plan p, const double *x, std::vector<double> &out, hipStream_t s) {
    const int nc = (int)p->h_chunks.size();
    const int ldp = p->gm_cap + 2;
    MFS_TRY(launch_multi_dot(nc, p->chunks.as<VecChunk>(), x, 0, 1, x, p->dots_partial.as<double>(), ldp, s));
    MFS_TRY(launch_reduce_sys((int)p->n_sys, p->sys_chunk_ptr.as<int32_t>(), p->dots_partial.as<double>(), ldp, 1,
                              p->nrm.as<double>(), 1, s));
    out.resize(p->n_sys);
    double *h = p->h_dots;
    MFS_HIP_TRY(hipMemcpyAsync(h, p->nrm.ptr, p->n_sys * sizeof(double), hipMemcpyDeviceToHost, s));
    MFS_HIP_TRY(hipStreamSynchronize(s));
    for (int64_t i = 0; i < p->n_sys; ++i)
        out[i] = std::isnan(h[i]) ? h[i] : std::sqrt(std::max(0.0, h[i]));  // keep NaN visible
    return MFS_OK;
}

typedef int (*MatvecFn)(mfs_plan, const double *, double *, int, const int32_t *, hipStream_t);

// w = A v for the GMRES loop (w must be the plan's Krylov work vector).  With
// graphs enabled the matvec is captured once per (precision, direction) on a
// library stream with fixed buffers (v is staged into p->stage first) and
// replayed on the caller's stream; the captured work holds kernel launches
// only (no memset, no host synchronisation).
int apply_A(mfs_plan p, MatvecFn A, const double *v, double *w, int prec, hipStream_t s) {
    if (!p->use_graph || p->timing) return A(p, v, w, prec, p->sys_active.as<int32_t>(), s);
    const int dir = A == matvec_impl ? 0 : 1;
    MFS_TRY(p->stage.reserve(std::max<int64_t>(1, p->n_gamma) * sizeof(double)));
    hipGraphExec_t &ex = p->graph[prec][dir];
    if (!ex) {
        if (!p->capture_stream) MFS_HIP_TRY(hipStreamCreateWithFlags(&p->capture_stream, hipStreamNonBlocking));
        MFS_HIP_TRY(hipStreamSynchronize(s));
        hipGraph_t g = nullptr;
        MFS_HIP_TRY(hipStreamBeginCapture(p->capture_stream, hipStreamCaptureModeThreadLocal));
        const int st = A(p, p->stage.as<double>(), p->Wv.as<double>(), prec, p->sys_active.as<int32_t>(),
                         p->capture_stream);
        hipError_t e = hipStreamEndCapture(p->capture_stream, &g);
        if (st < 0) {
            if (g) (void)hipGraphDestroy(g);
            return st;
        }
        if (e != hipSuccess) return fail(MFS_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
        e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) {
            ex = nullptr;
            return fail(MFS_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
        }
    }
    if (w != p->Wv.as<double>()) return fail(MFS_EINVAL, "internal: graph output must be the Krylov work vector");
    MFS_HIP_TRY(hipMemcpyAsync(p->stage.ptr, v, p->n_gamma * sizeof(double), hipMemcpyDeviceToDevice, s));
    MFS_HIP_TRY(hipGraphLaunch(ex, s));
    return MFS_OK;
}

// One unrestarted GMRES attempt on A dx = r for every active system; x += dx.
// target[s]: absolute residual target.  counts[s] += matvecs spent.  est[s]: final estimate.
//
// The least-squares update (Givens rotations, residual estimate, stopping test) and the
// normalisation of the next Krylov vector run on the device, so the host enqueues
// iteration j + 1 while iteration j runs: it only waits for the status block of iteration
// j - 1 (one small asynchronous copy) to count matvecs, report progress and stop once no
// system is live.  A system that stops drops out of the matvec mask on the device, before
// the next matvec; an iteration enqueued after the last system stopped finds no live system
// and does no pair work.  beta holds the per-system norms of r (the caller has them already).
int gmres_attempt(mfs_plan p, MatvecFn A, int prec, const double *r, double *x, const std::vector<double> &target,
                  int max_iter, std::vector<int> &active, std::vector<int> &counts, std::vector<double> &est,
                  const std::vector<double> &beta, hipStream_t s) {
    const int S = (int)p->n_sys;
    const int64_t n = p->n_gamma;
    const int nc = (int)p->h_chunks.size();
    const int ldp = p->gm_cap + 2;
    const int ldh = p->gm_cap + 2;
    double *V = p->V.as<double>();
    double *w = p->Wv.as<double>();
    std::vector<int> act(S, 0);
    int n_act = 0;
    for (int sy = 0; sy < S; ++sy) {
        act[sy] = active[sy] && beta[sy] > target[sy] && std::isfinite(beta[sy]);
        if (active[sy] && !std::isfinite(beta[sy])) return fail(MFS_ENUMERIC, "non-finite residual");
        est[sy] = beta[sy];
        n_act += act[sy];
    }
    if (n_act == 0) return MFS_OK;
    // initial state: targets, norms and the mask go up through pinned buffers (the last
    // synchronisation, in sys_norms, ended every earlier copy out of them)
    for (int sy = 0; sy < S; ++sy) {
        p->h_init[sy] = target[sy];
        p->h_init[S + sy] = std::isfinite(beta[sy]) ? beta[sy] : 0.0;
        p->h_act[sy] = act[sy];
    }
    MFS_HIP_TRY(hipMemcpyAsync(p->gvInit.ptr, p->h_init, (size_t)S * 2 * sizeof(double), hipMemcpyHostToDevice, s));
    MFS_HIP_TRY(hipMemcpyAsync(p->sys_active.ptr, p->h_act, (size_t)S * sizeof(int32_t), hipMemcpyHostToDevice, s));
    const GivensState st = p->givens();
    MFS_TRY(launch_givens_init(st, s));
    MFS_TRY(launch_scale_sys(nc, p->chunks.as<VecChunk>(), r, st.scale, 1, V, s));
    const size_t sb = p->stat_bytes();
    auto slot = [&](int j) { return p->h_stat + (size_t)(j % mfs_plan_s::STAT_SLOTS) * sb; };
    auto slot_est = [&](int j) { return reinterpret_cast<const double *>(slot(j)); };
    auto slot_flag = [&](int j) { return reinterpret_cast<const int32_t *>(slot(j) + 8 * (size_t)S); };
    auto slot_err = [&](int j) {
        const int32_t *f = slot_flag(j);
        return std::any_of(f, f + S, [](int32_t v) { return (v & 2) != 0; });
    };
    // Iteration j is enqueued before the status of iteration j - lag is read.  lag = 1 keeps
    // the GPU busy across iterations; with a progress callback (meant for minutes-long
    // solves) lag = 0, so every iteration is reported as it ends and a stop takes effect
    // before the next one starts.
    const int lag = p->progress ? 0 : 1;
    for (int sy = 0; sy < S; ++sy) counts[sy] += act[sy];  // the matvec of iteration 0
    int done = 0;                                          // iterations enqueued
    bool empty_tail = false;  // the last enqueued iteration found no live system
    std::vector<double> prev_est(S, 0.0);                  // estimates after the previous status read
    for (int j = 0; j < max_iter; ++j) {
        MFS_TRY(apply_A(p, A, V + (int64_t)j * n, w, prec, s));
        // classical Gram-Schmidt, twice: dots, then (axpy + the next dots) twice, the last
        // dots being |w|^2
        double *dots = p->dots.as<double>();
        const VecChunk *ck = p->chunks.as<VecChunk>();
        double *part = p->dots_partial.as<double>();
        const int32_t *scp = p->sys_chunk_ptr.as<int32_t>();
        MFS_TRY(launch_multi_dot(nc, ck, V, n, j + 1, w, part, ldp, s));
        MFS_TRY(launch_reduce_sys(S, scp, part, ldp, j + 1, dots, 2 * ldh, s));
        MFS_TRY(launch_axpy_dot(nc, ck, V, n, j + 1, dots, 2 * ldh, -1.0, w, V, n, j + 1, part, ldp, s));
        MFS_TRY(launch_reduce_sys(S, scp, part, ldp, j + 1, dots + ldh, 2 * ldh, s));
        MFS_TRY(launch_axpy_dot(nc, ck, V, n, j + 1, dots + ldh, 2 * ldh, -1.0, w, w, 0, 1, part, ldp, s));
        // |w|^2 and the Givens step in one launch; the status slot written here was last read
        // for iteration j - 3, before iteration j - 1 was enqueued
        char *dslot = p->d_stat + (size_t)(j % mfs_plan_s::STAT_SLOTS) * sb;
        MFS_TRY(launch_givens_step(st, scp, part, ldp, p->nrm.as<double>(), j, reinterpret_cast<double *>(dslot),
                                   reinterpret_cast<int32_t *>(dslot + 8 * (size_t)S), s));
        MFS_HIP_TRY(hipEventRecord(p->stat_ev[j % mfs_plan_s::STAT_SLOTS], s));
        MFS_TRY(launch_scale_sys(nc, p->chunks.as<VecChunk>(), w, st.scale, 1, V + (int64_t)(j + 1) * n, s));
        done = j + 1;
        const int q = j - lag;  // the iteration whose status is read now
        if (q < 0) continue;
        MFS_HIP_TRY(hipEventSynchronize(p->stat_ev[q % mfs_plan_s::STAT_SLOTS]));
        if (slot_err(q)) {
            (void)hipStreamSynchronize(s);
            return fail(MFS_ENUMERIC, "non-finite Arnoldi vector");
        }
        const int32_t *lv = slot_flag(q);  // bit 0: live (bit 1, an error, is handled above)
        int n_live = 0;
        for (int sy = 0; sy < S; ++sy) n_live += lv[sy] & 1;
        if (p->progress) {  // counts hold the matvecs of iterations 0..q
            const double *es = slot_est(q);
            int most = 0;
            double worst = 0.0;
            for (int sy = 0; sy < S; ++sy) {
                most = std::max(most, counts[sy]);
                if (!act[sy]) continue;
                const double bn = sy < (int)p->prog_bnorm.size() && p->prog_bnorm[sy] > 0 ? p->prog_bnorm[sy] : 1.0;
                worst = std::max(worst, es[sy] / bn);
            }
            if (p->progress(p->progress_user, most, n_live, worst) != 0) {
                p->stop_requested = true;
                break;
            }
        }
        if (n_live == 0) {
            empty_tail = lag == 1;
            break;
        }
        // iteration q + 1 runs its matvec on the systems live after iteration q: with lag 1 it
        // is already enqueued, with lag 0 it is enqueued next unless the capacity ends here
        if (lag == 1 || q + 1 < max_iter)
            for (int sy = 0; sy < S; ++sy) counts[sy] += lv[sy] & 1;
        // End in sight: when every live system's estimate, carried one iteration further by its
        // last reduction factor, is within twice its target, wait for iteration q + 1 (already
        // enqueued) before enqueueing q + 2.  If q + 1 ends the solve, no empty iteration
        // follows it; otherwise the GPU idles only while the host enqueues q + 2.
        if (lag == 1) {
            const double *es = slot_est(q);
            bool near = true;
            for (int sy = 0; sy < S; ++sy) {
                if (!(lv[sy] & 1)) continue;
                const double e = es[sy], e0 = prev_est[sy];
                near = near && e0 > 0.0 && std::isfinite(e) && e * (e / e0) <= 2.0 * target[sy];
            }
            for (int sy = 0; sy < S; ++sy) prev_est[sy] = es[sy];
            if (near) {
                MFS_HIP_TRY(hipEventSynchronize(p->stat_ev[(q + 1) % mfs_plan_s::STAT_SLOTS]));
                if (!slot_err(q + 1)) {  // an error is reported by the regular read of q + 1
                    const int32_t *l2 = slot_flag(q + 1);
                    int live2 = 0;
                    for (int sy = 0; sy < S; ++sy) live2 += l2[sy] & 1;
                    if (live2 == 0) break;
                }
            }
        }
    }
    // drain, then the final status and x += V y with y from the device back substitution
    MFS_HIP_TRY(hipStreamSynchronize(s));
    // the matvec of an empty tail iteration skipped every pair: keep its launch out of the
    // pair-kernel timing (it is the last launch the timer recorded)
    if (empty_tail && p->timing && A == matvec_impl && p->timer[prec].used > 0) --p->timer[prec].used;
    if (slot_err(done - 1)) return fail(MFS_ENUMERIC, "non-finite Arnoldi vector");
    const double *es = slot_est(done - 1);
    for (int sy = 0; sy < S; ++sy)
        if (act[sy]) est[sy] = es[sy];
    MFS_TRY(launch_givens_solve(st, p->coef.as<double>(), ldh, done, s));
    MFS_TRY(launch_multi_axpy(nc, p->chunks.as<VecChunk>(), V, n, done, p->coef.as<double>(), ldh, 1.0, x, s));
    MFS_HIP_TRY(hipStreamSynchronize(s));
    return MFS_OK;
}

int gmres_solve_impl(mfs_plan p, const double *b, double *x, double tol, int max_iter, int max_refine, bool adjoint,
                     int32_t *iters, double *relres, hipStream_t s) {
    MFS_TRY(ensure_krylov(p, max_iter));
    MatvecFn A = adjoint ? matvec_adjoint_impl : matvec_impl;
    const int S = (int)p->n_sys;
    const int64_t n = p->n_gamma;
    std::vector<double> bn;
    MFS_TRY(sys_norms(p, b, bn, s));
    for (int sy = 0; sy < S; ++sy)
        if (!std::isfinite(bn[sy])) return fail(MFS_ENUMERIC, "non-finite right-hand side");
    std::vector<double> target(S), est(S), rn(S, 0.0);
    std::vector<int> counts(S, 0), active(S, 1), checks(S, 0);
    for (int sy = 0; sy < S; ++sy)
        if (bn[sy] == 0.0) active[sy] = 0;  // b = 0: gamma = 0 is exact, nothing to iterate or check
    p->prog_bnorm = bn;
    p->stop_requested = false;
    MFS_TRY(launch_fill(n, 0.0, x, s));
    double *r = p->R.as<double>();
    MFS_HIP_TRY(hipMemcpyAsync(r, b, n * sizeof(double), hipMemcpyDeviceToDevice, s));
    // both precisions iterate until the residual is below stop_factor * tol
    // (mfs_plan_set_stop_factor): the relative residual bounds the outputs' error
    // only up to the conditioning, and the margin keeps them within tol of the exact
    // solution.  In a mixed plan the FP64 true residual can sit above the mixed
    // GMRES estimate (by about 1e-6 of |b| at 1000 ellipsoids), so a system whose
    // true residual is above stop_factor * tol restarts from its iterate and reduces
    // that residual by stop_factor again (iterative refinement); its status is
    // MFS_OK once the true residual is at most tol
    const double inner = p->stop_factor;
    for (int sy = 0; sy < S; ++sy) target[sy] = inner * tol * bn[sy];
    int status = MFS_OK;
    if (p->prec == MFS_FP64) {
        MFS_TRY(gmres_attempt(p, A, MFS_FP64, r, x, target, max_iter, active, counts, est, bn, s));
        for (int sy = 0; sy < S; ++sy) {
            rn[sy] = est[sy];
            if (!(est[sy] <= tol * bn[sy])) status = MFS_NOT_CONVERGED;
        }
    } else {
        std::vector<double> rnorm = bn;  // norms of r = b - A x, here with x = 0
        for (int attempt = 0; attempt <= max_refine; ++attempt) {
            if (std::find(active.begin(), active.end(), 1) == active.end()) break;
            MFS_TRY(gmres_attempt(p, A, MFS_MIXED, r, x, target, max_iter, active, counts, est, rnorm, s));
            // true residual in FP64 (the attempt ended with a synchronisation, so the pinned
            // mask buffer is free)
            std::copy(active.begin(), active.end(), p->h_act);
            MFS_HIP_TRY(hipMemcpyAsync(p->sys_active.ptr, p->h_act, S * sizeof(int32_t), hipMemcpyHostToDevice, s));
            MFS_TRY(A(p, x, p->Wv.as<double>(), MFS_FP64, p->sys_active.as<int32_t>(), s));
            for (int sy = 0; sy < S; ++sy) {
                counts[sy] += active[sy];
                checks[sy] += active[sy];
            }
            MFS_TRY(launch_sub(n, b, p->Wv.as<double>(), r, s));
            std::vector<double> &tn = rnorm;
            MFS_TRY(sys_norms(p, r, tn, s));
            bool all = true;
            for (int sy = 0; sy < S; ++sy) {
                if (!active[sy]) continue;
                if (!std::isfinite(tn[sy])) return fail(MFS_ENUMERIC, "non-finite residual");
                rn[sy] = tn[sy];
                if (tn[sy] <= inner * tol * bn[sy]) active[sy] = 0;
                else all = false;
            }
            if (all || p->stop_requested) break;
            // restart from x on the true residual: solve A dx = r until its residual is
            // below stop_factor * min(tol |b|, |r|)
            for (int sy = 0; sy < S; ++sy) target[sy] = inner * std::min(tol * bn[sy], tn[sy]);
            // gmres_attempt adds into x directly
        }
        for (int sy = 0; sy < S; ++sy)
            if (!(rn[sy] <= tol * bn[sy])) status = MFS_NOT_CONVERGED;
    }
    p->last_mixed.assign(S, 0);
    p->last_fp64.assign(S, 0);
    for (int sy = 0; sy < S; ++sy) {
        if (iters) iters[sy] = counts[sy];
        if (relres) relres[sy] = bn[sy] > 0 ? rn[sy] / bn[sy] : 0.0;
        (p->prec == MFS_MIXED ? p->last_mixed : p->last_fp64)[sy] = counts[sy] - checks[sy];
        if (p->prec == MFS_MIXED) p->last_fp64[sy] = checks[sy];
    }
    if (status == MFS_NOT_CONVERGED) set_error("GMRES: some system did not reach the tolerance");
    return status;
}

}  // namespace

extern "C" {

int mfs_gmres_solve(mfs_plan p, const double *b, double *gamma, double tol, int32_t max_iter, int32_t max_refine,
                    int32_t adjoint, int32_t *iters, double *relres, void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (!b || !gamma) return fail(MFS_EINVAL, "NULL b or gamma");
    if (b == gamma) return fail(MFS_EINVAL, "b and gamma must not alias");
    if (!(tol > 0.0) || !std::isfinite(tol)) return fail(MFS_EINVAL, "tol must be finite and > 0");
    if (max_iter < 1 || max_iter > 2000) return fail(MFS_EINVAL, "max_iter must be in [1, 2000]");
    if (max_refine < 0 || max_refine > 100) return fail(MFS_EINVAL, "max_refine must be in [0, 100]");
    return gmres_solve_impl(p, b, gamma, tol, max_iter, max_refine, adjoint != 0, iters, relres, (hipStream_t)stream);
}

}  // extern "C"

// ---------------------------------------------------------------------------
// gradient of J(out) with respect to the centres
// ---------------------------------------------------------------------------
extern "C" int mfs_plan_set_progress(mfs_plan p, mfs_progress_fn fn, void *user) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    p->progress = fn;
    p->progress_user = user;
    return MFS_OK;
}

extern "C" int mfs_gmres_solve_backward(mfs_plan p, const double *gamma, const double *strength0,
                                        const double *grad_out, double *grad_centre, double *grad_net, double tol,
                                        int32_t max_iter, int32_t max_refine, int32_t *iters, double *relres,
                                        void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (p->formulation != MFS_MOBILITY)
        return fail(MFS_EUNSUPPORTED, "gradients are defined for the mobility / elastance formulation");
    if (!gamma || !grad_out) return fail(MFS_EINVAL, "NULL gamma or grad_out");
    if (!grad_centre && !grad_net) return fail(MFS_EINVAL, "neither grad_centre nor grad_net requested");
    if (grad_centre && !strength0)
        return fail(MFS_EINVAL, "strength0 is required for grad_centre (the pair terms carry (I - L) lambda + s_0)");
    if (!(tol > 0.0) || !std::isfinite(tol)) return fail(MFS_EINVAL, "tol must be finite and > 0");
    if (max_iter < 1 || max_iter > 2000) return fail(MFS_EINVAL, "max_iter must be in [1, 2000]");
    if (max_refine < 0 || max_refine > 100) return fail(MFS_EINVAL, "max_refine must be in [0, 100]");
    hipStream_t s = (hipStream_t)stream;
    const int prec = p->prec;
    MFS_TRY(p->bw_sigma.reserve(std::max<int64_t>(1, p->n_lambda) * sizeof(double)));
    MFS_TRY(p->bw_glam.reserve(std::max<int64_t>(1, p->n_lambda) * sizeof(double)));
    MFS_TRY(p->bw_g.reserve(std::max<int64_t>(1, p->n_gamma) * sizeof(double)));
    MFS_TRY(p->bw_w.reserve(std::max<int64_t>(1, p->n_gamma) * sizeof(double)));
    MFS_TRY(p->bw_gt.reserve(std::max<int64_t>(1, 3 * p->n_trgp) * sizeof(double)));
    MFS_TRY(p->bw_gs.reserve(std::max<int64_t>(1, 3 * p->n_srcp) * sizeof(double)));
    BodyView bv = p->view();
    // sigma = (I - L) S_L^+ gamma + s0 (FP64)
    if (grad_centre) {
        MFS_TRY(precond_fwd(p, gamma, MFS_FP64, false, p->ws_l64c.as<double>(), -1, s));
        MFS_TRY(launch_extract(bv, p->ws_l64c.as<double>(), strength0, nullptr, p->bw_sigma.as<double>(), s));
    }
    // g = (S_L^+)^T dJ/dlambda
    MFS_TRY(launch_grad_lambda(bv, grad_out, p->bw_glam.as<double>(), s));
    MFS_TRY(precond_tr(p, p->bw_glam.as<double>(), MFS_FP64, false, p->bw_g.as<double>(), s));
    // A^T w = g
    int st = gmres_solve_impl(p, p->bw_g.as<double>(), p->bw_w.as<double>(), tol, max_iter, max_refine, true, iters,
                              relres, s);
    if (st < 0) return st;
    MFS_TRY(set_tr_strength(p, p->bw_w.as<double>(), prec, s));
    if (grad_centre) {
        // d(w^T R)/dx_i over off-body pairs (lanes: collocation points with w; sources: proxies with sigma)
        MFS_TRY(set_fwd_strength(p, p->bw_sigma.as<double>(), prec, s));
        P2PLaunch Lf = fwd_launch(p, prec);
        Lf.skip_same = true;
        Lf.alpha = -1.0;
        Lf.out = p->bw_gt.as<double>();
        Lf.n_val = 3 * p->n_trgp;
        MFS_TRY(launch_p2p_grad(p->p2p_fwd1, Lf, p->bw_w.as<double>(), p->n_trgp, s));
        // d(w^T R)/dy_j (lanes: proxies with sigma; sources: collocation points with w)
        P2PLaunch Lt = tr_launch(p, prec);
        Lt.skip_same = true;
        Lt.alpha = -1.0;
        Lt.out = p->bw_gs.as<double>();
        Lt.n_val = 3 * p->n_srcp;
        MFS_TRY(launch_p2p_grad(p->p2p_tr1, Lt, p->bw_sigma.as<double>(), p->n_srcp, s));
        MFS_TRY(launch_body_grad_reduce(p->n_body, p->d_trg_row32.as<int32_t>(), p->d_src_row32.as<int32_t>(),
                                        p->bw_gt.as<double>(), p->bw_gs.as<double>(), grad_centre, s));
    }
    if (grad_net) {
        // dJ/ds_0 = -sum_k S^(kk')T w^(k) over every pair of the system, self block
        // included (b = -u_0 sums them all), then the chain rule through s_0(net)
        P2PLaunch Ln = tr_launch(p, prec);
        Ln.skip_same = false;
        Ln.alpha = -1.0;
        Ln.out = p->ws_l64c.as<double>();
        MFS_TRY(launch_p2p(tr_items(p, prec), Ln, s));
        MFS_TRY(launch_grad_net(bv, p->ws_l64c.as<double>(), grad_net, s));
    }
    MFS_HIP_TRY(hipStreamSynchronize(s));
    return st;
}

// ---------------------------------------------------------------------------
// instrumentation
// ---------------------------------------------------------------------------
extern "C" int mfs_plan_set_timing(mfs_plan p, int32_t enable) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    p->timing = enable != 0;
    return MFS_OK;
}

extern "C" int mfs_plan_timing(mfs_plan p, int32_t prec, int32_t reset, int64_t *launches, double *total_ms,
                               double *pairs_per_launch) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    MFS_TRY(check_prec(prec));
    MFS_TRY(harvest_timer(p, prec));
    auto &t = p->timer[prec];
    if (launches) *launches = t.launches;
    if (total_ms) *total_ms = t.total_ms;
    if (pairs_per_launch) *pairs_per_launch = p->offbody_pairs;
    if (reset) {
        t.launches = 0;
        t.total_ms = 0.0;
    }
    return MFS_OK;
}

// ---------------------------------------------------------------------------
// options: graphs and autotuning
// ---------------------------------------------------------------------------
extern "C" int mfs_plan_set_stop_factor(mfs_plan p, double factor) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (!(factor > 0.0 && factor <= 1.0)) return fail(MFS_EINVAL, "stop factor must be in (0, 1]");
    p->stop_factor = factor;
    return MFS_OK;
}

extern "C" int mfs_plan_set_graph(mfs_plan p, int32_t enable) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    p->use_graph = enable != 0;
    return MFS_OK;
}

// Times candidate launch shapes of the matvec pair sum (targets per lane x
// number of work items, which sets the source split) with HIP events on
// `stream` and keeps the fastest for the forward and transposed sums.
// Grows the pair-sum partial workspace to at least n doubles, keeping every other
// buffer (the caller has synchronised; graphs are re-captured afterwards).
int grow_partial(mfs_plan p, int64_t n) {
    if ((size_t)n * sizeof(double) <= p->partial.bytes) return MFS_OK;
    return p->partial.reserve((size_t)n * sizeof(double));
}

extern "C" int mfs_plan_autotune(mfs_plan p, int32_t prec, int32_t reps, int32_t *best_tpl,
                                 int32_t *best_min_items, double *best_ms, void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    MFS_TRY(check_prec(prec));
    if (reps < 1 || reps > 100) return fail(MFS_EINVAL, "reps must be in [1, 100]");
    hipStream_t s = (hipStream_t)stream;
    std::vector<int64_t> src_row(p->src_row), trg_row(p->trg_row);
    struct Events {  // destroyed on every return path
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events() {
            for (auto x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } ev;
    MFS_HIP_TRY(hipEventCreate(&ev.e[0]));
    MFS_HIP_TRY(hipEventCreate(&ev.e[1]));
    hipEvent_t e0 = ev.e[0], e1 = ev.e[1];
    double best = 1e300;
    int btpl = p->tuned_tpl, bmi = p->tuned_min_items;
    // the shapes listed and the plan's own, so that tuning never ends in a slower one
    struct Shape { int tpl, mi, per; };
    const Shape own{p->tuned_tpl, p->tuned_min_items, p->tuned_persistent ? 1 : 0};
    std::vector<Shape> shapes;
    for (int per = 0; per < 2; ++per)
        for (int tpl = 1; tpl <= 2; ++tpl)
            for (int mi = 1024; mi <= 16384; mi *= 2) shapes.push_back(Shape{tpl, mi, per});
    size_t own_at = 0;
    while (own_at < shapes.size() && (shapes[own_at].tpl != own.tpl || shapes[own_at].mi != own.mi || shapes[own_at].per != own.per))
        ++own_at;
    if (own_at == shapes.size()) shapes.push_back(own);
    bool bper = own.per != 0;
    struct Cand { double ms; int n_split; size_t n_items; Shape sh; };
    std::vector<Cand> timed;
    for (const Shape &sh : shapes) {
        P2PPlan cand;
        MFS_TRY(build_p2p_items(cand, p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                                p->gam_off.data(), p->kind.data(), p->mu, sh.tpl, sh.mi, s,
                                prec == MFS_MIXED && p->far_fwd.use && sh.tpl == 1));
        cand.persistent = sh.per != 0;
        const int64_t need = (cand.n_split > 1 ? cand.n_split : 1) * std::max<int64_t>(1, p->n_gamma);
        if ((size_t)need * sizeof(double) > p->partial.bytes) {
            MFS_HIP_TRY(hipStreamSynchronize(s));
            MFS_TRY(grow_partial(p, need));
        }
        P2PLaunch L = fwd_launch(p, prec);
        L.skip_same = true;
        L.out = p->ws_g64.as<double>();
        MFS_TRY(launch_p2p(cand, L, s));  // warm-up
        MFS_HIP_TRY(hipEventRecord(e0, s));
        for (int r = 0; r < reps; ++r) MFS_TRY(launch_p2p(cand, L, s));
        MFS_HIP_TRY(hipEventRecord(e1, s));
        MFS_HIP_TRY(hipEventSynchronize(e1));
        float ms = 0.f;
        MFS_HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
        timed.push_back(Cand{ms / reps, std::max(cand.n_split, 1), cand.items.size(), sh});
    }
    // the fastest shape; among shapes within 1.5% of it (timing noise), the one with the fewest
    // source splits (fewer FP64 slices written and re-read), then the fewest work items; none that is
    // slower than the plan's own (the longest time of the listed shapes that make the same launch)
    const Cand mine = timed[own_at];
    double own_ms = mine.ms;
    for (const Cand &c : timed) {
        best = std::min(best, c.ms);
        if (c.sh.tpl == own.tpl && c.sh.per == own.per && c.n_split == mine.n_split && c.n_items == mine.n_items)
            own_ms = std::max(own_ms, c.ms);
    }
    const Cand *pick = nullptr;
    for (const Cand &c : timed)
        if (c.ms <= std::min(1.015 * best, own_ms) &&
            (!pick || c.n_split < pick->n_split || (c.n_split == pick->n_split && c.sh.mi < pick->sh.mi)))
            pick = &c;
    if (pick) {
        btpl = pick->sh.tpl;
        bmi = pick->sh.mi;
        bper = pick->sh.per != 0;
        best = pick->ms;
    }
    p->tuned_tpl = btpl;
    p->tuned_min_items = bmi;
    MFS_TRY(build_p2p_items(p->p2p_fwd, p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                            p->gam_off.data(), p->kind.data(), p->mu, btpl, bmi, s));
    MFS_TRY(build_p2p_items(p->p2p_tr, p->n_sys, p->sys_body_ptr.data(), src_row.data(), trg_row.data(),
                            p->lam_off.data(), p->kind.data(), p->mu, btpl, bmi, s));
    MFS_TRY(build_far_items(p, bmi, bper, s));
    p->p2p_fwd.persistent = p->p2p_tr.persistent = bper;
    p->tuned_persistent = bper;
    MFS_HIP_TRY(hipStreamSynchronize(s));
    MFS_TRY(grow_partial(p, (int64_t)std::max({p->p2p_fwd.n_split, p->far_fwd.items.n_split, 1}) *
                                std::max<int64_t>(1, p->n_gamma)));
    MFS_TRY(grow_partial(p, (int64_t)std::max({p->p2p_tr.n_split, p->far_tr.items.n_split, 1}) *
                                std::max<int64_t>(1, p->n_lambda)));
    // captured graphs hold the old work tables and buffers
    for (auto &row : p->graph)
        for (auto &g : row)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
    MFS_HIP_TRY(hipStreamSynchronize(s));
    if (best_tpl) *best_tpl = bper ? -btpl : btpl;
    if (best_min_items) *best_min_items = bmi;
    if (best_ms) *best_ms = best;
    return MFS_OK;
}

extern "C" int mfs_plan_last_solve(mfs_plan p, int32_t *mixed_matvecs, int32_t *fp64_matvecs) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    for (int64_t sy = 0; sy < p->n_sys; ++sy) {
        const bool have = (size_t)sy < p->last_mixed.size();
        if (mixed_matvecs) mixed_matvecs[sy] = have ? p->last_mixed[sy] : 0;
        if (fp64_matvecs) fp64_matvecs[sy] = have ? p->last_fp64[sy] : 0;
    }
    return MFS_OK;
}

extern "C" int mfs_plan_set_launch(mfs_plan p, int32_t targets_per_lane, int32_t work_items, int32_t persistent,
                                   void *stream) {
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    if (targets_per_lane != 1 && targets_per_lane != 2) return fail(MFS_EINVAL, "targets_per_lane must be 1 or 2");
    if (work_items < 1 || work_items > (1 << 20)) return fail(MFS_EINVAL, "work_items must be in [1, 2^20]");
    hipStream_t s = (hipStream_t)stream;
    std::vector<int64_t> src_row(p->src_row), trg_row(p->trg_row);
    MFS_HIP_TRY(hipStreamSynchronize(s));
    MFS_TRY(build_p2p_items(p->p2p_fwd, p->n_sys, p->sys_body_ptr.data(), trg_row.data(), src_row.data(),
                            p->gam_off.data(), p->kind.data(), p->mu, targets_per_lane, work_items, s));
    MFS_TRY(build_p2p_items(p->p2p_tr, p->n_sys, p->sys_body_ptr.data(), src_row.data(), trg_row.data(),
                            p->lam_off.data(), p->kind.data(), p->mu, targets_per_lane, work_items, s));
    MFS_TRY(build_far_items(p, work_items, persistent != 0, s));
    p->p2p_fwd.persistent = p->p2p_tr.persistent = persistent != 0;
    MFS_TRY(grow_partial(p, (int64_t)std::max({p->p2p_fwd.n_split, p->far_fwd.items.n_split, 1}) *
                                std::max<int64_t>(1, p->n_gamma)));
    MFS_TRY(grow_partial(p, (int64_t)std::max({p->p2p_tr.n_split, p->far_tr.items.n_split, 1}) *
                                std::max<int64_t>(1, p->n_lambda)));
    for (auto &row : p->graph)
        for (auto &g : row)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
    MFS_HIP_TRY(hipStreamSynchronize(s));
    p->tuned_tpl = targets_per_lane;
    p->tuned_min_items = work_items;
    p->tuned_persistent = persistent != 0;
    return MFS_OK;
}

extern "C" int mfs_surface_residual(mfs_plan p, const double *sigma, const double *motion,
                                    const int32_t *shape_n_test, const double *shape_test, double *eps, double *u_test,
                                    int prec, void *stream) {
    using namespace mfs;
    if (!p) return fail(MFS_EINVAL, "NULL plan");
    MFS_TRY(check_prec(prec));
    if (!sigma || !motion || !shape_n_test || !shape_test || !eps) return fail(MFS_EINVAL, "NULL argument");
    const int64_t nb = p->n_body;
    std::vector<int64_t> so(p->n_shape + 1, 0);
    for (int64_t sh = 0; sh < p->n_shape; ++sh) {
        if (shape_n_test[sh] < 0) return fail(MFS_EINVAL, "negative test point count");
        so[sh + 1] = so[sh] + shape_n_test[sh];
    }
    for (int64_t q = 0; q < 3 * so[p->n_shape]; ++q)
        if (!std::isfinite(shape_test[q])) return fail(MFS_EINVAL, "non-finite test point");
    // test points of every body in world axes relative to its centre, body by body
    std::vector<int64_t> tptr(nb + 1, 0), uptr(nb + 1, 0);
    for (int64_t b = 0; b < nb; ++b) {
        const int64_t m = shape_n_test[p->shape_of_body[b]];
        tptr[b + 1] = tptr[b] + m;
        uptr[b + 1] = uptr[b] + (p->kind[b] == MFS_STOKES ? 3 : 1) * m;
    }
    const int64_t n = tptr[nb], nu = uptr[nb];
    if (n == 0) return MFS_OK;
    if (n > INT32_MAX / 2) return fail(MFS_EINVAL, "too many test points");
    std::vector<double> o64(4 * n);
    std::vector<float> o32(4 * n);
    std::vector<int32_t> tb(n);
    std::vector<int64_t> uoff(n);
    for (int64_t b = 0; b < nb; ++b) {
        const double *R = p->rot_h.data() + 9 * b;
        const double *loc = shape_test + 3 * so[p->shape_of_body[b]];
        const int dim = p->kind[b] == MFS_STOKES ? 3 : 1;
        for (int64_t i = tptr[b]; i < tptr[b + 1]; ++i) {
            const double *q = loc + 3 * (i - tptr[b]);
            for (int a = 0; a < 3; ++a) {
                const double v = R[3 * a] * q[0] + R[3 * a + 1] * q[1] + R[3 * a + 2] * q[2];
                o64[4 * i + a] = v;
                o32[4 * i + a] = (float)v;
            }
            o64[4 * i + 3] = 0.0;
            o32[4 * i + 3] = 0.f;
            tb[i] = (int32_t)b;
            uoff[i] = uptr[b] + dim * (i - tptr[b]);
        }
    }
    hipStream_t s = (hipStream_t)stream;
    DevBuf d_o64, d_o32, d_tb, d_uoff, d_u, d_part;
    MFS_TRY(upload_vec(d_o64, o64, s));
    MFS_TRY(upload_vec(d_o32, o32, s));
    MFS_TRY(upload_vec(d_tb, tb, s));
    MFS_TRY(upload_vec(d_uoff, uoff, s));
    double *u = u_test;
    if (!u) {
        MFS_TRY(d_u.reserve(nu * sizeof(double)));
        u = d_u.as<double>();
    }
    // the representation with the full strengths over all proxies, self included
    MFS_TRY(set_fwd_strength(p, sigma, prec, s));
    std::vector<int64_t> src_row(p->src_row);
    P2PPlan pp;
    // items for this one call: making and sorting more of them costs more than it gains (40 Stokes bodies of
    // 1000 test points: 518 us with 2048 items, 569 with default_min_items' 6700)
    MFS_TRY(build_p2p_items(pp, p->n_sys, p->sys_body_ptr.data(), tptr.data(), src_row.data(), uptr.data(),
                            p->kind.data(), p->mu, 1, 2048, s, p->far_fwd.use && prec == MFS_MIXED));
    P2PLaunch L = fwd_launch(p, prec);
    L.trg_off = prec == MFS_MIXED ? d_o32.ptr : d_o64.ptr;
    L.trg_body = d_tb.as<int32_t>();
    L.skip_same = false;
    L.out = u;
    L.n_val = nu;
    if (pp.n_split > 1) {
        MFS_TRY(d_part.reserve((size_t)pp.n_split * nu * sizeof(double)));
        L.partial = d_part.as<double>();
    }
    MFS_TRY(launch_p2p(pp, L, s));
    MFS_TRY(launch_residual(n, d_tb.as<int32_t>(), p->d_kind.as<int32_t>(), p->d_net_off.as<int64_t>(),
                            d_o64.as<double>(), u, d_uoff.as<int64_t>(), motion, eps, s));
    MFS_HIP_TRY(hipStreamSynchronize(s));
    return MFS_OK;
}
