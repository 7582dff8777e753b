// Host side of libspamm.so: argument checks, workspace layout, and the
// enqueueing of the kernels of the SpAMM hot path on the caller's stream.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "spamm.h"
#include "spamm_noalloc.h"
#include "dma.h"
#include "host.h"
#include "internal.h"
#include "search.h"

namespace spamm_host {


thread_local char g_last_error[512] = "";

spamm_status fail(spamm_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
    return st;
}

spamm_status hip_check(hipError_t e, const char* what) {
    if (e == hipSuccess) return SPAMM_OK;
    return fail(SPAMM_EDEVICE, "%s: %s (%d)", what, hipGetErrorString(e), int(e));
}

bool make_geom(int64_t n, int32_t leaf, Geom* g) {
    if (n <= 0 || leaf <= 0 || leaf > 1024) return false;
    g->n = n;
    g->leaf = leaf;
    g->bdim = (n + leaf - 1) / leaf;
    int32_t lv = 0;
    while ((int64_t(1) << lv) < g->bdim) ++lv;
    g->lv = lv;
    g->side = int64_t(1) << lv;
    g->ntiles = g->bdim * g->bdim;
    g->pyr = spamm::level_offset(lv + 1);
    g->nwords = int32_t((g->bdim + 63) / 64);
    return true;
}

namespace {
constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
}  // namespace

namespace {
// lean: ragged sizes without the regions that only speed them up
Layout layout_of(const Geom& g, bool lean) {
    Layout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    for (int m = 0; m < 2; ++m) L.spyr[m] = take(sizeof(double) * size_t(g.pyr));
    for (int m = 0; m < 2; ++m) L.pyr[m] = take(sizeof(double) * size_t(g.pyr));
    L.counts = take(sizeof(int32_t) * size_t(g.ntiles));
    L.bsums = take(sizeof(int32_t) * size_t(g.bdim) * size_t(g.nwords));
    L.boffs = take(sizeof(int32_t) * size_t(g.bdim) * size_t(g.nwords));
    L.masks = take(sizeof(uint64_t) * size_t(g.ntiles) * size_t(g.nwords));
    L.offsets = take(sizeof(int32_t) * size_t(g.ntiles + 1));
    L.klist = take(sizeof(int32_t) * size_t(g.ntiles) * size_t(g.bdim));
    L.pair_scratch = take(sizeof(int32_t) * size_t(g.ntiles) * size_t(g.bdim));
    const size_t nm = size_t((g.bdim + 1) / 2) * size_t((g.bdim + 1) / 2);
    L.mwords = take(sizeof(uint64_t) * nm * 4 * size_t(g.nwords));
    L.mcount = take(sizeof(int32_t) * nm);
    L.mprefix = take(sizeof(int32_t) * (nm + 1));
    L.mitems = take(sizeof(uint32_t) * nm * size_t(g.bdim));
    // leaf 128 on the LDS-DMA kernel: two items per kept pair, their prefix
    const bool l128 = g.leaf == 128 && !lean && g.n >= 4 && g.bdim <= spamm::kLeaf128MaxBdim;
    L.leaf128_dma = l128;
    L.items128 = take(l128 ? sizeof(uint32_t) * 2 * size_t(g.ntiles) * size_t(g.bdim) : 0);
    L.uprefix128 = take(l128 ? sizeof(int32_t) * size_t(g.ntiles + 1) : 0);
    L.bounds = take(sizeof(int64_t) * 4 * spamm::kSplitMaxGroups);
    // partial sums of shared macro tiles (LDS-DMA kernel: leaf 64 or 128), two
    // slots per workgroup, at most one workgroup per macro tile
    const bool dma = (g.leaf == 64 && !lean) || l128;
    const size_t macros = l128 ? size_t(g.ntiles) : nm;
    const size_t groups =
        macros < size_t(spamm::kSplitMaxGroups) ? (macros + 7) / 8 * 8 : size_t(spamm::kSplitMaxGroups);
    L.fix_slot_bytes = dma ? sizeof(float) * groups * 2 * spamm::kSplitSlotFloats : 0;
    L.fix_slots = take(L.fix_slot_bytes);
    L.pm_state = take(sizeof(int64_t) * size_t(spamm::plan_macro_clear_words(g.bdim)));
    L.pairs = take(sizeof(int64_t));
    L.form = take(sizeof(int32_t));
    L.partials = take(sizeof(double) * 1024);
    L.total = o;
    return L;
}
}  // namespace

// The LDS-DMA kernel's regions (up to 32 MiB of partial sums, leaf 128's item
// list) are left out for a ragged size that fits the static scratch of
// spamm_multiply_noalloc only without them: its macro tiles are then not
// shared between workgroups (leaf 64), or it takes the single-tile kernel
// (leaf 128).  The choice is by size alone, so that every workspace of a size
// takes the same route.
Layout make_layout(const Geom& g) {
    const Layout full = layout_of(g, false);
    if (g.n % 128 == 0 || full.total <= size_t(SPAMM_NOALLOC_SCRATCH_BYTES)) return full;
    const Layout lean = layout_of(g, true);
    return lean.total <= size_t(SPAMM_NOALLOC_SCRATCH_BYTES) ? lean : full;
}

bool search_regions(const Geom& g, SearchRegions* out) {
    const Layout L = make_layout(g);
    const size_t bdim = size_t(g.bdim), nb = size_t((g.n + 63) / 64);
    const size_t starts[] = {L.spyr[0], L.spyr[1], L.pyr[0], L.pyr[1], L.counts, L.bsums, L.boffs, L.masks,
                             L.offsets, L.klist, L.pair_scratch, L.mwords, L.mcount, L.mprefix, L.mitems,
                             L.items128, L.uprefix128, L.bounds, L.fix_slots, L.pm_state, L.pairs, L.form,
                             L.partials, L.total};
    bool fits = true;
    auto borrow = [&](size_t at, size_t bytes) {  // up to the next region's start
        for (const size_t next : starts) fits = fits && (next <= at || at + bytes <= next);
        return at;
    };
    SearchRegions R{};
    R.blocks = int64_t(nb * nb);
    const size_t norms = sizeof(double) * bdim * bdim;
    R.rows_b = borrow(L.spyr[0], norms);
    R.cols_a = borrow(L.spyr[1], norms);
    R.ksums = borrow(L.partials, sizeof(double) * bdim);
    const size_t probe = sizeof(int32_t) * bdim * spamm::kProbeStride;
    R.count_even = borrow(L.klist, probe);
    R.count_odd = borrow(L.pair_scratch, probe);
    R.states = borrow(L.bounds, 2 * sizeof(spamm::SearchState));
    R.partials = borrow(L.mwords, sizeof(double) * bdim * spamm::kQueryPartial);
    R.answer = borrow(L.offsets, sizeof(spamm::StepAnswer));
    // the k-list regions hold bdim^3 int32, too little for the sums only on
    // the smallest grids
    R.sums = borrow(nb <= 32 ? L.bounds : L.klist, sizeof(double) * nb * nb);
    R.counts = borrow(L.pair_scratch, sizeof(int32_t) * nb * nb);
    *out = R;
    return fits;
}

bool overlaps(const void* p, size_t pbytes, const void* q, size_t qbytes) {
    const char* a = static_cast<const char*>(p);
    const char* b = static_cast<const char*>(q);
    return a < b + qbytes && b < a + pbytes;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int device_cus() {
    static std::mutex mu;
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    std::lock_guard<std::mutex> lock(mu);
    if (cached[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        cached[dev] = cus;
    }
    return cached[dev];
}

spamm_status check_grid(const Geom& g) {
    if (g.bdim > SPAMM_MAX_BDIM)
        return fail(SPAMM_EUNSUPPORTED, "tile grid %lld exceeds %d per side", (long long)g.bdim, SPAMM_MAX_BDIM);
    return SPAMM_OK;
}

// Workspaces the library keeps for callers that pass none: one per device,
// grown to the largest size asked for, freed by spamm_release.
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_cache_mu;
void* g_cache_ptr[kMaxDevices] = {};
size_t g_cache_bytes[kMaxDevices] = {};
}  // namespace

spamm_status cached_workspace(size_t need, void** ws, size_t* bytes) {
    int dev = 0;
    spamm_status st = hip_check(hipGetDevice(&dev), "hipGetDevice");
    if (st != SPAMM_OK) return st;
    if (dev < 0 || dev >= kMaxDevices) return fail(SPAMM_EUNSUPPORTED, "device %d beyond the workspace cache", dev);
    std::lock_guard<std::mutex> lock(g_cache_mu);
    if (g_cache_bytes[dev] < need) {
        if (g_cache_ptr[dev]) {
            // the old buffer may still be in use by enqueued work
            if ((st = hip_check(hipDeviceSynchronize(), "synchronize before growing the cached workspace")) !=
                SPAMM_OK)
                return st;
            if ((st = hip_check(hipFree(g_cache_ptr[dev]), "hipFree of the cached workspace")) != SPAMM_OK)
                return st;
            g_cache_ptr[dev] = nullptr;
            g_cache_bytes[dev] = 0;
        }
        void* p = nullptr;
        if (hipMalloc(&p, need) != hipSuccess || !p) {
            (void)hipGetLastError();
            return fail(SPAMM_ENOSPACE, "cannot allocate a cached workspace of %zu bytes on device %d", need, dev);
        }
        g_cache_ptr[dev] = p;
        g_cache_bytes[dev] = need;
    }
    *ws = g_cache_ptr[dev];
    *bytes = g_cache_bytes[dev];
    return SPAMM_OK;
}

spamm_status release_cached_workspaces() {
    std::lock_guard<std::mutex> lock(g_cache_mu);
    int cur = 0;
    spamm_status st = hip_check(hipGetDevice(&cur), "hipGetDevice");
    if (st != SPAMM_OK) return st;
    for (int d = 0; d < kMaxDevices; ++d) {
        if (!g_cache_ptr[d]) continue;
        if ((st = hip_check(hipSetDevice(d), "hipSetDevice")) != SPAMM_OK) break;
        if ((st = hip_check(hipDeviceSynchronize(), "synchronize before releasing the cached workspace")) != SPAMM_OK)
            break;
        if ((st = hip_check(hipFree(g_cache_ptr[d]), "hipFree of the cached workspace")) != SPAMM_OK) break;
        g_cache_ptr[d] = nullptr;
        g_cache_bytes[d] = 0;
    }
    const spamm_status st2 = hip_check(hipSetDevice(cur), "hipSetDevice");
    return st != SPAMM_OK ? st : st2;
}

spamm_status check_workspace(const Geom& g, void*& ws, size_t& bytes) {
    const size_t need = make_layout(g).total;
    if (!ws) return cached_workspace(need, &ws, &bytes);
    if (bytes < need)
        return fail(SPAMM_ENOSPACE, "workspace of %zu bytes, %zu needed", bytes, need);
    return SPAMM_OK;
}

spamm_status check_tau(double tau) {
    if (std::isnan(tau) || tau < 0.0) return fail(SPAMM_EINVAL, "tau must be >= 0 (got %g)", tau);
    return SPAMM_OK;
}

spamm_status enqueue_pyramids(const Geom& g, const float* const* x, int nmat, double* const* pyr_out, void* ws,
                              hipStream_t s, int64_t* clear, int64_t clear_count, bool levels) {
    const Layout L = make_layout(g);
    const int64_t leaf_level = spamm::level_offset(g.lv);
    spamm::NormJob nj{};
    spamm::PyramidJob pj{};
    nj.ld = g.side;  // the norm pass writes the padded leaf level of both pyramids
    nj.clear = clear;
    nj.clear_count = clear_count;
    bool vec = (g.n % 4) == 0;
    for (int m = 0; m < nmat; ++m) {
        nj.x[m] = x[m];
        pj.spyr[m] = at<double>(ws, L.spyr[m]);
        pj.pyr[m] = pyr_out[m];
        nj.sumsq[m] = pj.spyr[m] + leaf_level;
        nj.norms[m] = pj.pyr[m] + leaf_level;
        vec = vec && aligned16(x[m]);
    }
    spamm_status st = hip_check(spamm::launch_leaf_norms(nj, nmat, g.n, g.leaf, vec, s), "leaf norm kernel");
    if (st != SPAMM_OK || !levels) return st;
    return hip_check(spamm::launch_pyramid(pj, nmat, g.bdim, g.lv, s), "pyramid kernel");
}

spamm_status enqueue_plan(const Geom& g, const double* pa, const double* pb, double tau, int32_t* offsets,
                          int32_t* klist, int64_t* pairs, void* ws, hipStream_t s) {
    const Layout L = make_layout(g);
    uint64_t* masks = at<uint64_t>(ws, L.masks);
    int32_t* counts = at<int32_t>(ws, L.counts);
    int32_t* bsums = at<int32_t>(ws, L.bsums);
    int32_t* boffs = at<int32_t>(ws, L.boffs);
    spamm_status st = hip_check(spamm::launch_plan_mask(pa, pb, g.bdim, g.lv, tau, masks, counts, bsums, s),
                                "plan mask kernel");
    if (st != SPAMM_OK) return st;
    st = hip_check(spamm::launch_plan_scan(bsums, g.bdim * g.nwords, boffs, offsets, g.ntiles, pairs, s),
                   "plan scan kernel");
    if (st != SPAMM_OK) return st;
    return hip_check(spamm::launch_plan_fill(masks, counts, boffs, g.bdim, offsets, klist, s), "plan fill kernel");
}

spamm_status enqueue_prepare(const Geom& g, const float* a, const float* b, double tau, int32_t* offsets,
                             int32_t* klist, int64_t* pairs, void* ws, hipStream_t s, bool schedule) {
    const Layout L = make_layout(g);
    double* pa = at<double>(ws, L.pyr[0]);
    double* pb = at<double>(ws, L.pyr[1]);
    const float* xs[2] = {a, b};
    double* ps[2] = {pa, pb};
    const bool fused = schedule && (g.leaf == 32 || g.leaf == 64) && g.bdim <= spamm::kPlanMacroMaxBdim;
    // the fused plan tests on the leaf norms alone: no pyramid levels above
    int64_t* state = at<int64_t>(ws, L.pm_state);
    spamm_status st = enqueue_pyramids(g, xs, 2, ps, ws, s, fused ? state : nullptr,
                                       fused ? spamm::plan_macro_clear_words(g.bdim) : 0, !fused);
    if (st != SPAMM_OK) return st;
    if (!fused) {
        if ((st = enqueue_plan(g, pa, pb, tau, offsets, klist, pairs, ws, s)) != SPAMM_OK) return st;
        return schedule ? enqueue_schedule(g, offsets, klist, ws, s) : SPAMM_OK;
    }
    const spamm::MacroSchedule ms = macro_schedule(L, ws);
    spamm::PlanMacroOut o{};
    o.offsets = offsets;
    o.klist = klist;
    o.pairs = pairs;
    o.uprefix = ms.uprefix;
    o.items = ms.items;
    o.flags = reinterpret_cast<unsigned long long*>(state);
    o.ticket = reinterpret_cast<unsigned int*>(state + (g.bdim + 1) / 2);
    const int64_t leaf_level = spamm::level_offset(g.lv);
    return hip_check(spamm::launch_plan_macro(pa + leaf_level, pb + leaf_level, g.side, g.bdim, tau, o, s),
                     "plan and schedule kernel");
}

spamm_status check_mul_args(const Geom& g, const float* a, const float* b, const float* c) {
    if (!a || !b || !c) return fail(SPAMM_EINVAL, "null matrix pointer");
    const size_t bytes = sizeof(float) * size_t(g.n) * size_t(g.n);
    if (overlaps(c, bytes, a, bytes) || overlaps(c, bytes, b, bytes))
        return fail(SPAMM_EINVAL, "C overlaps A or B");
    if (!spamm_leaf_supported(g.leaf))
        return fail(SPAMM_EUNSUPPORTED, "leaf %d has no multiply kernel (16, 32, 64, 128)", g.leaf);
    return SPAMM_OK;
}


spamm::MacroSchedule macro_schedule(const Layout& L, void* ws) {
    spamm::MacroSchedule ms{};
    ms.words = at<uint64_t>(ws, L.mwords);
    ms.ucount = at<int32_t>(ws, L.mcount);
    ms.uprefix = at<int32_t>(ws, L.mprefix);
    ms.items = at<uint32_t>(ws, L.mitems);
    ms.bounds = at<int64_t>(ws, L.bounds);
    ms.fix_slots = L.fix_slot_bytes ? at<float>(ws, L.fix_slots) : nullptr;
    return ms;
}

spamm_status enqueue_schedule(const Geom& g, const int32_t* offsets, const int32_t* klist, void* ws, hipStream_t s) {
    const Layout L = make_layout(g);
    if (g.leaf == 128) {
        if (!L.leaf128_dma) return SPAMM_OK;  // the single-tile kernel reads the plan directly
        return hip_check(spamm::launch_leaf128_schedule(offsets, klist, g.bdim, at<int32_t>(ws, L.uprefix128),
                                                        at<uint32_t>(ws, L.items128), s),
                         "leaf-128 schedule kernel");
    }
    if (g.leaf != 32 && g.leaf != 64) return SPAMM_OK;
    return hip_check(spamm::launch_macro_schedule(offsets, klist, g.bdim, macro_schedule(L, ws), s),
                     "macro schedule kernels");
}

spamm_status enqueue_multiply(const Geom& g, const float* a, const float* b, const int32_t* offsets,
                              const int32_t* klist, float* c, void* ws, hipStream_t s) {
    const bool vec = (g.n % 4) == 0 && aligned16(a) && aligned16(b);
    const Layout L = make_layout(g);
    if (g.n < 4 && g.leaf >= 64)  // one tile, smaller than the 16-byte copies of the LDS-DMA kernel: any leaf is one tile
        return hip_check(spamm::launch_multiply_leaf16(a, b, c, g.n, g.bdim, offsets, klist, vec, s),
                         "multiply kernel");
    if (L.leaf128_dma)
        return hip_check(spamm::launch_leaf128_multiply(a, b, c, g.n, g.bdim, at<int32_t>(ws, L.uprefix128),
                                                        at<uint32_t>(ws, L.items128), at<int64_t>(ws, L.bounds),
                                                        at<float>(ws, L.fix_slots), device_cus(), s),
                         "leaf-128 multiply kernels");
    if (g.leaf == 32)
        return hip_check(spamm::launch_block_plan32(a, b, c, g.n, g.bdim, at<uint32_t>(ws, L.mitems),
                                                    at<int32_t>(ws, L.mprefix), s),
                         "block multiply kernel");
    if (g.leaf == 64)
        return hip_check(spamm::launch_macro_multiply(a, b, c, g.n, g.bdim, offsets, macro_schedule(L, ws),
                                                      device_cus(), s),
                         "macro multiply kernel");
    return hip_check(spamm::launch_multiply(a, b, c, g.n, g.leaf, g.bdim, offsets, klist,
                                            at<int32_t>(ws, L.pair_scratch), vec, device_cus(), s),
                     "multiply kernel");
}

spamm_status enqueue_execute(const Geom& g, const float* a, const float* b, const int32_t* offsets,
                             const int32_t* klist, float* c, void* ws, hipStream_t s) {
    spamm_status st = enqueue_schedule(g, offsets, klist, ws, s);
    if (st != SPAMM_OK) return st;
    return enqueue_multiply(g, a, b, offsets, klist, c, ws, s);
}

namespace {
constexpr size_t kSplitHeaderBytes = 256;  // scale exponents and largest leaf norms
size_t plane_bytes(int64_t n) { return (size_t(n) * size_t(n) * 2 + 255) / 256 * 256; }
int split_planes(int32_t precision) { return precision == spamm::kPrecF16x3 ? 4 : 2; }

spamm::SplitLayout split_layout(void* split, int64_t n, int32_t precision) {
    char* base = static_cast<char*>(split);
    const size_t pb = plane_bytes(n);
    spamm::SplitLayout L{};
    L.exps = reinterpret_cast<int32_t*>(base);
    char* p = base + kSplitHeaderBytes;
    auto next = [&]() {
        uint16_t* q = reinterpret_cast<uint16_t*>(p);
        p += pb;
        return q;
    };
    L.a_hi = next();
    L.a_lo = precision == spamm::kPrecF16x3 ? next() : nullptr;
    L.bt_hi = next();
    L.bt_lo = precision == spamm::kPrecF16x3 ? next() : nullptr;
    return L;
}
}  // namespace

spamm_status check_lowp(const Geom& g, int32_t precision) {
    if (precision != spamm::kPrecBf16 && precision != spamm::kPrecF16x3)
        return fail(SPAMM_EINVAL, "precision %d is not a reduced-precision form (1: bf16, 2: f16x3)", precision);
    if (g.leaf != 64 || g.n % 128 != 0)
        return fail(SPAMM_EUNSUPPORTED, "reduced-precision products need leaf 64 and n a multiple of 128 (n=%lld "
                    "leaf=%d)", (long long)g.n, g.leaf);
    return check_grid(g);
}

}  // namespace spamm_host

using namespace spamm_host;

extern "C" {

int64_t spamm_bdim(int64_t n, int32_t leaf) {
    Geom g;
    return make_geom(n, leaf, &g) ? g.bdim : 0;
}

int32_t spamm_levels(int64_t n, int32_t leaf) {
    Geom g;
    return make_geom(n, leaf, &g) ? g.lv : 0;
}

int64_t spamm_pyramid_size(int64_t n, int32_t leaf) {
    Geom g;
    return make_geom(n, leaf, &g) ? g.pyr : 0;
}

int32_t spamm_leaf_supported(int32_t leaf) { return (leaf == 16 || leaf == 32 || leaf == 64 || leaf == 128) ? 1 : 0; }

spamm_status spamm_release(void) {
    g_last_error[0] = '\0';
    return release_cached_workspaces();
}

size_t spamm_workspace_bytes(int64_t n, int32_t leaf) {
    Geom g;
    if (!make_geom(n, leaf, &g) || g.bdim > SPAMM_MAX_BDIM) return 0;
    return make_layout(g).total;
}

spamm_status spamm_norms(const float* x, int64_t n, int32_t leaf, double* norms, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!x || !norms) return fail(SPAMM_EINVAL, "null pointer");
    spamm::NormJob nj{};
    nj.x[0] = x;
    nj.sumsq[0] = nullptr;
    nj.norms[0] = norms;
    nj.ld = g.bdim;
    const bool vec = (n % 4) == 0 && aligned16(x);
    return hip_check(spamm::launch_leaf_norms(nj, 1, n, leaf, vec, static_cast<hipStream_t>(stream)),
                     "leaf norm kernel");
}

spamm_status spamm_pyramid(const float* x, int64_t n, int32_t leaf, double* pyramid, void* workspace,
                           size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!x || !pyramid) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_grid(g);
    if (st != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    const float* xs[1] = {x};
    double* ps[1] = {pyramid};
    return enqueue_pyramids(g, xs, 1, ps, workspace, static_cast<hipStream_t>(stream));
}

spamm_status spamm_plan(const double* pyr_a, const double* pyr_b, int64_t n, int32_t leaf, double tau,
                        int32_t* offsets, int32_t* klist, int64_t klist_capacity, int64_t* pairs, void* workspace,
                        size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!pyr_a || !pyr_b || !offsets || !klist || !pairs) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_tau(tau);
    if (st != SPAMM_OK) return st;
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (klist_capacity < g.ntiles * g.bdim)
        return fail(SPAMM_ENOSPACE, "klist capacity %lld < bdim^3 = %lld", (long long)klist_capacity,
                    (long long)(g.ntiles * g.bdim));
    return enqueue_plan(g, pyr_a, pyr_b, tau, offsets, klist, pairs, workspace, static_cast<hipStream_t>(stream));
}

spamm_status spamm_execute(const float* a, const float* b, int64_t n, int32_t leaf, const int32_t* offsets,
                           const int32_t* klist, float* c, void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if (!offsets || !klist) return fail(SPAMM_EINVAL, "null plan pointer");
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    return enqueue_execute(g, a, b, offsets, klist, c, workspace, static_cast<hipStream_t>(stream));
}

spamm_status spamm_schedule(const int32_t* offsets, const int32_t* klist, int64_t n, int32_t leaf, void* workspace,
                            size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!offsets || !klist) return fail(SPAMM_EINVAL, "null plan pointer");
    if (!spamm_leaf_supported(leaf))
        return fail(SPAMM_EUNSUPPORTED, "leaf %d has no multiply kernel (16, 32, 64, 128)", leaf);
    spamm_status st = check_grid(g);
    if (st != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    return enqueue_schedule(g, offsets, klist, workspace, static_cast<hipStream_t>(stream));
}

spamm_status spamm_execute_scheduled(const float* a, const float* b, int64_t n, int32_t leaf, const int32_t* offsets,
                                     const int32_t* klist, float* c, void* workspace, size_t workspace_bytes,
                                     void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if (!offsets || !klist) return fail(SPAMM_EINVAL, "null plan pointer");
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    return enqueue_multiply(g, a, b, offsets, klist, c, workspace, static_cast<hipStream_t>(stream));
}

spamm_status spamm_prepare(const float* a, const float* b, int64_t n, double tau, int32_t leaf, int32_t* offsets,
                           int32_t* klist, int64_t klist_capacity, int64_t* pairs, void* workspace,
                           size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!a || !b || !offsets || !klist || !pairs) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_tau(tau);
    if (st != SPAMM_OK) return st;
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (klist_capacity < g.ntiles * g.bdim)
        return fail(SPAMM_ENOSPACE, "klist capacity %lld < bdim^3 = %lld", (long long)klist_capacity,
                    (long long)(g.ntiles * g.bdim));
    return enqueue_prepare(g, a, b, tau, offsets, klist, pairs, workspace, static_cast<hipStream_t>(stream), false);
}

spamm_status spamm_prepare_schedule(const float* a, const float* b, int64_t n, double tau, int32_t leaf,
                                    int32_t* offsets, int32_t* klist, int64_t klist_capacity, int64_t* pairs,
                                    void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!a || !b || !offsets || !klist || !pairs) return fail(SPAMM_EINVAL, "null pointer");
    if (!spamm_leaf_supported(leaf))
        return fail(SPAMM_EUNSUPPORTED, "leaf %d has no multiply kernel (16, 32, 64, 128)", leaf);
    spamm_status st = check_tau(tau);
    if (st != SPAMM_OK) return st;
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (klist_capacity < g.ntiles * g.bdim)
        return fail(SPAMM_ENOSPACE, "klist capacity %lld < bdim^3 = %lld", (long long)klist_capacity,
                    (long long)(g.ntiles * g.bdim));
    return enqueue_prepare(g, a, b, tau, offsets, klist, pairs, workspace, static_cast<hipStream_t>(stream), true);
}

namespace {
// The leaf norms of a and b into the workspace pyramids (norms[2]), with `sums`
// also their squares, which a pyramid is built from; *pairs = 0.
spamm_status enqueue_leaf_norms(const Geom& g, const float* a, const float* b, int64_t* pairs, bool sums,
                                double** norms, void* ws, hipStream_t s) {
    const Layout L = make_layout(g);
    const int64_t leaf_level = spamm::level_offset(g.lv);
    spamm::NormJob nj{};
    nj.ld = g.side;
    nj.clear = pairs;
    const float* xs[2] = {a, b};
    for (int m = 0; m < 2; ++m) {
        nj.x[m] = xs[m];
        nj.sumsq[m] = sums ? at<double>(ws, L.spyr[m]) + leaf_level : nullptr;
        nj.norms[m] = norms[m] = at<double>(ws, L.pyr[m]) + leaf_level;
    }
    const bool vec = (g.n % 4) == 0 && aligned16(a) && aligned16(b);
    return hip_check(spamm::launch_leaf_norms(nj, 2, g.n, g.leaf, vec, s), "leaf norm kernel");
}

// The leaf norm pass (which also clears the pair counter), then the threshold
// test and the multiply in one launch.
spamm_status enqueue_direct(const Geom& g, const float* a, const float* b, double tau, float* c, int64_t* pairs,
                           void* ws, hipStream_t s) {
    double* norms[2];
    const spamm_status st = enqueue_leaf_norms(g, a, b, pairs, false, norms, ws, s);
    if (st != SPAMM_OK) return st;
    if (g.leaf >= 32 && g.n <= spamm::kTileMaxN)
        return hip_check(spamm::launch_tile_multiply(a, b, c, g.n, g.leaf, norms[0], norms[1], g.side, tau, pairs, s),
                         "tile multiply kernel");
    if (g.leaf == 16 && g.n <= spamm::kSmallMaxN) {
        const bool vec = (g.n % 4) == 0 && aligned16(a) && aligned16(b);
        return hip_check(spamm::launch_small_multiply16(a, b, c, g.n, vec, g.bdim, norms[0], norms[1], g.side, tau,
                                                        pairs, s),
                         "small multiply kernel");
    }
    return hip_check(spamm::launch_block_test(a, b, c, g.n, g.leaf, g.bdim, norms[0], norms[1], g.side, tau, pairs,
                                              s),
                     "block multiply kernel");
}

// After the leaf norms: the choice of form and, where it falls on the planes, the
// planes, the plan with its schedule and the multiply (*pairs is the plan's).
spamm_status enqueue_planes(const Geom& g, const float* a, const float* b, spamm::FormChoice& choice,
                            const spamm::SplitLayout& SL, float* c, int64_t* pairs, void* ws, hipStream_t s) {
    const Layout L = make_layout(g);
    const spamm::MacroSchedule ms = macro_schedule(L, ws);
    const int32_t* run = choice.form;
    int32_t* offsets = at<int32_t>(ws, L.offsets);
    int32_t* klist = at<int32_t>(ws, L.klist);
    int64_t* state = at<int64_t>(ws, L.pm_state);
    choice.clear = state;
    choice.clear_count = spamm::plan_macro_clear_words(g.bdim);
    spamm_status st = hip_check(spamm::launch_split_choice(a, b, g.n, g.bdim, choice, SL, s), "split kernel");
    if (st != SPAMM_OK) return st;
    if (g.bdim <= spamm::kPlanMacroMaxBdim) {
        const spamm::PlanMacroOut o{offsets, klist, pairs, ms.uprefix, ms.items,
                                    reinterpret_cast<unsigned long long*>(state),
                                    reinterpret_cast<unsigned int*>(state + (g.bdim + 1) / 2), run};
        st = hip_check(spamm::launch_plan_macro(choice.na, choice.nb, g.side, g.bdim, choice.tau, o, s),
                       "plan and schedule kernel");
    } else {
        uint64_t* masks = at<uint64_t>(ws, L.masks);
        int32_t *counts = at<int32_t>(ws, L.counts), *bsums = at<int32_t>(ws, L.bsums),
                *boffs = at<int32_t>(ws, L.boffs);
        const spamm::PyramidJob pj{{at<double>(ws, L.spyr[0]), at<double>(ws, L.spyr[1])},
                                   {at<double>(ws, L.pyr[0]), at<double>(ws, L.pyr[1])}};
        hipError_t e = spamm::launch_pyramid(pj, 2, g.bdim, g.lv, s, run);
        if (e == hipSuccess)
            e = spamm::launch_plan_mask(pj.pyr[0], pj.pyr[1], g.bdim, g.lv, choice.tau, masks, counts, bsums, s, run);
        if (e == hipSuccess)
            e = spamm::launch_plan_scan(bsums, g.bdim * g.nwords, boffs, offsets, g.ntiles, pairs, s, run);
        if (e == hipSuccess) e = spamm::launch_plan_fill(masks, counts, boffs, g.bdim, offsets, klist, s, run);
        if (e == hipSuccess) e = spamm::launch_macro_schedule(offsets, klist, g.bdim, ms, s, run);
        st = hip_check(e, "plan and schedule kernels");
    }
    if (st != SPAMM_OK) return st;
    return hip_check(spamm::launch_lowp_multiply(SL, c, g.n, g.bdim, spamm::kPrecBf16, ms.items, ms.uprefix,
                                                 device_cus(), s, run),
                     "reduced-precision multiply kernel");
}
}  // namespace

spamm_status spamm_multiply(const float* a, const float* b, int64_t n, double tau, int32_t leaf, float* c,
                            int64_t* pairs, void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if ((st = check_tau(tau)) != SPAMM_OK) return st;
    if ((st = check_grid(g)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    const Layout L = make_layout(g);
    int64_t* np = pairs ? pairs : at<int64_t>(workspace, L.pairs);
    if (spamm::block_product(g.n, g.leaf))
        return enqueue_direct(g, a, b, tau, c, np, workspace, static_cast<hipStream_t>(stream));
    int32_t* offsets = at<int32_t>(workspace, L.offsets);
    int32_t* klist = at<int32_t>(workspace, L.klist);
    hipStream_t s = static_cast<hipStream_t>(stream);
    if ((st = enqueue_prepare(g, a, b, tau, offsets, klist, np, workspace, s, true)) != SPAMM_OK) return st;
    return enqueue_multiply(g, a, b, offsets, klist, c, workspace, s);
}

size_t spamm_split_bytes(int64_t n, int32_t precision) {
    if (n <= 0 || (precision != spamm::kPrecBf16 && precision != spamm::kPrecF16x3)) return 0;
    return kSplitHeaderBytes + size_t(split_planes(precision)) * plane_bytes(n);
}

spamm_status spamm_split(const float* a, const float* b, int64_t n, int32_t leaf, int32_t precision,
                         const double* pyr_a, const double* pyr_b, void* split, size_t split_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!a || !b || !pyr_a || !pyr_b || !split) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_lowp(g, precision);
    if (st != SPAMM_OK) return st;
    if (!aligned16(a) || !aligned16(b) || (reinterpret_cast<uintptr_t>(split) & 255u) != 0)
        return fail(SPAMM_EINVAL, "a, b need 16-byte and split 256-byte alignment");
    if (split_bytes < spamm_split_bytes(n, precision))
        return fail(SPAMM_ENOSPACE, "split buffer of %zu bytes, %zu needed", split_bytes,
                    spamm_split_bytes(n, precision));
    const size_t sb = spamm_split_bytes(n, precision);
    const size_t mb = sizeof(float) * size_t(n) * size_t(n);
    if (overlaps(split, sb, a, mb) || overlaps(split, sb, b, mb))
        return fail(SPAMM_EINVAL, "split buffer overlaps a or b");
    return hip_check(spamm::launch_split(a, b, n, g.bdim, g.lv, pyr_a, pyr_b, precision,
                                         split_layout(split, n, precision), static_cast<hipStream_t>(stream)),
                     "split kernels");
}

spamm_status spamm_execute_split_scheduled(const void* split, int64_t n, int32_t leaf, int32_t precision,
                                           const int32_t* offsets, const int32_t* klist, float* c, void* workspace,
                                           size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!split || !offsets || !klist || !c) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_lowp(g, precision);
    if (st != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (overlaps(c, sizeof(float) * size_t(n) * size_t(n), split, spamm_split_bytes(n, precision)))
        return fail(SPAMM_EINVAL, "c overlaps the split buffer");
    const Layout L = make_layout(g);
    return hip_check(spamm::launch_lowp_multiply(split_layout(const_cast<void*>(split), n, precision), c, n, g.bdim,
                                                 precision, at<uint32_t>(workspace, L.mitems),
                                                 at<int32_t>(workspace, L.mprefix), device_cus(),
                                                 static_cast<hipStream_t>(stream)),
                     "reduced-precision multiply kernel");
}

spamm_status spamm_execute_split(const void* split, int64_t n, int32_t leaf, int32_t precision,
                                 const int32_t* offsets, const int32_t* klist, float* c, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    spamm_status st = spamm_schedule(offsets, klist, n, leaf, workspace, workspace_bytes, stream);
    if (st != SPAMM_OK) return st;
    return spamm_execute_split_scheduled(split, n, leaf, precision, offsets, klist, c, workspace, workspace_bytes,
                                         stream);
}

spamm_status spamm_split_scales(const double* pyr_a, const double* pyr_b, int64_t n, int32_t leaf, void* header,
                                size_t header_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!pyr_a || !pyr_b || !header) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_lowp(g, spamm::kPrecF16x3);
    if (st != SPAMM_OK) return st;
    if ((reinterpret_cast<uintptr_t>(header) & 255u) != 0) return fail(SPAMM_EINVAL, "header must be 256-byte aligned");
    if (header_bytes < kSplitHeaderBytes)
        return fail(SPAMM_ENOSPACE, "header of %zu bytes, %zu needed", header_bytes, kSplitHeaderBytes);
    return hip_check(spamm::launch_split_scales(g.bdim, g.lv, pyr_a, pyr_b, static_cast<int32_t*>(header),
                                                static_cast<hipStream_t>(stream)),
                     "scale kernels");
}

spamm_status spamm_execute_f16x3_scheduled(const float* a, const float* b, int64_t n, int32_t leaf,
                                           const void* header, const int32_t* offsets, const int32_t* klist,
                                           float* c, void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!header || !offsets || !klist) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if ((st = check_lowp(g, spamm::kPrecF16x3)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (!aligned16(a) || !aligned16(b)) return fail(SPAMM_EINVAL, "a and b need 16-byte alignment");
    if (overlaps(c, sizeof(float) * size_t(n) * size_t(n), header, kSplitHeaderBytes))
        return fail(SPAMM_EINVAL, "c overlaps the header");
    const Layout L = make_layout(g);
    return hip_check(spamm::launch_convert_plan(a, b, spamm::kPrecF16x3, static_cast<const int32_t*>(header), c, n,
                                                g.bdim, at<uint32_t>(workspace, L.mitems),
                                                at<int32_t>(workspace, L.mprefix), static_cast<hipStream_t>(stream)),
                     "fused f16x3 multiply kernel");
}

spamm_status spamm_execute_bf16_scheduled(const float* a, const float* b, int64_t n, int32_t leaf,
                                          const int32_t* offsets, const int32_t* klist, float* c, void* workspace,
                                          size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!offsets || !klist) return fail(SPAMM_EINVAL, "null pointer");
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if ((st = check_lowp(g, spamm::kPrecBf16)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    if (!aligned16(a) || !aligned16(b)) return fail(SPAMM_EINVAL, "a and b need 16-byte alignment");
    const Layout L = make_layout(g);
    return hip_check(spamm::launch_convert_plan(a, b, spamm::kPrecBf16, nullptr, c, n, g.bdim,
                                                at<uint32_t>(workspace, L.mitems),
                                                at<int32_t>(workspace, L.mprefix), static_cast<hipStream_t>(stream)),
                     "fused bf16 multiply kernel");
}

spamm_status spamm_prepare_scales(const float* a, const float* b, int64_t n, double tau, int32_t leaf,
                                  int32_t* offsets, int32_t* klist, int64_t klist_capacity, int64_t* pairs,
                                  void* header, size_t header_bytes, void* workspace, size_t workspace_bytes,
                                  void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_lowp(g, spamm::kPrecF16x3);
    if (st != SPAMM_OK) return st;
    const size_t mbytes = sizeof(float) * size_t(n) * size_t(n);
    if (header && (overlaps(header, kSplitHeaderBytes, a, mbytes) || overlaps(header, kSplitHeaderBytes, b, mbytes)))
        return fail(SPAMM_EINVAL, "header overlaps a or b");
    st = spamm_prepare(a, b, n, tau, leaf, offsets, klist, klist_capacity, pairs, workspace, workspace_bytes, stream);
    if (st != SPAMM_OK) return st;
    const Layout L = make_layout(g);
    return spamm_split_scales(at<double>(workspace, L.pyr[0]), at<double>(workspace, L.pyr[1]), n, leaf, header,
                              header_bytes, stream);
}

spamm_status spamm_prepare_schedule_scales(const float* a, const float* b, int64_t n, double tau, int32_t leaf,
                                           int32_t* offsets, int32_t* klist, int64_t klist_capacity,
                                           int64_t* pairs, void* header, size_t header_bytes, void* workspace,
                                           size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_lowp(g, spamm::kPrecF16x3);
    if (st != SPAMM_OK) return st;
    // the header is checked before anything is enqueued
    if (!header || (reinterpret_cast<uintptr_t>(header) & 255u) != 0)
        return fail(SPAMM_EINVAL, "the header must be non-null and 256-byte aligned");
    if (header_bytes < kSplitHeaderBytes)
        return fail(SPAMM_ENOSPACE, "header of %zu bytes, %zu needed", header_bytes, kSplitHeaderBytes);
    const size_t mbytes = sizeof(float) * size_t(n) * size_t(n);
    if (overlaps(header, kSplitHeaderBytes, a, mbytes) || overlaps(header, kSplitHeaderBytes, b, mbytes))
        return fail(SPAMM_EINVAL, "header overlaps a or b");
    st = spamm_prepare_schedule(a, b, n, tau, leaf, offsets, klist, klist_capacity, pairs, workspace,
                                workspace_bytes, stream);
    if (st != SPAMM_OK) return st;
    // the scale kernels read the leaf level, which either form of the plan leaves
    const Layout L = make_layout(g);
    return spamm_split_scales(at<double>(workspace, L.pyr[0]), at<double>(workspace, L.pyr[1]), n, leaf, header,
                              header_bytes, stream);
}

spamm_status spamm_prepare_split(const float* a, const float* b, int64_t n, double tau, int32_t leaf,
                                 int32_t precision, int32_t* offsets, int32_t* klist, int64_t klist_capacity,
                                 int64_t* pairs, void* split, size_t split_bytes, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_lowp(g, precision);
    if (st != SPAMM_OK) return st;
    st = spamm_prepare(a, b, n, tau, leaf, offsets, klist, klist_capacity, pairs, workspace, workspace_bytes, stream);
    if (st != SPAMM_OK) return st;
    const Layout L = make_layout(g);
    return spamm_split(a, b, n, leaf, precision, at<double>(workspace, L.pyr[0]), at<double>(workspace, L.pyr[1]),
                       split, split_bytes, stream);
}

spamm_status spamm_multiply_precision(const float* a, const float* b, int64_t n, double tau, int32_t leaf,
                                      int32_t precision, float* c, int64_t* pairs, void* split, size_t split_bytes,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    if (precision == spamm::kPrecFp32)
        return spamm_multiply(a, b, n, tau, leaf, c, pairs, workspace, workspace_bytes, stream);
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    spamm_status st = check_mul_args(g, a, b, c);
    if (st != SPAMM_OK) return st;
    if ((st = check_lowp(g, precision)) != SPAMM_OK) return st;
    if ((st = check_tau(tau)) != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    const Layout L = make_layout(g);
    int64_t* np = pairs ? pairs : at<int64_t>(workspace, L.pairs);
    const bool f16 = precision == spamm::kPrecF16x3;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (!aligned16(a) || !aligned16(b)) return fail(SPAMM_EINVAL, "a and b need 16-byte alignment");
    const bool planes = split_bytes >= spamm_split_bytes(n, precision);
    if (planes) {
        const size_t sb = spamm_split_bytes(n, precision), mbytes = sizeof(float) * size_t(n) * size_t(n);
        if (!split || overlaps(split, sb, a, mbytes) || overlaps(split, sb, b, mbytes) ||
            overlaps(split, sb, c, mbytes))
            return fail(SPAMM_EINVAL, "split buffer null or overlapping a, b or c");
    }
    if (f16) {  // the scale exponents go to the split buffer's 256-byte header
        const size_t mbytes = sizeof(float) * size_t(n) * size_t(n);
        if (!split || (reinterpret_cast<uintptr_t>(split) & 255u) != 0)
            return fail(SPAMM_EINVAL, "the split header must be non-null and 256-byte aligned");
        if (split_bytes < kSplitHeaderBytes)
            return fail(SPAMM_ENOSPACE, "header of %zu bytes, %zu needed", split_bytes, kSplitHeaderBytes);
        if (overlaps(split, kSplitHeaderBytes, a, mbytes) || overlaps(split, kSplitHeaderBytes, b, mbytes) ||
            overlaps(split, kSplitHeaderBytes, c, mbytes))
            return fail(SPAMM_EINVAL, "header overlaps a, b or c");
    }
    // BF16 with room for the planes (at the alignment that spamm_split asks for):
    // the device picks between them and the FP32 inputs; both give the same C
    const int32_t* form = nullptr;
    spamm::FormChoice choice{};
    const bool choose = !f16 && planes && (reinterpret_cast<uintptr_t>(split) & 255u) == 0 &&
                        spamm::bf16_choice(n, g.bdim, &choice);
    double* norms[2];
    if ((st = enqueue_leaf_norms(g, a, b, np, choose && g.bdim > spamm::kPlanMacroMaxBdim, norms, workspace, s)) !=
        SPAMM_OK)
        return st;
    if (choose) {
        choice.na = norms[0];
        choice.nb = norms[1];
        choice.ld = g.side;
        choice.tau = tau;
        choice.form = at<int32_t>(workspace, L.form);
        if ((st = enqueue_planes(g, a, b, choice, split_layout(split, n, precision), c, np, workspace, s)) != SPAMM_OK)
            return st;
        form = choice.form;
    }
    int32_t* exps = f16 ? static_cast<int32_t*>(split) : nullptr;
    if (f16 && (st = hip_check(spamm::launch_split_scales(g.bdim, g.lv, at<double>(workspace, L.pyr[0]),
                                                          at<double>(workspace, L.pyr[1]), exps, s),
                               "scale kernel")) != SPAMM_OK)
        return st;
    return hip_check(spamm::launch_convert_test(a, b, precision, exps, c, n, g.bdim, norms[0], norms[1], g.side, tau,
                                                np, form, s),
                     "reduced-precision multiply kernel (FP32 inputs)");
}

spamm_status spamm_search_valid_ratio(const double* pyr_a, const double* pyr_b, int64_t n, int32_t leaf,
                                      double target, double tol, int32_t max_iters, double* tau_out,
                                      int64_t* pairs_out, int32_t* iters_out, void* workspace, size_t workspace_bytes,
                                      void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!pyr_a || !pyr_b || !tau_out) return fail(SPAMM_EINVAL, "null pointer");
    if (!(target > 0.0 && target <= 1.0)) return fail(SPAMM_EINVAL, "target valid ratio must be in (0, 1]");
    if (!(tol >= 0.0) || max_iters < 0) return fail(SPAMM_EINVAL, "tol must be >= 0 and max_iters >= 0");
    spamm_status st = check_grid(g);
    if (st != SPAMM_OK) return st;
    if ((st = check_workspace(g, workspace, workspace_bytes)) != SPAMM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    SearchRegions R;
    if (!search_regions(g, &R)) return fail(SPAMM_ENOSPACE, "no room for the search in the workspace");
    double* rows_b = at<double>(workspace, R.rows_b);
    double* cols_a = at<double>(workspace, R.cols_a);
    double* ksums = at<double>(workspace, R.ksums);
    int32_t* counts[2] = {at<int32_t>(workspace, R.count_even), at<int32_t>(workspace, R.count_odd)};
    auto* states = at<spamm::SearchState>(workspace, R.states);
    spamm::SearchState h{};
    h.target = target;
    h.tol = tol;
    h.triples = double(g.bdim) * double(g.bdim) * double(g.bdim);
    h.max_iters = max_iters;
    if ((st = hip_check(spamm::launch_norms_sort(pyr_a, pyr_b, g.bdim, g.lv, rows_b, cols_a, ksums, states, h, s),
                        "norm sort kernel")) != SPAMM_OK)
        return st;
    // kRounds rounds per host read: one round of bounds and up to 4 bisection
    // steps in each of the others (a search at tol 0.01 takes 5 to 10)
    constexpr int kRounds = 4;
    for (int round = 0; !h.done;) {
        for (int q = 0; q < kRounds; ++q, ++round)
            if ((st = hip_check(spamm::launch_ratio_probe(rows_b, cols_a, ksums, g.bdim, states, counts, round, s),
                                "count kernel")) != SPAMM_OK)
                return st;
        if ((st = hip_check(spamm::launch_ratio_finish(g.bdim, states, counts, round, s), "count kernel")) != SPAMM_OK)
            return st;
        if ((st = hip_check(hipMemcpyAsync(&h, states + (round & 1), sizeof(h), hipMemcpyDeviceToHost, s), "copy")) !=
            SPAMM_OK)
            return st;
        if ((st = hip_check(hipStreamSynchronize(s), "synchronize")) != SPAMM_OK) return st;
    }
    *tau_out = h.tau;
    if (pairs_out) *pairs_out = h.kept;
    if (iters_out) *iters_out = h.iters;
    return SPAMM_OK;
}

const char* spamm_strerror(spamm_status status) {
    switch (status) {
        case SPAMM_OK: return "success";
        case SPAMM_EINVAL: return "invalid argument";
        case SPAMM_ENOSPACE: return "workspace or output capacity too small";
        case SPAMM_EDEVICE: return "HIP runtime or kernel launch failure";
        case SPAMM_EUNSUPPORTED: return "unsupported leaf or problem size";
    }
    return "unknown status";
}

const char* spamm_last_error(void) { return g_last_error; }

}  // extern "C"
