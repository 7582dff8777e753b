// Host side of the batched entry points: many independent SpAMM products, each
// stage of the path one launch over all of them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "host.h"
#include "internal.h"
#include "spamm.h"

using namespace spamm_host;

namespace {

constexpr size_t kAlignB = 256;
size_t up(size_t v) { return (v + kAlignB - 1) / kAlignB * kAlignB; }

int leaf_class(int32_t leaf) { return leaf == 32 ? 0 : leaf == 64 ? 1 : leaf == 128 ? 2 : -1; }

// Workspace: the descriptors in the order of the launches, the prefix of the
// norm pass's blocks over them and of the multiply's within each leaf class,
// then every product's leaf norms.
struct BatchPlan {
    size_t strips_at = 0, blocks_at = 0, total = 0;
    std::vector<size_t> base;  // per product region offset
    std::vector<Geom> geom;
    int64_t strips = 0;
    double bytes = 0.0;  // of all inputs
    int32_t class_count[spamm::kBatchClasses] = {0, 0, 0};
    int64_t class_blocks[spamm::kBatchClasses] = {0, 0, 0};
};

size_t norm_bytes(const Geom& g) { return up(sizeof(double) * size_t(g.ntiles)); }

spamm_status plan_batch(int32_t count, const int64_t* n, const int32_t* leaf, BatchPlan* bp) {
    if (count < 1 || !n || !leaf) return fail(SPAMM_EINVAL, "empty batch or null size arrays");
    bp->geom.resize(size_t(count));
    bp->base.resize(size_t(count));
    bp->strips_at = up(sizeof(spamm::BatchProduct) * size_t(count));
    bp->blocks_at = bp->strips_at + up(sizeof(int64_t) * size_t(count));
    size_t o = bp->blocks_at + up(sizeof(int64_t) * size_t(count));
    for (int32_t p = 0; p < count; ++p) {
        Geom& g = bp->geom[size_t(p)];
        if (!make_geom(n[p], leaf[p], &g)) return fail(SPAMM_EINVAL, "product %d: bad size n=%lld leaf=%d", p,
                                                       (long long)n[p], leaf[p]);
        if (leaf_class(leaf[p]) < 0) return fail(SPAMM_EUNSUPPORTED, "product %d: leaf %d (32, 64, 128)", p, leaf[p]);
        if (g.bdim > SPAMM_MAX_BDIM)
            return fail(SPAMM_EUNSUPPORTED, "product %d: tile grid %lld exceeds %d", p, (long long)g.bdim,
                        SPAMM_MAX_BDIM);
        bp->base[size_t(p)] = o;
        o += 2 * norm_bytes(g);
        bp->strips += spamm::batch_strips(g.n, g.bdim);
        bp->bytes += 8.0 * double(g.n) * double(g.n);
        bp->class_blocks[leaf_class(leaf[p])] += spamm::batch_blocks(g.n);
        ++bp->class_count[leaf_class(leaf[p])];
    }
    bp->total = o;
    return SPAMM_OK;
}

}  // namespace

extern "C" {

size_t spamm_batch_workspace_bytes(int32_t count, const int64_t* n, const int32_t* leaf) {
    BatchPlan bp;
    return plan_batch(count, n, leaf, &bp) == SPAMM_OK ? bp.total : 0;
}

spamm_status spamm_batch_setup(int32_t count, const float* const* a, const float* const* b, float* const* c,
                               const int64_t* n, const int32_t* leaf, const double* tau, int64_t* pairs,
                               void* workspace, size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    BatchPlan bp;
    spamm_status st = plan_batch(count, n, leaf, &bp);
    if (st != SPAMM_OK) return st;
    if (!a || !b || !c || !tau || !pairs || !workspace) return fail(SPAMM_EINVAL, "null pointer");
    if (workspace_bytes < bp.total)
        return fail(SPAMM_ENOSPACE, "batch workspace of %zu bytes, %zu needed", workspace_bytes, bp.total);
    if ((reinterpret_cast<uintptr_t>(workspace) & (kAlignB - 1)) != 0)
        return fail(SPAMM_EINVAL, "workspace must be 256-byte aligned");
    for (int32_t p = 0; p < count; ++p) {
        if ((st = check_mul_args(bp.geom[size_t(p)], a[p], b[p], c[p])) != SPAMM_OK ||
            (st = check_tau(tau[p])) != SPAMM_OK) {
            char why[sizeof(g_last_error)];
            std::memcpy(why, g_last_error, sizeof(why));
            return fail(st, "product %d: %s", p, why);
        }
    }
    // class after class, in each the largest products first
    std::vector<int32_t> order(static_cast<size_t>(count));
    for (int32_t p = 0; p < count; ++p) order[size_t(p)] = p;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        const int cx = leaf_class(leaf[x]), cy = leaf_class(leaf[y]);
        return cx != cy ? cx < cy : n[x] > n[y];
    });
    std::vector<spamm::BatchProduct> prods(static_cast<size_t>(count));
    std::vector<int64_t> strip_base(static_cast<size_t>(count)), block_base(static_cast<size_t>(count));
    char* ws = static_cast<char*>(workspace);
    int64_t strips = 0, blocks = 0;
    for (int32_t i = 0; i < count; ++i) {
        const int32_t p = order[size_t(i)];
        const Geom& g = bp.geom[size_t(p)];
        if (i == 0 || leaf_class(leaf[p]) != leaf_class(leaf[order[size_t(i - 1)]])) blocks = 0;
        strip_base[size_t(i)] = strips;
        block_base[size_t(i)] = blocks;
        strips += spamm::batch_strips(g.n, g.bdim);
        blocks += spamm::batch_blocks(g.n);
        spamm::BatchProduct& q = prods[size_t(i)];
        std::memset(&q, 0, sizeof(q));
        char* r = ws + bp.base[size_t(p)];
        for (int m = 0; m < 2; ++m) q.norms[m] = reinterpret_cast<double*>(r + size_t(m) * norm_bytes(g));
        q.a = a[p];
        q.b = b[p];
        q.c = c[p];
        q.pairs = pairs + p;
        q.n = g.n;
        q.bdim = g.bdim;
        q.leaf = g.leaf;
        q.vec = (g.n % 4) == 0 && aligned16(a[p]) && aligned16(b[p]);
        q.tau = tau[p];
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    st = hip_check(hipMemcpyAsync(ws, prods.data(), sizeof(spamm::BatchProduct) * size_t(count),
                                  hipMemcpyHostToDevice, s),
                   "descriptor upload");
    if (st != SPAMM_OK) return st;
    st = hip_check(hipMemcpyAsync(ws + bp.strips_at, strip_base.data(), sizeof(int64_t) * size_t(count),
                                  hipMemcpyHostToDevice, s),
                   "descriptor upload");
    if (st != SPAMM_OK) return st;
    st = hip_check(hipMemcpyAsync(ws + bp.blocks_at, block_base.data(), sizeof(int64_t) * size_t(count),
                                  hipMemcpyHostToDevice, s),
                   "descriptor upload");
    if (st != SPAMM_OK) return st;
    return hip_check(hipStreamSynchronize(s), "synchronize");
}

spamm_status spamm_batch_run(int32_t count, const int64_t* n, const int32_t* leaf, void* workspace,
                             size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    BatchPlan bp;
    spamm_status st = plan_batch(count, n, leaf, &bp);
    if (st != SPAMM_OK) return st;
    if (!workspace) return fail(SPAMM_EINVAL, "null workspace");
    if (workspace_bytes < bp.total)
        return fail(SPAMM_ENOSPACE, "batch workspace of %zu bytes, %zu needed", workspace_bytes, bp.total);
    char* ws = static_cast<char*>(workspace);
    return hip_check(spamm::launch_batch(reinterpret_cast<const spamm::BatchProduct*>(ws),
                                         reinterpret_cast<const int64_t*>(ws + bp.strips_at),
                                         reinterpret_cast<const int64_t*>(ws + bp.blocks_at), bp.class_count,
                                         bp.class_blocks, bp.strips, bp.bytes, count, static_cast<hipStream_t>(stream)),
                     "batch kernels");
}

}  // extern "C"
