// Host side of the threshold-selection entry points (spamm_tau.h): error of
// SpAMM at a given tau, the search for the largest tau meeting an error
// target, and the network kernels' launchers.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <limits>

#include "host.h"
#include "internal.h"
#include "search.h"
#include "spamm_tau.h"

using namespace spamm_host;

namespace {

constexpr double kInf = std::numeric_limits<double>::infinity();

// The device-side pieces of one (A, B) problem that the search uses.
struct Probe {
    Geom g;
    const float *a, *b;
    const double *pa, *pb;
    double ab_sumsq;
    float* e;
    void* ws;
    hipStream_t s;
    // what the norm queries and the error evaluations keep in the workspace
    double *rows_b, *cols_a, *ksums, *partials, *sums;
    int32_t* counts;
    spamm::StepAnswer* answer;
    int64_t blocks;

    spamm_status bind() {
        SearchRegions R;
        if (!search_regions(g, &R)) return fail(SPAMM_ENOSPACE, "no room for the search in the workspace");
        rows_b = at<double>(ws, R.rows_b);
        cols_a = at<double>(ws, R.cols_a);
        ksums = at<double>(ws, R.ksums);
        partials = at<double>(ws, R.partials);
        answer = at<spamm::StepAnswer>(ws, R.answer);
        blocks = R.blocks;
        sums = at<double>(ws, R.sums);
        counts = at<int32_t>(ws, R.counts);
        return SPAMM_OK;
    }

    spamm_status sort() const {
        return hip_check(spamm::launch_norms_sort(pa, pb, g.bdim, g.lv, rows_b, cols_a, ksums, nullptr, {}, s),
                         "norm sort kernel");
    }

    // E at tau from the E of band.base (launch_block_dropped)
    spamm_status dropped(double tau, spamm::BandJob band) const {
        const int64_t leaf_level = spamm::level_offset(g.lv);
        band.sums = sums;
        band.counts = counts;
        return hip_check(spamm::launch_block_dropped(a, b, e, g.n, g.leaf, g.bdim, pa + leaf_level, pb + leaf_level,
                                                     g.side, tau, band, s),
                         "error kernel");
    }

    // the answers of the last queries (q.count of them, 0: none) and error
    // evaluation (evaluated), read back
    spamm_status read(const spamm::StepQuery& q, bool evaluated, spamm::StepAnswer* h) const {
        spamm_status st = SPAMM_OK;
        if (q.count > 0 && (st = hip_check(spamm::launch_norm_query(rows_b, cols_a, g.bdim, q, partials, s),
                                           "norm query kernel")) != SPAMM_OK)
            return st;
        st = hip_check(spamm::launch_step_answer(partials, g.bdim, q.count, sums, counts, evaluated ? blocks : 0, answer,
                                                 s),
                       "answer kernel");
        if (st != SPAMM_OK) return st;
        if ((st = hip_check(hipMemcpyAsync(h, answer, sizeof(*h), hipMemcpyDeviceToHost, s), "copy")) != SPAMM_OK)
            return st;
        return hip_check(hipStreamSynchronize(s), "synchronize");
    }

    // relative error at tau, E formed from nothing and, with store, left in e;
    // and the number of dropped triples
    spamm_status error(double tau, bool store, double* err, int64_t* count) const {
        spamm::BandJob band;
        band.store = store ? 1 : 0;
        spamm_status st = dropped(tau, band);
        if (st != SPAMM_OK) return st;
        spamm::StepAnswer h;
        if ((st = read(spamm::StepQuery{}, true, &h)) != SPAMM_OK) return st;
        *err = std::sqrt(h.sumsq / ab_sumsq);
        if (count) *count = h.dropped;
        return SPAMM_OK;
    }

    // kept triples at tau (count-only plan)
    spamm_status kept(double tau, int64_t* out) const {
        const Layout L = make_layout(g);
        int32_t* bsums = at<int32_t>(ws, L.bsums);
        int64_t* d_pairs = at<int64_t>(ws, L.pairs);
        spamm_status st =
            hip_check(spamm::launch_plan_count(pa, pb, g.bdim, g.lv, tau, bsums, s), "count kernel");
        if (st != SPAMM_OK) return st;
        st = hip_check(spamm::launch_plan_scan(bsums, g.bdim * g.nwords, nullptr, nullptr, 0, d_pairs, s),
                       "scan kernel");
        if (st != SPAMM_OK) return st;
        if ((st = hip_check(hipMemcpyAsync(out, d_pairs, sizeof(int64_t), hipMemcpyDeviceToHost, s), "copy")) !=
            SPAMM_OK)
            return st;
        return hip_check(hipStreamSynchronize(s), "synchronize");
    }
};

// The search's view of a Probe: thresholds snapped up to norm products, and
// errors at products.  An evaluation carries along the queries that the search
// asks next whichever way it turns out, so that a step of the bisection costs
// one synchronisation; the E of the largest passing product is kept in e, and
// an evaluation adds to it only the products between the two thresholds.
//
// Such an E holds the same products as one formed from nothing, added in another
// order, so its error is spamm_error_for_tau's to rounding only (1.7e-7 of it at
// most on 150 problems of N = 300 .. 3000, 7e-8 on 32 of 8192).  An error within
// kNear of the target is formed again from nothing, so that what passes does not
// depend on the thresholds tried before.
class Search {
public:
    struct Snap {
        double x, least;  // the smallest norm product >= x (+inf: none)
        int64_t kept;     // how many products are >= x
    };

    Search(const Probe& p, double target) : p_(p), target_(target) {}

    spamm_status start(double x, Snap* out, double* most) {
        spamm_status st = p_.sort();
        if (st != SPAMM_OK) return st;
        return ask(&x, 1, nullptr, out, most);
    }

    spamm_status snap(double x, Snap* out) {
        for (const Snap& k : known_)
            if (k.x == x) {
                *out = k;
                return SPAMM_OK;
            }
        return ask(&x, 1, nullptr, out, nullptr);
    }

    // error at the product t, with the queries that may follow
    spamm_status eval(double t, const double* next, int count, bool* pass, double* err) {
        spamm_status st;
        if (pending_) {  // the product evaluated last passed: its E becomes the base
            spamm::BandJob keep = base_;
            keep.store = 1;
            if ((st = p_.dropped(passed_, keep)) != SPAMM_OK) return st;
            base_.base = passed_;
            base_.has_base = 1;
            pending_ = false;
        }
        if ((st = p_.dropped(t, base_)) != SPAMM_OK) return st;
        double esq = 0.0;
        if ((st = ask(next, count, &esq, nullptr, nullptr)) != SPAMM_OK) return st;
        *err = std::sqrt(esq / p_.ab_sumsq);
        if (base_.has_base && std::fabs(*err - target_) < kNear * target_ &&
            (st = p_.error(t, false, err, nullptr)) != SPAMM_OK)
            return st;
        *pass = *err <= target_;
        if (*pass) {
            pending_ = true;
            passed_ = t;
        }
        return SPAMM_OK;
    }

private:
    // queries (those > 0 and finite) and, with esq, the evaluation just enqueued
    spamm_status ask(const double* x, int count, double* esq, Snap* first, double* most) {
        spamm::StepQuery q{};
        for (int c = 0; c < count; ++c)
            if (x[c] > 0.0 && (!std::isinf(x[c]) || first)) q.x[q.count++] = x[c];
        spamm::StepAnswer h;
        const spamm_status st = p_.read(q, esq != nullptr, &h);
        if (st != SPAMM_OK) return st;
        for (int c = 0; c < q.count; ++c) {
            known_[at_] = {q.x[c], h.least[c], h.kept[c]};
            if (c == 0 && first) *first = known_[at_];
            at_ = (at_ + 1) % kKnown;
        }
        if (most) *most = h.most;
        if (esq) *esq = h.sumsq;
        return SPAMM_OK;
    }

    static constexpr int kKnown = 12;
    static constexpr double kNear = 1e-5;
    const Probe& p_;
    double target_;
    Snap known_[kKnown] = {};
    int at_ = 0;
    spamm::BandJob base_;
    bool pending_ = false;
    double passed_ = 0.0;
};

spamm_status make_probe(const float* a, const float* b, int64_t n, int32_t leaf, const double* pa, const double* pb,
                        double ab_sumsq, float* e, void* ws, size_t ws_bytes, void* stream, Probe* p) {
    if (!make_geom(n, leaf, &p->g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!pa || !pb) return fail(SPAMM_EINVAL, "null pyramid pointer");
    spamm_status st = check_mul_args(p->g, a, b, e);
    if (st != SPAMM_OK) return st;
    if (!(ab_sumsq > 0.0) || std::isinf(ab_sumsq))
        return fail(SPAMM_EINVAL, "||AB||_F^2 must be positive and finite (got %g)", ab_sumsq);
    if ((st = check_grid(p->g)) != SPAMM_OK) return st;
    if ((st = check_workspace(p->g, ws, ws_bytes)) != SPAMM_OK) return st;
    p->a = a;
    p->b = b;
    p->pa = pa;
    p->pb = pb;
    p->ab_sumsq = ab_sumsq;
    p->e = e;
    p->ws = ws;
    p->s = static_cast<hipStream_t>(stream);
    return p->bind();
}

}  // namespace

extern "C" {

int64_t spamm_mlp_param_count(void) { return spamm::MlpLayout{}.count; }

int64_t spamm_mlp_acts_floats(int32_t batch) { return batch < 1 ? 0 : spamm::MlpLayout::acts(batch).acts_total; }

spamm_status spamm_tau_features(const double* pyr_a, const double* pyr_b, int64_t n, int32_t leaf, double target,
                                float* features, void* stream) {
    g_last_error[0] = '\0';
    Geom g;
    if (!make_geom(n, leaf, &g)) return fail(SPAMM_EINVAL, "bad size n=%lld leaf=%d", (long long)n, leaf);
    if (!pyr_a || !pyr_b || !features) return fail(SPAMM_EINVAL, "null pointer");
    if (!(target > 0.0) || std::isinf(target)) return fail(SPAMM_EINVAL, "target must be positive and finite");
    return hip_check(spamm::launch_tau_features(pyr_a, pyr_b, g.bdim, g.lv, float(std::log10(target)), features,
                                                static_cast<hipStream_t>(stream)),
                     "features kernel");
}

spamm_status spamm_mlp_forward(const float* params, const float* x, int32_t batch, float* y, float* acts,
                               void* stream) {
    g_last_error[0] = '\0';
    if (!params || !x || !y || !acts) return fail(SPAMM_EINVAL, "null pointer");
    if (batch < 1) return fail(SPAMM_EINVAL, "batch must be >= 1");
    return hip_check(spamm::launch_mlp_forward(params, x, batch, acts, y, static_cast<hipStream_t>(stream)),
                     "network forward kernels");
}

spamm_status spamm_mlp_loss_grad(const float* params, const float* x, const float* t, int32_t batch, float* acts,
                                 float* grad, float* loss, void* stream) {
    g_last_error[0] = '\0';
    if (!params || !x || !t || !acts || !grad || !loss) return fail(SPAMM_EINVAL, "null pointer");
    if (batch < 1) return fail(SPAMM_EINVAL, "batch must be >= 1");
    return hip_check(
        spamm::launch_mlp_loss_grad(params, x, t, batch, acts, grad, loss, static_cast<hipStream_t>(stream)),
        "network gradient kernels");
}

spamm_status spamm_mlp_adam(float* params, const float* grad, float* m, float* v, int32_t step, float lr,
                            float beta1, float beta2, float eps, void* stream) {
    g_last_error[0] = '\0';
    if (!params || !grad || !m || !v) return fail(SPAMM_EINVAL, "null pointer");
    if (step < 1) return fail(SPAMM_EINVAL, "step counts from 1");
    const float c1 = float(1.0 - std::pow(double(beta1), double(step)));
    const float c2 = float(1.0 - std::pow(double(beta2), double(step)));
    return hip_check(spamm::launch_adam(params, grad, m, v, spamm::MlpLayout{}.count, lr, beta1, beta2, eps, c1, c2,
                                        static_cast<hipStream_t>(stream)),
                     "adam kernel");
}

size_t spamm_sumsq_scratch_bytes(void) { return sizeof(double) * spamm::kSumBlocks; }

spamm_status spamm_sumsq(const float* x, int64_t count, double* out, void* scratch, size_t scratch_bytes,
                         void* stream) {
    g_last_error[0] = '\0';
    if ((!x && count > 0) || !out || !scratch) return fail(SPAMM_EINVAL, "null pointer");
    if (count < 0) return fail(SPAMM_EINVAL, "count must be >= 0");
    if (scratch_bytes < spamm_sumsq_scratch_bytes())
        return fail(SPAMM_ENOSPACE, "scratch of %zu bytes, %zu needed", scratch_bytes, spamm_sumsq_scratch_bytes());
    return hip_check(
        spamm::launch_sumsq(x, count, static_cast<double*>(scratch), out, static_cast<hipStream_t>(stream)),
        "sumsq kernels");
}

spamm_status spamm_error_for_tau(const float* a, const float* b, int64_t n, int32_t leaf, double tau,
                                 const double* pyr_a, const double* pyr_b, double ab_sumsq, float* e_scratch,
                                 double* err_out, int64_t* dropped_out, void* workspace, size_t workspace_bytes,
                                 void* stream) {
    g_last_error[0] = '\0';
    Probe p;
    spamm_status st = make_probe(a, b, n, leaf, pyr_a, pyr_b, ab_sumsq, e_scratch, workspace, workspace_bytes,
                                 stream, &p);
    if (st != SPAMM_OK) return st;
    if (!err_out) return fail(SPAMM_EINVAL, "null err_out");
    if ((st = check_tau(tau)) != SPAMM_OK) return st;
    return p.error(tau, true, err_out, dropped_out);
}

spamm_status spamm_search_tau_for_error(const float* a, const float* b, int64_t n, int32_t leaf, double target,
                                        double tau_guess, int32_t max_evals, const double* pyr_a,
                                        const double* pyr_b, double ab_sumsq, float* e_scratch, double* tau_out,
                                        double* err_out, int64_t* pairs_out, int32_t* evals_out, void* workspace,
                                        size_t workspace_bytes, void* stream) {
    g_last_error[0] = '\0';
    Probe p;
    spamm_status st = make_probe(a, b, n, leaf, pyr_a, pyr_b, ab_sumsq, e_scratch, workspace, workspace_bytes,
                                 stream, &p);
    if (st != SPAMM_OK) return st;
    if (!tau_out) return fail(SPAMM_EINVAL, "null tau_out");
    if (!(target > 0.0)) return fail(SPAMM_EINVAL, "target must be > 0");
    if (max_evals < 1) return fail(SPAMM_EINVAL, "max_evals must be >= 1");
    if (std::isnan(tau_guess)) return fail(SPAMM_EINVAL, "tau_guess is NaN");

    int evals = 0;
    double pmax = 0.0;
    Search find(p, target);
    Search::Snap low{};
    if ((st = find.start(DBL_TRUE_MIN, &low, &pmax)) != SPAMM_OK) return st;
    const double pmin = low.least;
    double lo = 0.0, lo_err = 0.0;  // passing threshold (a product) and its error
    int64_t kept = low.kept;
    if (std::isinf(pmin)) {
        // every norm product is zero: SpAMM is exactly AB for every tau, and
        // the largest product is 0
        lo = 0.0;
        if ((st = p.kept(lo, &kept)) != SPAMM_OK) return st;
    } else {
        // invariant: lo is a product with error <= target (the smallest positive
        // product keeps every nonzero pair: error 0); hi is a threshold whose
        // error exceeds the target, +inf standing for "above every product"
        lo = pmin;
        double hi = kInf;
        bool pass = false, bracket = true;
        double e = 0.0;
        Search::Snap c{};
        auto middle = [&](double l, double h) { return std::isinf(h) ? pmax : std::sqrt(l) * std::sqrt(h); };
        auto eval = [&]() -> spamm_status {  // at c, with what may be asked next
            const double next[3] = {std::nextafter(c.least, kInf), bracket ? c.least * 4.0 : middle(c.least, hi),
                                    bracket ? c.least / 4.0 : middle(lo, c.least)};
            const spamm_status r = find.eval(c.least, next, 3, &pass, &e);
            ++evals;
            return r;
        };
        auto accept = [&]() {
            lo = c.least;
            lo_err = e;
            kept = c.kept;
        };
        if (tau_guess > 0.0 && evals < max_evals) {
            const double g0 = tau_guess < pmin ? pmin : (tau_guess > pmax ? pmax : tau_guess);
            if ((st = find.snap(g0, &c)) != SPAMM_OK) return st;
            if ((st = eval()) != SPAMM_OK) return st;
            if (pass) {
                accept();
                while (evals < max_evals) {  // grow upwards
                    const double up = lo * 4.0;
                    if (up > pmax) break;
                    if ((st = find.snap(up, &c)) != SPAMM_OK) return st;
                    if ((st = eval()) != SPAMM_OK) return st;
                    if (!pass) {
                        hi = c.least;
                        break;
                    }
                    accept();
                }
            } else {
                hi = c.least;
                while (evals < max_evals) {  // grow downwards
                    const double down = hi / 4.0;
                    if (down <= pmin) break;
                    if ((st = find.snap(down, &c)) != SPAMM_OK) return st;
                    if (c.least >= hi) {  // no product in [down, hi): same mask as hi
                        hi = down;
                        continue;
                    }
                    if ((st = eval()) != SPAMM_OK) return st;
                    if (pass) {
                        accept();
                        break;
                    }
                    hi = c.least;
                }
            }
        }
        bracket = false;
        for (int guard = 0; evals < max_evals && guard < 8192; ++guard) {
            Search::Snap next{};  // the smallest product above lo
            if ((st = find.snap(std::nextafter(lo, kInf), &next)) != SPAMM_OK) return st;
            if (next.least >= hi) break;  // lo is the largest passing product
            double mid = middle(lo, hi);
            if (!(mid > lo)) mid = next.least;
            if ((st = find.snap(mid, &c)) != SPAMM_OK) return st;
            if (c.least >= hi) {  // no product in [mid, hi): mid fails like hi
                hi = mid;
                continue;
            }
            if ((st = eval()) != SPAMM_OK) return st;
            if (pass)
                accept();
            else
                hi = c.least;
        }
    }
    *tau_out = lo;
    if (err_out) *err_out = lo_err;
    if (pairs_out) *pairs_out = kept;
    if (evals_out) *evals_out = evals;
    return SPAMM_OK;
}

}  // extern "C"
