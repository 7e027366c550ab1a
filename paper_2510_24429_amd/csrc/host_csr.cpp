// host_csr.cpp -- host-only logic of the library: parameter defaults,
// Algorithm 1's level schedule, CSR validation, the transpose check and the
// row-length binning of a CSR matrix into workgroup row blocks.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <future>
#include <numeric>

#include "internal.h"

namespace {

void put_msg(char *msg, int len, const char *text) {
    if (msg && len > 0) {
        std::snprintf(msg, (size_t)len, "%s", text);
    }
}

}  // namespace

extern "C" int pdhg_params_default(pdhg_params *p) {
    if (!p) return PDHG_E_ARG;
    std::memset(p, 0, sizeof(*p));
    p->precision = PDHG_FP64;
    p->ruiz_passes = 10;
    p->power_iters = 100;
    p->eval_every = 64;
    p->literal_snapshots = 0;
    p->n_levels = 0;
    p->levels = nullptr;
    p->eps_rel = 1e-6;
    p->eta = 0.0;
    p->omega0 = 0.0;
    p->eta_factor = 0.9;
    p->beta_suff = 0.2;
    p->beta_nec = 0.8;
    p->beta_art = 0.36;
    p->omega_theta = 0.5;
    p->max_iters = (int64_t)1 << 62;
    p->time_limit_s = 3600.0;
    p->use_graph = 1;
    p->variant = 0;
    p->reflect = 1.0;
    p->omega_rule = 0;
    p->pid_kp = 0.99;
    p->pid_ki = 0.01;
    p->pid_kd = 0.0;
    p->stop_on = 0;
    p->polish = 0;
    p->polish_frac = 0.125;
    return PDHG_OK;
}

extern "C" int pdhg_refine_params_default(pdhg_refine_params *p) {
    if (!p) return PDHG_E_ARG;
    std::memset(p, 0, sizeof(*p));
    p->outer_eps = 1e-8;
    p->inner_eps = 1e-4;
    p->max_rounds = 8;
    p->cap_log2 = 10;
    p->max_inner_iters = 200000;
    p->progress = 1e-2;
    p->inner_precision = PDHG_FP32;
    p->omega_carry = 1;
    return PDHG_OK;
}

// Algorithm 1 (Section 3.1) lowers its target tenfold after every launch,
// starting at eps_cross, and stops PDHG at eps_rel.  The levels are formed
// as eps_cross / 10^j so that rounding cannot leave a level a hair above
// eps_rel (repeated multiplication by 0.1 does).
extern "C" int pdhg_alg1_levels(double eps_cross, double eps_rel, double *out,
                                int cap) {
    if (!out || cap < 1 || !(eps_cross > 0.0) || !(eps_rel > 0.0))
        return PDHG_E_ARG;
    int k = 0;
    double p10 = 1.0;
    for (int j = 0; j < 64 && k < cap; ++j) {
        double lev = eps_cross / p10;
        p10 *= 10.0;
        if (lev <= eps_rel * (1.0 + 1e-9)) break;
        out[k++] = lev;
    }
    if (k < cap) out[k++] = eps_rel;
    return k;
}

extern "C" int pdhg_validate_csr(int64_t rows, int64_t cols, int64_t nnz,
                                 const int64_t *rp, const int32_t *ci,
                                 char *msg, int msg_len) {
    char buf[256];
    if (rows < 1 || cols < 1) {
        put_msg(msg, msg_len, "matrix must have at least one row and column");
        return PDHG_E_CSR;
    }
    if (nnz < 0 || nnz >= ((int64_t)1 << 31)) {
        put_msg(msg, msg_len, "nnz must be in [0, 2^31)");
        return PDHG_E_CSR;
    }
    if (cols >= ((int64_t)1 << 31) || rows >= ((int64_t)1 << 31)) {
        put_msg(msg, msg_len, "dimensions must be below 2^31");
        return PDHG_E_CSR;
    }
    if (!rp || (nnz > 0 && !ci)) {
        put_msg(msg, msg_len, "null CSR array");
        return PDHG_E_CSR;
    }
    if (rp[0] != 0 || rp[rows] != nnz) {
        std::snprintf(buf, sizeof buf,
                      "row pointers must start at 0 and end at nnz=%lld "
                      "(got %lld..%lld)",
                      (long long)nnz, (long long)rp[0], (long long)rp[rows]);
        put_msg(msg, msg_len, buf);
        return PDHG_E_CSR;
    }
    for (int64_t i = 0; i < rows; ++i) {
        if (rp[i + 1] < rp[i]) {
            std::snprintf(buf, sizeof buf, "row pointers decrease at row %lld",
                          (long long)i);
            put_msg(msg, msg_len, buf);
            return PDHG_E_CSR;
        }
        for (int64_t p = rp[i]; p < rp[i + 1]; ++p) {
            if (ci[p] < 0 || ci[p] >= cols) {
                std::snprintf(buf, sizeof buf,
                              "column index %d out of range in row %lld",
                              ci[p], (long long)i);
                put_msg(msg, msg_len, buf);
                return PDHG_E_CSR;
            }
            if (p > rp[i] && ci[p] <= ci[p - 1]) {
                std::snprintf(buf, sizeof buf,
                              "column indices not strictly increasing in "
                              "row %lld",
                              (long long)i);
                put_msg(msg, msg_len, buf);
                return PDHG_E_CSR;
            }
        }
    }
    return PDHG_OK;
}

// A^T's row j lists the rows i of A's column j in increasing order.  Walking
// A row by row and appending each (i, j) to a cursor per column therefore
// visits A^T's entries in storage order, which gives the permutation and
// the check in one O(nnz) pass.
extern "C" int pdhg_check_transpose(int64_t m, int64_t n, int64_t nnz,
                                    const int64_t *a_rp, const int32_t *a_ci,
                                    const double *a_v, const int64_t *at_rp,
                                    const int32_t *at_ci, const double *at_v,
                                    int64_t *perm, char *msg, int msg_len) {
    int rc = pdhg_validate_csr(m, n, nnz, a_rp, a_ci, msg, msg_len);
    if (rc != PDHG_OK) return rc;
    rc = pdhg_validate_csr(n, m, nnz, at_rp, at_ci, msg, msg_len);
    if (rc != PDHG_OK) return rc;
    if (nnz > 0 && (!a_v || !at_v)) {
        put_msg(msg, msg_len, "null value array");
        return PDHG_E_ARG;
    }
    std::vector<int64_t> cur(at_rp, at_rp + n);
    char buf[256];
    for (int64_t i = 0; i < m; ++i) {
        for (int64_t p = a_rp[i]; p < a_rp[i + 1]; ++p) {
            int32_t j = a_ci[p];
            int64_t q = cur[j]++;
            if (q >= at_rp[j + 1] || at_ci[q] != (int32_t)i ||
                std::memcmp(&at_v[q], &a_v[p], sizeof(double)) != 0) {
                std::snprintf(buf, sizeof buf,
                              "A^T differs from the transpose of A at "
                              "A(%lld,%d)",
                              (long long)i, j);
                put_msg(msg, msg_len, buf);
                return PDHG_E_TRANSPOSE;
            }
            if (perm) perm[p] = q;
        }
    }
    for (int64_t j = 0; j < n; ++j) {
        if (cur[j] != at_rp[j + 1]) {
            std::snprintf(buf, sizeof buf,
                          "A^T row %lld has entries absent from A",
                          (long long)j);
            put_msg(msg, msg_len, buf);
            return PDHG_E_TRANSPOSE;
        }
    }
    return PDHG_OK;
}

extern "C" int pdhg_plan_bins(int64_t rows, const int64_t *rp, int tile,
                              int64_t split_threshold, int64_t split_chunk,
                              int32_t *out, int64_t cap) {
    if (rows < 1 || !rp || tile < 1 || split_chunk < 1 ||
        split_threshold < tile)
        return PDHG_E_ARG;
    pdhg::HostBins hb =
        pdhg::build_row_blocks(rows, rp, tile, split_threshold, split_chunk);
    const int64_t k = (int64_t)hb.blocks.size();
    for (int64_t i = 0; i < k && i < cap && out; ++i) {
        out[4 * i + 0] = hb.blocks[i].r0;
        out[4 * i + 1] = hb.blocks[i].r1;
        out[4 * i + 2] = hb.blocks[i].part;
        out[4 * i + 3] = hb.blocks[i].nparts;
    }
    return (int)k;
}

extern "C" int pdhg_choose_panels(int64_t rows, int64_t cols, int64_t nnz) {
    if (rows < 1 || cols < 1 || nnz < 0) return PDHG_E_ARG;
    return pdhg::choose_panels(rows, cols, nnz);
}

extern "C" int pdhg_plan_panels(int64_t rows, int64_t cols, const int64_t *rp,
                                const int32_t *ci, int P, const int64_t *cut,
                                int tile, int64_t *srp, int32_t *src,
                                int32_t *out, int64_t cap) {
    if (rows < 1 || cols < 1 || !rp || !cut || tile < 1 ||
        !(P == 1 || P == 2 || P == 4 || P == 8) || !srp || !src ||
        (int64_t)P * rows >= ((int64_t)1 << 31))
        return PDHG_E_ARG;
    if (rp[rows] > 0 && !ci) return PDHG_E_ARG;
    if (cut[0] != 0 || cut[P] != cols) return PDHG_E_ARG;
    for (int p = 0; p < P; ++p)
        if (cut[p + 1] < cut[p]) return PDHG_E_ARG;
    std::vector<int64_t> vc(cut, cut + P + 1);
    pdhg::Panels S = pdhg::build_panels(rows, rp, ci, P, vc);
    std::memcpy(srp, S.rp.data(), S.rp.size() * sizeof(int64_t));
    if (!S.src.empty())
        std::memcpy(src, S.src.data(), S.src.size() * sizeof(int32_t));
    pdhg::HostBins hb = pdhg::build_panel_blocks(rows, S.rp.data(), P, tile,
                                                 (int64_t)1 << 40, (int64_t)1 << 20);
    const int64_t k = (int64_t)hb.blocks.size();
    for (int64_t i = 0; i < k && i < cap && out; ++i) {
        out[4 * i + 0] = hb.blocks[i].r0;
        out[4 * i + 1] = hb.blocks[i].r1;
        out[4 * i + 2] = hb.blocks[i].part;
        out[4 * i + 3] = hb.blocks[i].nparts;
    }
    return (int)k;
}

namespace pdhg {

// Row-length bins.  Consecutive rows are packed into multi-row blocks of at
// most `tile` nonzeros (and at most `tile` rows); a row longer than `tile`
// gets a workgroup of its own, and a row longer than split_threshold is cut
// into parts of split_chunk nonzeros on several workgroups.  Single-row and
// split blocks are placed first so that the longest work starts first.
HostBins build_row_blocks(int64_t rows, const int64_t *rp, int tile,
                          int64_t split_threshold, int64_t split_chunk,
                          int max_rows, bool skip_empty) {
    HostBins hb;
    // rows per multi-row block: at most `tile`, and at most max_rows if set
    const int64_t row_cap = max_rows > 0 ? std::min<int64_t>(tile, max_rows) : tile;
    std::vector<RowBlock> longb, multi;
    std::vector<std::pair<int64_t, int64_t>> singles;  // (len, row)
    int64_t r = 0;
    while (r < rows) {
        int64_t len = rp[r + 1] - rp[r];
        if (skip_empty && len == 0) {   // no block starts at an empty row
            ++r;
            continue;
        }
        if (len > tile) {
            if (len > split_threshold) {
                int nparts = (int)((len + split_chunk - 1) / split_chunk);
                for (int q = 0; q < nparts; ++q)
                    longb.push_back({(int32_t)r, (int32_t)(r + 1), q, nparts,
                                     hb.parts, 0, 0, 0});
                hb.splits.push_back({(int32_t)r, nparts, hb.parts});
                hb.parts += nparts;
                hb.counts[2] += nparts;
            } else {
                singles.push_back({len, r});
            }
            ++r;
            continue;
        }
        int64_t r1 = r, acc = 0;
        while (r1 < rows && (r1 - r) < row_cap) {
            int64_t l = rp[r1 + 1] - rp[r1];
            if (l > tile || acc + l > tile) break;
            acc += l;
            ++r1;
        }
        multi.push_back({(int32_t)r, (int32_t)r1, 0, 1, -1, 0, 0, 0});
        if (r1 - r == 1)
            hb.counts[1] += 1;
        else
            hb.counts[0] += 1;
        r = r1;
    }
    std::stable_sort(singles.begin(), singles.end(),
                     [](const std::pair<int64_t, int64_t> &a,
                        const std::pair<int64_t, int64_t> &b) {
                         return a.first > b.first;
                     });
    hb.blocks.reserve(longb.size() + singles.size() + multi.size());
    for (auto &b : longb) hb.blocks.push_back(b);
    for (auto &s : singles) {
        hb.blocks.push_back({(int32_t)s.second, (int32_t)(s.second + 1), 0, 1,
                             -1, 0, 0, 0});
        hb.counts[1] += 1;
    }
    for (auto &b : multi) hb.blocks.push_back(b);
    // nonzero range of each block, so that its loads need no row pointer
    for (auto &b : hb.blocks) {
        b.p0 = (int32_t)rp[b.r0];
        b.p1 = (int32_t)rp[b.r1];
    }
    return hb;
}

// fn(t) for every t below nt, on threads beside the caller's.  What one of them
// throws (it may run out of memory) reaches the caller once all have ended, and
// where no thread is to be had the caller does its share.
template <class Fn>
static void on_threads(int nt, Fn fn) {
    std::vector<std::future<void>> th;
    for (int t = 1; t < nt; ++t)
        th.push_back(std::async(std::launch::async | std::launch::deferred, [&fn, t] { fn(t); }));
    fn(0);
    for (auto &t : th) t.get();
}

// Internal relabeling: rows of A and columns of A in order of decreasing
// length (stable).  With rows sorted, the row-length bins of both A and A^T
// are contiguous runs; with columns sorted, the most-referenced entries of x
// sit together, so on skewed matrices most gathers of x hit a small region
// that stays in cache.  A' keeps each row's entries sorted by the new column
// index; A'^T is built from A' by one pass with a cursor per column.
//
// A dimension split into P > 1 panels (column panels of the gather table of
// one SpMV side, see choose_panels) is dealt rather than sorted when it is
// skewed: rank r of the decreasing-length order goes to panel r % P, so every
// panel holds the same number of entries and the same share of long ones,
// each panel still in decreasing-length order.  Unskewed dimensions keep
// their order and are cut into P equal ranges.
static std::vector<int64_t> deal(std::vector<int32_t> &order, int P) {
    const int64_t k = (int64_t)order.size();
    std::vector<int64_t> cut((size_t)P + 1, 0);
    for (int p = 0; p < P; ++p) cut[p + 1] = cut[p] + (k - p + P - 1) / P;
    std::vector<int32_t> dealt((size_t)k);
    for (int64_t r = 0; r < k; ++r) dealt[cut[r % P] + r / P] = order[r];
    order.swap(dealt);
    return cut;
}

static std::vector<int64_t> even_cuts(int64_t k, int P) {
    std::vector<int64_t> cut((size_t)P + 1);
    for (int p = 0; p <= P; ++p) cut[p] = k * p / P;
    return cut;
}

Relabeled relabel(int64_t m, int64_t n, int64_t nnz, const int64_t *a_rp,
                  const int32_t *a_ci, const double *a_v,
                  const int64_t *at_rp, int panels_a, int panels_at,
                  int sort_rows, int sort_cols) {
    Relabeled R;
    R.pr.resize((size_t)m);
    R.pc.resize((size_t)n);
    std::iota(R.pr.begin(), R.pr.end(), 0);
    std::iota(R.pc.begin(), R.pc.end(), 0);
    // a dimension is reordered only when its lengths are skewed (longest
    // more than kSkew times the mean); otherwise its given order, which may
    // carry locality of its own, is kept
    auto skewed = [](const int64_t *rp, int64_t k) {
        int64_t mx = 0;
        for (int64_t i = 0; i < k; ++i) mx = std::max(mx, rp[i + 1] - rp[i]);
        return k > 0 && (double)mx > kSkew * (double)rp[k] / (double)k;
    };
    // sort_rows / sort_cols: -1 decides by skew, 0 keeps, 1 sorts
    R.sorted_rows = sort_rows < 0 ? skewed(a_rp, m) : sort_rows == 1;
    R.sorted_cols = sort_cols < 0 ? skewed(at_rp, n) : sort_cols == 1;
    if (R.sorted_rows)
        std::stable_sort(R.pr.begin(), R.pr.end(), [&](int32_t a, int32_t b) {
            return a_rp[a + 1] - a_rp[a] > a_rp[b + 1] - a_rp[b];
        });
    if (R.sorted_cols)
        std::stable_sort(R.pc.begin(), R.pc.end(), [&](int32_t a, int32_t b) {
            return at_rp[a + 1] - at_rp[a] > at_rp[b + 1] - at_rp[b];
        });
    // panels of A's columns (the table the dual step gathers) and of A^T's
    // columns, i.e. A's rows (the table the primal step gathers)
    R.a_cut = (R.sorted_cols && panels_a > 1) ? deal(R.pc, panels_a)
                                              : even_cuts(n, panels_a);
    R.at_cut = (R.sorted_rows && panels_at > 1) ? deal(R.pr, panels_at)
                                                : even_cuts(m, panels_at);
    std::vector<int32_t> ic((size_t)n), ir((size_t)m);
    for (int64_t j = 0; j < n; ++j) ic[R.pc[j]] = (int32_t)j;
    for (int64_t i = 0; i < m; ++i) ir[R.pr[i]] = (int32_t)i;
    R.a_rp.assign((size_t)m + 1, 0);
    for (int64_t i = 0; i < m; ++i)
        R.a_rp[i + 1] = R.a_rp[i] + (a_rp[R.pr[i] + 1] - a_rp[R.pr[i]]);
    R.a_ci.resize((size_t)nnz);
    R.a_v.resize((size_t)nnz);
    R.apos.resize((size_t)nnz);
    // rows are independent: fill them on a few host threads
    const bool same_cols = !R.sorted_cols;    // the columns keep their order
    auto fill_rows = [&](int64_t lo, int64_t hi) {
        std::vector<std::pair<int32_t, int32_t>> tmp;
        for (int64_t i2 = lo; i2 < hi; ++i2) {
            const int64_t i = R.pr[i2];
            const int64_t p0 = a_rp[i], L = a_rp[i + 1] - p0;
            if (same_cols) {
                const int64_t o = R.a_rp[i2];
                for (int64_t q = 0; q < L; ++q) {
                    R.a_ci[o + q] = a_ci[p0 + q];
                    R.a_v[o + q] = a_v[p0 + q];
                    R.apos[o + q] = (int32_t)(p0 + q);
                }
                continue;
            }
            tmp.resize((size_t)L);
            for (int64_t q = 0; q < L; ++q)
                tmp[q] = {ic[a_ci[p0 + q]], (int32_t)(p0 + q)};
            std::sort(tmp.begin(), tmp.end());
            const int64_t o = R.a_rp[i2];
            for (int64_t q = 0; q < L; ++q) {
                R.a_ci[o + q] = tmp[q].first;
                R.a_v[o + q] = a_v[tmp[q].second];
                R.apos[o + q] = tmp[q].second;
            }
        }
    };
    const int nt = (int)std::max<int64_t>(1, std::min<int64_t>(8, nnz / 100000));
    if (nt == 1) {
        fill_rows(0, m);
    } else {
        on_threads(nt, [&](int t) { fill_rows(m * t / nt, m * (t + 1) / nt); });
    }
    R.at_rp.assign((size_t)n + 1, 0);
    for (int64_t j = 0; j < n; ++j)
        R.at_rp[j + 1] = R.at_rp[j] + (at_rp[R.pc[j] + 1] - at_rp[R.pc[j]]);
    R.at_ci.resize((size_t)nnz);
    R.at_v.resize((size_t)nnz);
    R.perm.resize((size_t)nnz);
    std::vector<int64_t> cur(R.at_rp.begin(), R.at_rp.end() - 1);
    for (int64_t i = 0; i < m; ++i)
        for (int64_t p = R.a_rp[i]; p < R.a_rp[i + 1]; ++p) {
            const int64_t q = cur[R.a_ci[p]]++;
            R.at_ci[q] = (int32_t)i;
            R.at_v[q] = R.a_v[p];
            R.perm[p] = (int32_t)q;
        }
    (void)ir;
    return R;
}

// Column panels and XCD affinity.  A random gather is served at a rate that
// falls steeply once its table no longer fits the 4 MB L2 of one XCD.
// Measured on MI355X, random 8-byte gathers per second by table size:
// <= 2 MB 195e9, 4 MB 180e9, 8 MB 110e9, 16 MB 77e9, 32 MB 63e9,
// >= 128 MB 54e9.  The same gathers confined per XCD to 1/P of the table run
// at the rate of the smaller table.  So an SpMV whose table overflows L2 is
// split into P column panels, each handled only by the workgroups that the
// hardware places on the XCDs x with x % P == p (workgroups go to the 8 XCDs
// round-robin by workgroup index).  The price is P stacked rows per row,
// each with its row pointer, its partial sum written and read once, and its
// share of the per-row work of the row-block kernel: measured, about 7 ps
// per stacked row on the whole chip, plus one extra launch that adds the
// partial sums.  Short rows over a table that fits L2 therefore stay whole.
static double gather_rate(double bytes) {
    static const double mb[] = {2, 4, 8, 16, 32, 128};
    static const double g[] = {195e9, 180e9, 110e9, 77e9, 63e9, 54e9};
    const double x = bytes / 1048576.0;
    if (x <= mb[0]) return g[0];
    for (int i = 1; i < 6; ++i)
        if (x <= mb[i]) {
            const double f = std::log(x / mb[i - 1]) / std::log(mb[i] / mb[i - 1]);
            return g[i - 1] * std::pow(g[i] / g[i - 1], f);
        }
    return g[5];
}

int choose_panels(int64_t rows, int64_t cols, int64_t nnz) {
    constexpr double kRow = 7e-12;        // seconds per stacked row
    constexpr double kLaunch = 4e-6;      // the extra launch, seconds
    const double table = 8.0 * (double)cols;
    const double whole = (double)nnz / gather_rate(table);
    double best = 0.95 * whole;           // a split must win clearly
    int bestP = 1;
    for (int P = 2; P <= 8; P *= 2) {
        const double t = (double)nnz / gather_rate(table / P) +
                         kRow * P * (double)rows + kLaunch;
        if (t < best) {
            best = t;
            bestP = P;
        }
    }
    return bestP;
}

// The stacked matrix of P column panels: row p * rows + i holds the entries
// of row i with column in [cut[p], cut[p + 1]) (a contiguous run, since
// columns are sorted within rows); src maps each entry to its position in
// the source arrays.
Panels build_panels(int64_t rows, const int64_t *rp, const int32_t *ci, int P,
                    const std::vector<int64_t> &cut) {
    Panels S;
    const int64_t nnz = rp[rows];
    S.rp.assign((size_t)P * rows + 1, 0);
    std::vector<int64_t> start((size_t)P * rows + 1);
    for (int64_t i = 0; i < rows; ++i) {
        int64_t q = rp[i];
        for (int p = 0; p < P; ++p) {
            start[(size_t)p * rows + i] = q;
            const int64_t e = rp[i + 1];
            int64_t q1 = q;
            while (q1 < e && ci[q1] < cut[p + 1]) ++q1;
            S.rp[(size_t)p * rows + i + 1] = q1 - q;   // length for now
            q = q1;
        }
    }
    S.mask.assign((size_t)rows, 0);
    for (int p = 0; p < P; ++p)
        for (int64_t i = 0; i < rows; ++i)
            if (S.rp[(size_t)p * rows + i + 1] > 0) S.mask[i] |= (uint8_t)(1u << p);
    for (int64_t r = 0; r < (int64_t)P * rows; ++r) S.rp[r + 1] += S.rp[r];
    S.ci.resize((size_t)nnz);
    S.src.resize((size_t)nnz);
    for (int64_t r = 0; r < (int64_t)P * rows; ++r) {
        const int64_t o = S.rp[r], L = S.rp[r + 1] - o, q0 = start[r];
        for (int64_t t = 0; t < L; ++t) {
            S.ci[o + t] = ci[q0 + t];
            S.src[o + t] = (int32_t)(q0 + t);
        }
    }
    return S;
}

// Row blocks of the stacked matrix, built per panel and dealt to the XCDs:
// the blocks of panel p are spread over the XCDs x with x % P == p, and the
// launch order puts XCD x's i-th block at index 8 i + x (empty blocks, r0 ==
// r1, pad queues of unequal length).  Split slots are renumbered to be global.
// No block starts at an empty stacked row, so runs of them (a row whose
// entries all lie in other panels, as in block-structured LPs) cost no
// blocks; the combine reads only the partials of a row's non-empty panels.
HostBins build_panel_blocks(int64_t rows, const int64_t *srp, int P, int tile,
                            int64_t split_threshold, int64_t split_chunk,
                            int max_rows) {
    constexpr int kXcd = 8;
    HostBins out;
    std::vector<std::vector<RowBlock>> q(kXcd);
    for (int p = 0; p < P; ++p) {
        HostBins hb = build_row_blocks(rows, srp + (size_t)p * rows, tile,
                                       split_threshold, split_chunk, max_rows,
                                       true);
        const int32_t roff = (int32_t)((int64_t)p * rows);
        const int32_t slot0 = out.parts;
        for (auto sp : hb.splits) {
            sp.row += roff;
            sp.first += slot0;
            out.splits.push_back(sp);
        }
        out.parts += hb.parts;
        for (int k = 0; k < 3; ++k) out.counts[k] += hb.counts[k];
        const int per = kXcd / P;     // XCDs serving this panel
        for (size_t b = 0; b < hb.blocks.size(); ++b) {
            RowBlock rb = hb.blocks[b];
            rb.r0 += roff;
            rb.r1 += roff;
            if (rb.nparts > 1) rb.slot += slot0;
            q[p + P * (int)(b % per)].push_back(rb);
        }
    }
    size_t depth = 0;
    for (auto &v : q) depth = std::max(depth, v.size());
    out.blocks.reserve(depth * kXcd);
    for (size_t i = 0; i < depth; ++i)
        for (int x = 0; x < kXcd; ++x)
            out.blocks.push_back(i < q[x].size() ? q[x][i]
                                                 : RowBlock{0, 0, 0, 1, -1, 0, 0, 0});
    return out;
}

constexpr int64_t kBktCus = 256;

// Cost of rows [r0, r1) to a bucket: its nonzeros, and the epilogue's operands
// of a row (40 to 56 bytes) as three more.
static int64_t bucket_cost(const int64_t *rp, int64_t r0, int64_t r1) {
    return rp[r1] - rp[r0] + 3 * (r1 - r0);
}

// Rounds of one bucket of at most `cap` nonzeros on each CU.
static int64_t bucket_rounds(int64_t cost, int64_t nnz, int64_t cap) {
    const int64_t round = kBktCus * cap;
    return std::max<int64_t>(1, std::max((nnz + round - 1) / round, (cost + 2 * round - 1) / (2 * round)));
}

// Cost per bucket: equal shares of whole rounds.
static int64_t bucket_fill(int64_t cost, int64_t rounds) {
    return (int64_t)(1.01 * (double)cost / (double)(kBktCus * rounds)) + 64;
}

// Consecutive rows of [row0, row1) packed into buckets of about cost `fill`
// and at most `cap` nonzeros; a longer row is cut into parts.  skip_empty:
// no bucket starts at an empty row.
static void pack_buckets(HostBuckets &B, int64_t row0, int64_t row1,
                         const int64_t *rp, int64_t fill, int64_t cap, bool skip_empty) {
    for (int64_t r = row0; r < row1;) {
        const int64_t len = rp[r + 1] - rp[r];
        if (skip_empty && len == 0) {
            ++r;
            continue;
        }
        if (len > cap) {
            const int np = (int)((len + cap - 1) / cap);
            const int64_t chunk = (len + np - 1) / np;
            for (int q = 0; q < np; ++q) {
                const int64_t a = rp[r] + q * chunk, e = std::min(rp[r + 1], a + chunk);
                B.buckets.push_back({(int32_t)r, (int32_t)(r + 1), (int32_t)a,
                                     (int32_t)e, 0, 0, B.parts, q});
            }
            B.splits.push_back({(int32_t)r, np, B.parts});
            B.parts += np;
            ++r;
            continue;
        }
        // G lanes (a power of two, at most 64) sum each of R rows: no row may
        // keep its lanes longer than 64 steps because of many short ones
        int64_t r1 = r + 1, longest = len;
        while (r1 < row1 && rp[r1 + 1] - rp[r] <= cap &&
               bucket_cost(rp, r, r1 + 1) <= fill) {
            const int64_t mx = std::max(longest, rp[r1 + 1] - rp[r1]);
            const int64_t G = std::min<int64_t>(64, kBktThreads / (r1 + 1 - r));
            if (mx > 64 && mx > 64 * G && G < 64) break;
            longest = mx;
            ++r1;
        }
        B.buckets.push_back({(int32_t)r, (int32_t)r1, (int32_t)rp[r], (int32_t)rp[r1], 0, 0, -1, 0});
        r = r1;
    }
}

// Stable sort by the high 32 bits (below 2^31), in radix passes of as many bits
// as give each key a counter, at most 11 (always 11: a plan of 55,000 nonzeros in
// buckets of 256 took 1.5 ms against 0.6).
static void sort_high(std::vector<uint64_t> &key, std::vector<uint64_t> &tmp) {
    constexpr int kMost = 11;
    uint64_t lo = ~0ull, hi = 0;
    for (uint64_t k : key) {
        lo = std::min(lo, k >> 32);
        hi = std::max(hi, k >> 32);
    }
    tmp.resize(key.size());
    int bits = 4;
    while (bits < kMost && (size_t)1 << bits < key.size()) ++bits;
    const uint64_t mask = ((uint64_t)1 << bits) - 1;
    for (int sh = 0; key.size() > 1 && sh < 32 && ((hi - lo) >> sh) != 0; sh += bits) {
        uint32_t at[(1 << kMost) + 1];
        std::fill(at, at + mask + 2, 0);
        auto digit = [&](uint64_t k) { return (((k >> 32) - lo) >> sh) & mask; };
        for (uint64_t k : key) ++at[digit(k) + 1];
        for (uint64_t d = 0; d <= mask; ++d) at[d + 1] += at[d];
        for (uint64_t k : key) tmp[at[digit(k)]++] = k;
        key.swap(tmp);
    }
}

// fn(b0, b1) over the buckets [0, nb) on a few threads.
template <class Fn>
static void over_buckets(int64_t nb, int64_t nnz, Fn fn) {
    const int nt = (int)std::max<int64_t>(1, std::min<int64_t>(8, nnz / 50000));
    on_threads(nt, [&](int t) { fn(nb * t / nt, nb * (t + 1) / nt); });
}

// Push buckets.  Columns are cut into blocks, as many as divide a round of one
// workgroup per CU or are divided by it (303 blocks of 16,384 columns of the
// multicommodity dual left the second round nearly empty, 114 us a step
// against 99 with 256; 610 blocks of the 55M-nonzero coupled one 468 us
// against 420 with 512).  The nonzeros of one (column block, bucket) pair form
// a run, padded to whole quads: the push pass walks the runs of a column block
// one after the other, and each run is contiguous among its bucket's products.
HostBuckets build_push(int64_t rows, int64_t cols, const int64_t *rp,
                       const int32_t *ci, bool force) {
    HostBuckets B;
    const int64_t nnz = rp[rows], cost = bucket_cost(rp, 0, rows);
    int64_t ncb = 1;
    while (ncb * kBktCols < cols) ncb = ncb < kBktCus ? 2 * ncb : ncb + kBktCus;
    // (whole 16-byte units of the vector)
    B.width = (int)std::min<int64_t>(kBktCols, ((cols + ncb - 1) / ncb + 3) / 4 * 4);
    ncb = (cols + B.width - 1) / B.width;
    const int64_t fill = bucket_fill(cost, bucket_rounds(cost, nnz, kBktCap));
    pack_buckets(B, 0, rows, rp, fill, kBktCap, false);
    const int64_t nb = (int64_t)B.buckets.size();
    B.fragmented = nb > 2 * (cost / fill) + 64;
    if (B.fragmented && !force) return B;
    // quads of each run; then the runs' places in both orders
    std::vector<int32_t> run((size_t)(ncb * nb)), at((size_t)(ncb * nb));
    over_buckets(nb, nnz, [&](int64_t b0, int64_t b1) {
        std::vector<int32_t> cnt((size_t)ncb);
        for (int64_t b = b0; b < b1; ++b) {
            std::fill(cnt.begin(), cnt.end(), 0);
            for (int64_t p = B.buckets[b].p0; p < B.buckets[b].p1; ++p) ++cnt[ci[p] / B.width];
            for (int64_t k = 0; k < ncb; ++k) run[k * nb + b] = (cnt[k] + 3) / 4;
        }
    });
    std::vector<int64_t> cq((size_t)ncb + 1, 0);
    int64_t q = 0;
    for (int64_t k = 0; k < ncb; ++k) {
        for (int64_t b = 0; b < nb; ++b) {
            at[k * nb + b] = (int32_t)q;
            q += run[k * nb + b];
        }
        cq[k + 1] = q;
    }
    B.quads = q;
    q = 0;
    for (int64_t b = 0; b < nb; ++b) {
        B.buckets[b].q0 = (int32_t)q;
        for (int64_t k = 0; k < ncb; ++k) q += run[k * nb + b];
        B.buckets[b].q1 = (int32_t)q;
    }
    B.col.assign((size_t)(4 * B.quads), 0);
    B.pos.assign((size_t)(4 * B.quads), (uint16_t)kBktCap);
    B.src.assign((size_t)(4 * B.quads), -1);
    B.dest.resize((size_t)B.quads);
    over_buckets(nb, nnz, [&](int64_t b0, int64_t b1) {
        std::vector<int64_t> c1((size_t)ncb), c2((size_t)ncb);
        for (int64_t b = b0; b < b1; ++b) {
            const Bucket &K = B.buckets[b];
            int64_t o = K.q0;
            for (int64_t k = 0; k < ncb; ++k) {
                const int64_t a = at[k * nb + b], n = run[k * nb + b];
                for (int64_t i = 0; i < n; ++i) B.dest[a + i] = (int32_t)(o + i);
                c1[k] = 4 * a;
                c2[k] = 4 * o;
                o += n;
            }
            for (int64_t p = K.p0; p < K.p1; ++p) {
                const int64_t k = ci[p] / B.width;
                B.col[c1[k]] = (uint16_t)(ci[p] % B.width);
                B.src[c1[k]++] = (int32_t)p;
                B.pos[c2[k]++] = (uint16_t)(p - K.p0);
            }
        }
    });
    // items: slices of single blocks, of equal size and as many as fill whole
    // rounds (at most four); each XCD (workgroups go to the 8 XCDs
    // round-robin) takes neighbouring ones, so that runs that share lines of
    // the products are written through one L2
    constexpr int64_t kXcd = 8;
    const int64_t want = kBktCus * std::max<int64_t>(1, std::min<int64_t>(4, B.quads / (kBktCus * 8192)));
    auto count = [&](int64_t S) {
        int64_t n = 0;
        for (int64_t k = 0; k < ncb; ++k) n += (cq[k + 1] - cq[k] + S - 1) / S;
        return n;
    };
    int64_t lo = 1, hi = std::max<int64_t>(1, B.quads);
    const int64_t most = std::max<int64_t>(want, count(hi));
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (count(mid) <= most) hi = mid; else lo = mid + 1;
    }
    std::vector<PushItem> it;
    for (int64_t k = 0; k < ncb; ++k) {
        const int64_t len = cq[k + 1] - cq[k], ns = (len + lo - 1) / lo;
        for (int64_t i = 0; i < ns; ++i)
            it.push_back({(int32_t)k, (int32_t)(cq[k] + len * i / ns), (int32_t)(cq[k] + len * (i + 1) / ns), 0});
    }
    const int64_t ni = (int64_t)it.size(), per = (ni + kXcd - 1) / kXcd;
    for (int64_t i = 0; i < per; ++i)
        for (int64_t x = 0; x < kXcd; ++x)
            B.items.push_back(x * per + i < ni ? it[x * per + i] : PushItem{0, 0, 0, 0});
    return B;
}

// Tiles.  A tile's nonzeros are kept in column order, so that neighbouring
// lanes gather from neighbouring lines; its products go to their CSR positions
// in LDS.  Position and column share 32 bits, the column relative to a base
// per group of 64 quads (48 bits: 9M nonzeros 53 us a step against 46, FP32 36
// against 26, 16,384 nonzeros a tile included).  Within a group of 64 quads lane l's quad holds the entries l,
// l + 64, l + 128 and l + 192 of that order: each of the four gathers of a
// wave then covers 64 neighbours.  Tiles of panel p are dealt to the XCDs x
// with x % P == p (r0 == r1 pads queues of unequal length).
HostBuckets build_tiles(int64_t rows, const int64_t *rp, const int32_t *ci,
                        int P, bool force) {
    constexpr int kXcd = 8;
    HostBuckets B;
    const int64_t nnz = rp[P * rows], cost = bucket_cost(rp, 0, P * rows);
    std::vector<int64_t> first;
    int64_t fill = 0, nb = 0;
    // one round more where long rows fill more buckets than the rounds hold
    for (int64_t nr = bucket_rounds(cost, nnz, kTileCap), k = 0; k < 2; ++k) {
        fill = bucket_fill(cost, nr + k);
        B = HostBuckets();
        first.clear();
        for (int p = 0; p < P; ++p) {
            first.push_back((int64_t)B.buckets.size());
            pack_buckets(B, p * rows, (p + 1) * rows, rp, fill, kTileCap, P > 1);
        }
        nb = (int64_t)B.buckets.size();
        first.push_back(nb);
        if (nb <= kBktCus * (nr + k)) break;
    }
    B.fragmented = nb > 2 * (cost / fill) + 64;
    if (B.fragmented && !force) return B;
    // groups of 64 quads: a full one, one that the next column's offset does
    // not fit, or the last
    constexpr int64_t kGroup = 256, kSpan = (int64_t)1 << (32 - kTilePos);
    over_buckets(nb, nnz, [&](int64_t b0, int64_t b1) {
        for (int64_t b = b0; b < b1; ++b) {
            Bucket &K = B.buckets[b];
            const auto mm = std::minmax_element(ci + K.p0, ci + K.p1);
            K.q1 = K.p0 == K.p1 ? 0 : (int32_t)(64 * ((K.p1 - K.p0) / kGroup + (*mm.second - *mm.first) / kSpan + 1));
        }
    });
    int64_t q = 0;
    for (auto &b : B.buckets) {
        b.q0 = (int32_t)q;
        q += b.q1;
    }
    B.quads = q;
    B.word.assign((size_t)(4 * q), 0);
    B.base.assign((size_t)(q / 64), 0);
    B.first.assign((size_t)(q / 64), 0);
    over_buckets(nb, nnz, [&](int64_t b0, int64_t b1) {
        std::vector<uint64_t> key, tmp;
        for (int64_t b = b0; b < b1; ++b) {
            Bucket &K = B.buckets[b];
            const int64_t nz = K.p1 - K.p0;
            key.resize((size_t)nz);
            for (int64_t t = 0; t < nz; ++t)
                key[t] = (uint64_t)(uint32_t)ci[K.p0 + t] << 32 | (uint64_t)t;
            sort_high(key, tmp);
            K.q1 = K.q0;
            for (int64_t t = 0; t < nz;) {
                const int64_t c0 = (int64_t)(key[t] >> 32);
                int64_t n = 1;
                while (n < kGroup && t + n < nz && (int64_t)(key[t + n] >> 32) - c0 < kSpan) ++n;
                // neighbours in the order on neighbouring lanes (L of them)
                const int64_t L = t + n < nz ? 64 : (n + 3) / 4;
                int64_t i = t;
                for (int64_t u = 0; u < 4; ++u)
                    for (int64_t l = 0; l < L; ++l, ++i) {
                        const uint64_t e = key[std::min(i, t + n - 1)];
                        const int64_t o = 4 * (K.q1 + l) + u, p = (int64_t)(e & 0xffffffffu);
                        B.word[o] = (int32_t)((uint32_t)((int64_t)(e >> 32) - c0) << kTilePos | (uint32_t)p);
                    }
                B.base[K.q1 / 64] = (int32_t)c0;
                B.first[K.q1 / 64] = K.p0;
                K.q1 += (int32_t)L;
                t += n;
            }
        }
    });
    std::vector<std::vector<Bucket>> xq(kXcd);
    const int per = kXcd / P;
    for (int p = 0; p < P; ++p)
        for (int64_t i = 0; i < first[p + 1] - first[p]; ++i)
            xq[p + P * (int)(i % per)].push_back(B.buckets[first[p] + i]);
    size_t depth = 0;
    for (auto &v : xq) depth = std::max(depth, v.size());
    B.buckets.clear();
    for (size_t i = 0; i < depth; ++i)
        for (int x = 0; x < kXcd; ++x)
            B.buckets.push_back(i < xq[x].size() ? xq[x][i] : Bucket{0, 0, 0, 0, 0, 0, -1, 0});
    return B;
}

HostSmall build_small(int64_t rows, int64_t cols, const int64_t *rp,
                      const int32_t *ci) {
    HostSmall S;
    S.G = 64;
    while (S.G > 1 && S.G * rows > kSmallThreads) S.G >>= 1;
    const int64_t per = kSmallThreads / S.G;     // rows per slot
    S.K = (int)((rows + per - 1) / per);
    std::vector<int32_t> order((size_t)rows);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return rp[a + 1] - rp[a] > rp[b + 1] - rp[b];
    });
    S.row.assign((size_t)(S.K * per), -1);
    for (int64_t r = 0; r < rows; ++r) {
        // every second slot from the other end: long rows next to short ones
        const int64_t k = r / per, i = r % per;
        S.row[k * per + (k & 1 ? per - 1 - i : i)] = order[r];
    }
    S.off.assign(1, 0);
    for (int64_t sl = 0; sl < (int64_t)S.K * kSmallWaves; ++sl) {
        int64_t steps = 0;
        for (int64_t l = 0; l < 64; l += S.G) {
            const int32_t r = S.row[(sl * 64 + l) / S.G];
            if (r >= 0) steps = std::max(steps, (rp[r + 1] - rp[r] + S.G - 1) / S.G);
        }
        S.off.push_back(S.off.back() + (int32_t)((steps + 1) / 2));
    }
    S.src.assign((size_t)S.off.back() * 128, -1);
    S.col.assign((size_t)S.off.back() * 128, (uint16_t)cols);
    for (int64_t sl = 0; sl < (int64_t)S.K * kSmallWaves; ++sl)
        for (int64_t l = 0; l < 64; ++l) {
            const int32_t r = S.row[(sl * 64 + l) / S.G];
            if (r < 0) continue;
            // lane g of the row's G takes entries g, g + G, ...
            int64_t step = 0;
            for (int64_t p = rp[r] + l % S.G; p < rp[r + 1]; p += S.G, ++step) {
                const int64_t e = ((S.off[sl] + step / 2) * 64 + l) * 2 + step % 2;
                S.src[e] = (int32_t)p;
                S.col[e] = (uint16_t)ci[p];
            }
        }
    return S;
}

// Which layout a side runs in, from its sizes (P: its column panels).  A
// gather costs a line from L2 to the CU; a tile shares a line among its
// gathers, which pays while a panel's part of the vector has few more lines
// than a tile has nonzeros, and stacked rows are not short.  Pushing the
// products costs 17 (FP64) or 9 (FP32) more bytes per nonzero and a second
// launch, but gathers from LDS only; its runs shorten as the columns grow.
// Measured, us a step, rows | tiles | push (FP64; FP32):
//   power-law primal, 9.4M nonzeros, 1.6 MB:  65 | 51 | 65;  51 | 31 | 40
//   ... dual, 8 MB in 4 panels, 47 a row:     63 | 45 | 65;  47 | 29 | 40
//   1M x 400k primal, 8M, 3.2 MB:             65 | 50 | 56;  51 | 32 | 35
//   ... dual, 8 MB, 20 a row:                 72 | 55 | 55;  54 | 37 | 34
//   700k x 600k primal, 9.8M, 4.8 MB:         83 | 59 | 65;  62 | 38 | 41
//   ... dual, 5.6 MB:                         89 | 65 | 67;  63 | 41 | 40
//   multicommodity primal, 14.6M, 10.8 MB:   134 | 117 | 120;  98 | 73 | 71
//   ... dual, 40 MB in 8 panels:             145 | 141 | 100; 100 | 98 | 58
//   840k-column one, primal, 2.4M, 1.9 MB:    23 | 19 | 28;  21 | 14 | 19
//   600k x 200k dual, 2.4M, 4.8 MB:           28 | 21 | 26;  21 | 17 | 18
//   power-law 300k dual, 2.8M, 2.4 MB:        21 | 16 | 26;  18 | 13 | 19
//   400k x 160k dual, 1.2M, 3.2 MB:           16 | 14 | 18;  14 | 12 | 13
//   2M x 1M dual, 24M, 16 MB:                199 | 165 | 148; 151 | 115 | 83
//   ... primal, 8 MB:                        200 | 166 | 143; 151 | 118 | 83
//   coupled dual, 55M, 80 MB in 8 panels:    709 | 550 | 420; 427 | 390 | 210
//   ... primal, 20 MB in 4 panels:           643 | 580 | 421; 487 | 394 | 214
//   ... dual, 110M, 160 MB in 8 panels:     1740 | 1469 | 982; 1250 | 971 | 540
//   ... primal, 40 MB in 4 panels:          1599 | 1246 | 1005; 1038 | 865 | 547
// and panelled sides of uniform LPs, the second of a multicommodity one
// (nonzeros, MB a panel, nonzeros a stacked row):
//   2.2M, 4.20,  5.5:  30 | 24 | 24; 24 | 19 | 17    5.0M, 3.81, 12.5:  47 | 40 | 39; 41 | 28 | 26
//   2.4M, 3.35,  5.1:  30 | 25 | 26; 21 | 19 | 18    5.2M, 2.48,  3.3:  42 | 43 | 41; 36 | 30 | 26
//   3.3M, 4.20,  5.5:  38 | 30 | 30; 33 | 23 | 21    5.6M, 2.67, 11.7:  40 | 40 | 41; 38 | 27 | 26
//   3.9M, 2.48,  9.8:  32 | 28 | 30; 30 | 21 | 21    7.5M, 2.38,  6.3:  62 | 52 | 52; 46 | 33 | 33
//   4.0M, 1.91, 10.0:  32 | 27 | 31; 30 | 20 | 22    8.4M, 2.29, 10.5:  58 | 51 | 57; 49 | 32 | 36
//   4.8M, 2.29,  4.8:  37 | 32 | 40; 35 | 24 | 26    9.6M, 2.29,  6.0:  76 | 61 | 66; 55 | 36 | 40
//   5.0M, 2.38, 10.4:  38 | 38 | 39; 36 | 27 | 27   10.4M, 2.48,  3.7:  93 | 83 | 69; 64 | 50 | 42
//   7.0M, 3.81, 11.7:  62 | 49 | 50; 49 | 34 | 31   11.6M, 2.77,  9.7:  92 | 78 | 74; 66 | 51 | 45
//   7.7M, 4.20,  7.7:  73 | 56 | 53; 53 | 37 | 33   23.2M, 2.77, 11.6: 173 | 137 | 139; 145 | 98 | 80
// So panels take tiles up to 2.5 MB and from four nonzeros a stacked row on, and
// below 2M nonzeros, where the alternative is row blocks, up to what an
// unpanelled side takes.
int choose_layout(int64_t rows, int64_t cols, int64_t nnz, int P) {
    constexpr double kMiB = 1048576.0;
    const double panel = 8.0 * (double)cols / P;
    if (nnz < kTileMin32) return LAYOUT_ROWS;
    if (panel <= (P == 1 || nnz < 2000000 ? 5.5 : 2.5) * kMiB &&
        (P == 1 || nnz >= 4 * (int64_t)P * rows))
        return LAYOUT_TILES;
    // runs of eight nonzeros or more (41M columns)
    const bool runs = (cols + kBktCols - 1) / kBktCols <= kBktCap / 8;
    return nnz >= 2000000 && runs ? LAYOUT_PUSH : LAYOUT_ROWS;
}

}  // namespace pdhg
