// Plans of the bucketed SpMV layouts (push and tiles), executed on the host as
// the kernels execute them and compared with the plain CSR product on integer
// data (exact).  Every index is checked against its buffer.  Then the planners
// run out of memory at every allocation.  Prints one line per matrix and layout.
#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>

#include "internal.h"

using namespace pdhg;

#define CHECK(c)                                                   \
    do {                                                           \
        if (!(c)) {                                                \
            std::printf("FAILED %s line %d\n", #c, __LINE__);      \
            std::exit(1);                                          \
        }                                                          \
    } while (0)

// Allocations fail once `left` are made, on whichever thread.
static std::atomic<long> left{LONG_MAX};
void *operator new(size_t n) {
    void *p = left.fetch_sub(1) > 0 ? std::malloc(n ? n : 1) : nullptr;
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace {

struct Csr {
    int64_t m, n;
    std::vector<int64_t> rp{0};
    std::vector<int32_t> ci;
};

// kind 0: even lengths; 1: every 97th row 60 times longer; 2: empty stretches
// and one full row; 3: a row 1,500 times longer among every 40
Csr make(int64_t m, int64_t n, double avg, int kind, std::mt19937_64 &g) {
    Csr A{m, n};
    for (int64_t i = 0; i < m; ++i) {
        double a = avg;
        if (kind == 1 && i % 97 == 0) a *= 60;
        if (kind == 2 && (i / 20000) % 2) a = 0;
        if (kind == 3 && i % 40 == 0) a *= 1500;
        int64_t L = std::min<int64_t>(n, (int64_t)(a * (0.5 + (double)(g() % 1000) / 1000.0) + 0.5));
        if (kind == 2 && i == 77) L = n;
        std::vector<int32_t> r;
        for (int64_t k = 0; k < L; ++k) r.push_back(L == n ? (int32_t)k : (int32_t)(g() % n));
        std::sort(r.begin(), r.end());
        r.erase(std::unique(r.begin(), r.end()), r.end());
        A.ci.insert(A.ci.end(), r.begin(), r.end());
        A.rp.push_back((int64_t)A.ci.size());
    }
    return A;
}

// Rows of a bucket summed from its products in LDS order.
void sum_rows(const Bucket &b, const std::vector<double> &s,
              const std::vector<int64_t> &rp, std::vector<double> &part,
              std::vector<double> &y) {
    if (b.slot >= 0) {
        double t = 0;
        for (int64_t p = 0; p < b.p1 - b.p0; ++p) t += s[p];
        const size_t k = (size_t)(b.slot + b.part);
        CHECK(k < part.size() && std::isnan(part[k]));
        part[k] = t;
        return;
    }
    for (int64_t r = b.r0; r < b.r1; ++r) {
        double t = 0;
        CHECK(rp[r] >= b.p0 && rp[r + 1] <= b.p1);
        for (int64_t p = rp[r]; p < rp[r + 1]; ++p) t += s[p - b.p0];
        CHECK(std::isnan(y[r]));
        y[r] = t;
    }
}

// Every partial sum belongs to one row, none is left over.
void finish(const std::vector<SplitRow> &splits, const std::vector<double> &part, std::vector<double> &y) {
    size_t used = 0;
    for (const SplitRow &r : splits) {
        double q = 0;
        CHECK((size_t)r.first == used && used + r.nparts <= part.size());
        for (int k = 0; k < r.nparts; ++k) q += part[r.first + k];
        used += r.nparts;
        y[r.row] = q;
    }
    CHECK(used == part.size());
}

// The same of the row blocks' split rows.
void check_blocks(const HostBins &H) {
    std::vector<double> part(H.parts, NAN);
    for (const RowBlock &b : H.blocks)
        if (b.nparts > 1) {
            const size_t k = (size_t)(b.slot + b.part);
            CHECK(k < part.size() && std::isnan(part[k]));
            part[k] = b.r0;
        }
    size_t used = 0;
    for (const SplitRow &r : H.splits)
        for (int k = 0; k < r.nparts; ++k, ++used) CHECK(part[r.first + k] == r.row);
    CHECK(used == part.size());
}

}  // namespace

int main() {
    std::mt19937_64 g(1);
    struct Case {
        int64_t m, n;
        double avg;
        int kind;
    };
    for (Case c : {Case{1, 1, 1, 0}, Case{5, 3, 0, 0}, Case{3000, 40000, 7, 0},
                   Case{40000, 3000, 3, 0}, Case{200, 100000, 300, 1},
                   Case{100000, 50000, 2, 2}, Case{1, 50000, 40000, 0}, Case{2, 700000, 600, 0},
                   Case{30000, kBktCols, 9, 1}, Case{30000, kBktCols + 1, 0.3, 0},
                   Case{20000, 70001, 3, 3}, Case{300000, 400000, 12, 0},
                   Case{2000, 300 * kBktCols, 100, 0}}) {
        const Csr A = make(c.m, c.n, c.avg, c.kind, g);
        const int64_t nnz = (int64_t)A.ci.size();
        std::vector<double> x(c.n), v(nnz), ref(c.m);
        for (auto &t : x) t = (double)(int64_t)(g() % 2001) - 1000;
        for (auto &t : v) t = (double)(int64_t)(g() % 201) - 100;
        for (int64_t i = 0; i < c.m; ++i)
            for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) ref[i] += v[p] * x[A.ci[p]];
        check_blocks(build_row_blocks(c.m, A.rp.data(), kTile64 - 3, 4096, 1000));
        {
            const HostBuckets B = build_push(c.m, c.n, A.rp.data(), A.ci.data(), true);
            std::vector<double> prod(4 * B.quads, NAN), y(c.m, NAN);
            std::vector<char> written(B.quads, 0), seen(nnz, 0);
            int64_t covered = 0;
            CHECK(B.width > 0 && B.width <= kBktCols && (B.width % 4 == 0 || B.width == kBktCols));
            for (const PushItem &it : B.items) {
                if (it.q0 == it.q1) continue;
                CHECK(it.q0 >= 0 && it.q0 < it.q1 && it.q1 <= B.quads);
                const int64_t c0 = (int64_t)it.cb * B.width;
                CHECK(it.cb >= 0 && c0 < c.n);
                for (int64_t q = it.q0; q < it.q1; ++q, ++covered) {
                    CHECK(B.dest[q] >= 0 && B.dest[q] < B.quads && !written[B.dest[q]]);
                    written[B.dest[q]] = 1;
                    for (int i = 0; i < 4; ++i) {
                        const int64_t e = 4 * q + i, p = B.src[e];
                        CHECK(B.col[e] < B.width && p < nnz);
                        if (p >= 0) {
                            CHECK(!seen[p] && A.ci[p] == c0 + B.col[e]);
                            seen[p] = 1;
                        } else {
                            CHECK(B.col[e] == 0);
                        }
                        prod[4 * (int64_t)B.dest[q] + i] = (p < 0 ? 0.0 : v[p]) * x[c0 + B.col[e]];
                    }
                }
            }
            CHECK(covered == B.quads);
            CHECK(std::count(seen.begin(), seen.end(), 1) == nnz);
            std::vector<double> part(B.parts, NAN);
            for (const Bucket &b : B.buckets) {
                std::vector<double> s(kBktCap + 1, NAN);
                CHECK(b.r0 >= 0 && b.r0 < b.r1 && b.r1 <= c.m && b.p1 - b.p0 <= kBktCap);
                CHECK(b.q0 >= 0 && b.q0 <= b.q1 && b.q1 <= B.quads);
                for (int64_t e = 4 * (int64_t)b.q0; e < 4 * (int64_t)b.q1; ++e) {
                    CHECK(B.pos[e] <= kBktCap);
                    s[B.pos[e]] = prod[e];
                }
                sum_rows(b, s, A.rp, part, y);
            }
            finish(B.splits, part, y);
            CHECK(y == ref);
            std::printf("push m %ld n %ld nnz %ld kind %d quads %ld buckets %zu splits %zu fragmented %d\n",
                        (long)c.m, (long)c.n, (long)nnz, c.kind, (long)B.quads,
                        B.buckets.size(), B.splits.size(), (int)B.fragmented);
        }
        for (int P : {1, 2, 8}) {
            std::vector<int64_t> cut;
            for (int p = 0; p <= P; ++p) cut.push_back(c.n * p / P);
            const Panels S = build_panels(c.m, A.rp.data(), A.ci.data(), P, cut);
            check_blocks(build_panel_blocks(c.m, S.rp.data(), P, kTile64 - 3, 4096, 1000));
            const HostBuckets B = build_tiles(c.m, S.rp.data(), S.ci.data(), P, true);
            std::vector<double> part(B.parts, NAN), ys(P * c.m, NAN), y(c.m, 0.0);
            std::vector<char> seen(nnz, 0);
            CHECK((int64_t)B.word.size() == 4 * B.quads && B.src.empty() &&
                  64 * (int64_t)B.base.size() == B.quads && B.first.size() == B.base.size());
            // the values of every entry, padding too, come from a nonzero
            for (int64_t e = 0; e < 4 * B.quads; ++e) {
                const int64_t p = B.first[e / 256] + (B.word[e] & ((1 << kTilePos) - 1));
                CHECK(p >= 0 && p < nnz);
            }
            for (size_t w = 0; w < B.buckets.size(); ++w) {
                const Bucket &b = B.buckets[w];
                if (b.r0 == b.r1) continue;
                CHECK(b.r0 / c.m == (b.r1 - 1) / c.m && (int)(w % 8) % P == b.r0 / c.m);
                CHECK(b.p1 - b.p0 <= kTileCap && b.q0 >= 0 && b.q0 % 64 == 0 && b.q0 <= b.q1 && b.q1 <= B.quads);
                std::vector<double> s(kTileCap + 1, NAN);
                for (int64_t e = 4 * (int64_t)b.q0; e < 4 * (int64_t)b.q1; ++e) {
                    const int64_t pos = B.word[e] & ((1 << kTilePos) - 1), p = b.p0 + pos,
                                  col = B.base[e / 256] + (int64_t)((uint32_t)B.word[e] >> kTilePos);
                    CHECK(B.first[e / 256] == b.p0 && p < b.p1 && S.ci[p] == col);
                    seen[p] = 1;
                    s[pos] = v[S.src[p]] * x[col];
                }
                sum_rows(b, s, S.rp, part, ys);
            }
            CHECK(std::count(seen.begin(), seen.end(), 1) == nnz);
            finish(B.splits, part, ys);
            for (int64_t i = 0; i < c.m; ++i)
                for (int p = 0; p < P; ++p)
                    if (P == 1 || (S.mask[i] >> p & 1)) y[i] += ys[(int64_t)p * c.m + i];
            CHECK(y == ref);
            std::printf("tiles m %ld n %ld nnz %ld kind %d panels %d quads %ld buckets %zu splits %zu fragmented %d\n",
                        (long)c.m, (long)c.n, (long)nnz, c.kind, P, (long)B.quads,
                        B.buckets.size(), B.splits.size(), (int)B.fragmented);
        }
    }
    // the one-workgroup layout of small LPs, as its lanes walk it
    for (Case c : {Case{1, 1, 1, 0}, Case{5, 3, 0, 0}, Case{3, 8192, 300, 0}, Case{500, 1000, 10, 0},
                   Case{1024, 1025, 4, 0}, Case{1025, 700, 6, 1}, Case{4096, 8192, 12, 0},
                   Case{8192, 4096, 5, 3}}) {
        const Csr A = make(c.m, c.n, c.avg, c.kind, g);
        const int64_t nnz = (int64_t)A.ci.size();
        std::vector<double> x(c.n + 1), v(nnz), ref(c.m), y(c.m, NAN);
        for (int64_t j = 0; j < c.n; ++j) x[j] = (double)(int64_t)(g() % 2001) - 1000;
        for (auto &t : v) t = (double)(int64_t)(g() % 201) - 100;
        for (int64_t i = 0; i < c.m; ++i)
            for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) ref[i] += v[p] * x[A.ci[p]];
        const HostSmall S = build_small(c.m, c.n, A.rp.data(), A.ci.data());
        CHECK(S.off.size() == (size_t)S.K * kSmallWaves + 1 && S.row.size() == (size_t)S.K * kSmallThreads / S.G);
        CHECK(S.src.size() == 128 * (size_t)S.off.back() && S.col.size() == S.src.size());
        CHECK((S.G & (S.G - 1)) == 0 && (S.G == 1 || S.G * c.m <= kSmallThreads));
        std::vector<char> seen(nnz, 0);
        for (int k = 0; k < S.K; ++k)
            for (int tid = 0; tid < kSmallThreads; tid += S.G) {
                const int32_t r = S.row[((int64_t)k * kSmallThreads + tid) / S.G];
                double t = 0;
                for (int l = tid; l < tid + S.G; ++l) {
                    const int sl = k * kSmallWaves + l / 64;
                    for (int q = S.off[sl]; q < S.off[sl + 1]; ++q)
                        for (int u = 0; u < 2; ++u) {
                            const size_t e = ((size_t)q * 64 + l % 64) * 2 + u;
                            CHECK(S.col[e] <= c.n && S.src[e] < nnz);
                            if (S.src[e] >= 0) {
                                CHECK(r >= 0 && !seen[S.src[e]] && A.ci[S.src[e]] == S.col[e]);
                                seen[S.src[e]] = 1;
                                t += v[S.src[e]] * x[S.col[e]];
                            } else {
                                CHECK(S.col[e] == c.n);
                            }
                        }
                }
                if (r >= 0) {
                    CHECK(r < c.m && std::isnan(y[r]));
                    y[r] = t;
                }
            }
        CHECK(y == ref && std::count(seen.begin(), seen.end(), 1) == nnz);
        std::printf("small m %ld n %ld nnz %ld kind %d lanes %d slots %d entries %zu\n",
                    (long)c.m, (long)c.n, (long)nnz, c.kind, S.G, S.K, S.src.size());
    }
    // without memory the planners throw bad_alloc, from their threads too
    {
        const Csr A = make(30000, 50000, 25, 0, g);
        std::vector<int64_t> trp(A.n + 1, 0);
        for (int32_t j : A.ci) ++trp[j + 1];
        for (int64_t j = 0; j < A.n; ++j) trp[j + 1] += trp[j];
        const std::vector<double> v(A.ci.size(), 1.0);
        long thrown = 0;
        for (int kind = 0; kind < 4; ++kind)
            for (long k = 0;; ++k) {
                bool ok = true;
                left = k;
                try {
                    if (kind == 0) build_push(A.m, A.n, A.rp.data(), A.ci.data(), true);
                    if (kind == 1) build_tiles(A.m, A.rp.data(), A.ci.data(), 1, true);
                    if (kind >= 2)
                        relabel(A.m, A.n, A.rp[A.m], A.rp.data(), A.ci.data(), v.data(), trp.data(), 1, 1, 0, kind - 2);
                } catch (const std::bad_alloc &) {
                    ok = false;
                }
                left = LONG_MAX;
                if (ok) break;
                ++thrown;
            }
        std::printf("memory %ld\n", thrown);
    }
    std::printf("done\n");
    return 0;
}
