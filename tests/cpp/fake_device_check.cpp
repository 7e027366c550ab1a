// The library's host paths against a stand-in for the HIP runtime, on the CPU:
// device memory is host memory, kernels do nothing.  Every device allocation
// of a load, an FP32 configure and an unrolled pass fails in turn; whatever
// happens, the calls return an error code and nothing stays allocated.  A load
// that fits without the bucketed layouts never fails for want of theirs, and
// what a failed call left out the next one allocates.  And
// products with the loaded values launch nothing for layouts they don't use.
// Usage: fake_device_check LIBRARY.  Prints one line per case.
#include <dlfcn.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <random>
#include <vector>

#include "pdhg.h"

#define CHECK(c)                                                   \
    do {                                                           \
        if (!(c)) {                                                \
            std::printf("FAILED %s line %d\n", #c, __LINE__);      \
            std::exit(1);                                          \
        }                                                          \
    } while (0)

// ---------------------------------------------------------- the runtime

static std::mutex mu;
static std::map<void *, size_t> live;       // device allocations
static size_t used = 0, peak = 0, budget = SIZE_MAX;
static long calls = 0, fail_at = -1;        // fail the fail_at-th allocation
static long from = LONG_MAX;                // ... all from this one on

extern "C" {
int hipMalloc(void **p, size_t n) {
    std::lock_guard<std::mutex> lk(mu);
    *p = nullptr;
    const long k = calls++;
    if (k == fail_at || k >= from || n > budget || used > budget - n) return 2;
    *p = std::calloc(1, n);
    live[*p] = n;
    used += n;
    peak = std::max(peak, used);
    return 0;
}
int hipFree(void *p) {
    std::lock_guard<std::mutex> lk(mu);
    if (!p) return 0;
    auto it = live.find(p);
    CHECK(it != live.end());
    used -= it->second;
    live.erase(it);
    std::free(p);
    return 0;
}
static int copy(void *d, const void *s, size_t n) {
    std::memmove(d, s, n);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { return copy(d, s, n); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return copy(d, s, n); }
int hipMemset(void *d, int v, size_t n) { return std::memset(d, v, n), 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { return std::memset(d, v, n), 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::calloc(1, n), 0; }
int hipHostFree(void *p) { return std::free(p), 0; }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "error"; }
int hipGetSymbolAddress(void **p, const void *) {
    static char dummy[256];
    return *p = dummy, 0;
}
static long launches = 0;
int hipLaunchKernel(const void *, ...) { return ++launches, 0; }
int __hipPushCallConfiguration(...) { return 0; }
int __hipPopCallConfiguration(...) { return 0; }
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipRegisterFunction(...) {}
void __hipRegisterVar(...) {}
void __hipUnregisterFatBinary(void **) {}
static int make(void **p) { return *p = std::malloc(1), 0; }
int hipStreamCreate(void **s) { return make(s); }
int hipStreamCreateWithFlags(void **s, unsigned) { return make(s); }
int hipStreamDestroy(void *s) { return std::free(s), 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreate(void **e) { return make(e); }
int hipEventCreateWithFlags(void **e, unsigned) { return make(e); }
int hipEventDestroy(void *e) { return std::free(e), 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *t, void *, void *) { return *t = 0, 0; }
}

// ------------------------------------------------------------- the calls

#define LIB(f) decltype(&f) p_##f
LIB(pdhg_create);
LIB(pdhg_destroy);
LIB(pdhg_load);
LIB(pdhg_set_tuning);
LIB(pdhg_configure);
LIB(pdhg_params_default);
LIB(pdhg_unrolled_forward);
LIB(pdhg_unrolled_backward);
LIB(pdhg_tape_free);
LIB(pdhg_spmv);
LIB(pdhg_iterate);
#undef LIB

struct Lp {
    int64_t m, n;
    std::vector<int64_t> arp, atrp;
    std::vector<int32_t> aci, atci;
    std::vector<double> v, b, c;
};

// k distinct rows in each column, all values 1
static Lp make_lp(int64_t m, int64_t n, int k) {
    Lp L{m, n, std::vector<int64_t>(m + 1, 0), {0}, {}, {}, {}, std::vector<double>(m, 1.0), std::vector<double>(n, 1.0)};
    std::mt19937_64 g(7);
    for (int64_t j = 0; j < n; ++j) {
        std::vector<int32_t> r;
        while ((int)r.size() < k) {
            const int32_t i = (int32_t)(g() % m);
            if (std::find(r.begin(), r.end(), i) == r.end()) r.push_back(i);
        }
        std::sort(r.begin(), r.end());
        for (int32_t i : r) ++L.arp[i + 1];
        L.atci.insert(L.atci.end(), r.begin(), r.end());
        L.atrp.push_back((int64_t)L.atci.size());
    }
    for (int64_t i = 0; i < m; ++i) L.arp[i + 1] += L.arp[i];
    L.aci.resize(L.atci.size());
    L.v.assign(L.atci.size(), 1.0);
    std::vector<int64_t> at(L.arp.begin(), L.arp.end() - 1);
    for (int64_t j = 0; j < n; ++j)
        for (int64_t p = L.atrp[j]; p < L.atrp[j + 1]; ++p) L.aci[at[L.atci[p]]++] = (int32_t)j;
    return L;
}

typedef std::vector<std::pair<const char *, int64_t>> Tuning;

static int load(pdhg_ctx *c, const Lp &L) {
    return p_pdhg_load(c, L.m, L.n, (int64_t)L.v.size(), L.arp.data(), L.aci.data(), L.v.data(),
                       L.atrp.data(), L.atci.data(), L.v.data(), L.b.data(), L.c.data(), nullptr, PDHG_MEM_HOST);
}

// One user's program; codes of load, FP32 configure and the two passes (none
// where there is no context).
static std::vector<int> program(const Lp &L, const Tuning &tuning) {
    pdhg_ctx *c = nullptr;
    std::vector<int> rc;
    if (p_pdhg_create(0, nullptr, &c) != PDHG_OK) return {};
    for (auto &t : tuning) CHECK(p_pdhg_set_tuning(c, t.first, t.second) == PDHG_OK);
    rc.push_back(load(c, L));
    if (rc.back() == PDHG_OK) {
        pdhg_params p;
        p_pdhg_params_default(&p);
        p.precision = PDHG_FP32;
        rc.push_back(p_pdhg_configure(c, &p));
    }
    if (rc.back() == PDHG_OK) {
        pdhg_tape *tape = nullptr;
        std::vector<double> x(L.n), gb(L.m), gA(L.v.size());
        rc.push_back(p_pdhg_unrolled_forward(c, 5, 2, PDHG_FP32, 0.1, 0.1, nullptr, nullptr, x.data(), PDHG_MEM_HOST, &tape));
        CHECK((rc.back() == PDHG_OK) == (tape != nullptr));
        if (tape) {
            rc.push_back(p_pdhg_unrolled_backward(tape, x.data(), x.data(), gb.data(), gA.data(), PDHG_MEM_HOST));
            p_pdhg_tape_free(tape);
        }
    }
    p_pdhg_destroy(c);
    return rc;
}

int main(int argc, char **argv) {
    CHECK(argc == 2);
    void *so = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!so) std::printf("%s\n", dlerror());
    CHECK(so);
#define LIB(f) CHECK(p_##f = (decltype(&f))dlsym(so, #f))
    LIB(pdhg_create);
    LIB(pdhg_destroy);
    LIB(pdhg_load);
    LIB(pdhg_set_tuning);
    LIB(pdhg_configure);
    LIB(pdhg_params_default);
    LIB(pdhg_unrolled_forward);
    LIB(pdhg_unrolled_backward);
    LIB(pdhg_tape_free);
    LIB(pdhg_spmv);
    LIB(pdhg_iterate);
    struct Case {
        const char *name;
        int64_t m, n;
        int k;
        Tuning tuning;
    };
    const std::vector<Case> all = {
        {"one workgroup", 300, 700, 5, {}},
        {"FP32 tiles", 8000, 20000, 5, {}},
        {"FP32 tiles, planned late", 20000, 62000, 5, {}},
        {"tiles", 3000, 7000, 5, {{"layout_a", 1}, {"layout_at", 1}}},
        {"panelled tiles", 3000, 7000, 5, {{"layout_a", 1}, {"layout_at", 1}, {"panels_a", 4}, {"panels_at", 2}}},
        {"pushed", 3000, 7000, 5, {{"layout_a", 2}, {"layout_at", 2}}},
        {"panels", 3000, 7000, 5, {{"panels_a", 4}, {"panels_at", 2}}}};
    for (const Case &c : all) {
        const Lp L = make_lp(c.m, c.n, c.k);
        const bool asked = !c.tuning.empty();
        long tried = 0, failed = 0;
        for (fail_at = 0;; ++fail_at, ++tried) {
            calls = 0;
            const std::vector<int> rc = program(L, c.tuning);
            for (int r : rc) CHECK(r == PDHG_OK || r == PDHG_E_OOM);
            CHECK(live.empty() && used == 0);
            // one allocation that fails does not fail a load that chose its layouts
            CHECK(asked || rc.size() != 1);
            failed += rc.empty() || rc.back() != PDHG_OK;
            if (calls <= fail_at) {
                CHECK(rc.size() == 4 && rc.back() == PDHG_OK);
                break;
            }
        }
        std::printf("%s: %ld allocations, %ld failed a call\n", c.name, tried, failed);
    }
    // the memory that row blocks and checkpoints need is enough, whatever the
    // sizes choose, for a whole program
    fail_at = -1;
    for (const Case &c : {Case{"one workgroup", 300, 700, 5, {}}, Case{"FP32 tiles", 8000, 20000, 5, {}},
                          Case{"tiles", 90000, 200000, 4, {}}, Case{"pushed", 500000, 1100000, 2, {}}}) {
        const Lp L = make_lp(c.m, c.n, c.k);
        auto calls_of = [&](const Tuning &tuning) {
            pdhg_ctx *x = nullptr;
            CHECK(p_pdhg_create(0, nullptr, &x) == PDHG_OK);
            for (auto &t : tuning) CHECK(p_pdhg_set_tuning(x, t.first, t.second) == PDHG_OK);
            CHECK(load(x, L) == PDHG_OK);
            pdhg_params p;
            p_pdhg_params_default(&p);
            const double level = 1e-3;
            std::vector<double> in(L.n), gb(L.m), gA(L.v.size()), out(L.n);
            for (int prec : {PDHG_FP64, PDHG_FP32}) {
                p.precision = prec;
                p.levels = &level;
                p.n_levels = 1;
                CHECK(p_pdhg_configure(x, &p) == PDHG_OK);
                for (int K : {3, 40}) {
                    pdhg_tape *tape = nullptr;
                    CHECK(p_pdhg_unrolled_forward(x, K, 2, prec, 0.1, 0.1, nullptr, nullptr, in.data(), PDHG_MEM_HOST, &tape) == PDHG_OK);
                    CHECK(p_pdhg_unrolled_backward(tape, in.data(), out.data(), gb.data(), gA.data(), PDHG_MEM_HOST) == PDHG_OK);
                    p_pdhg_tape_free(tape);
                }
            }
            p.polish = 1;
            CHECK(p_pdhg_configure(x, &p) == PDHG_OK);
            CHECK(p_pdhg_spmv(x, 0, 1, PDHG_FP32, in.data(), out.data(), PDHG_MEM_HOST) == PDHG_OK);
            p_pdhg_destroy(x);
            CHECK(live.empty());
        };
        budget = SIZE_MAX;
        peak = 0;
        calls_of({{"layout_a", 0}, {"layout_at", 0}, {"small", 0}, {"tape_bytes", 0}});
        const size_t least = peak;
        peak = 0;
        calls_of({});
        const size_t most = peak;
        CHECK(most > least);
        for (size_t part = 0; part <= 8; ++part) {
            budget = least + (most - least) * part / 8;
            calls_of({});
        }
        budget = SIZE_MAX;
        std::printf("%s: %zu bytes, %zu as chosen\n", c.name, least, most);
    }
    // calls that ran out of memory leave nothing half done: no solve runs before
    // a configure has succeeded, and the next one finds or makes every array
    {
        const Lp L = make_lp(3000, 7000, 5);
        const double level = 1e-3;
        size_t full = 0;
        long tried = 0;
        for (long k = -1;; ++k, ++tried) {
            pdhg_ctx *x = nullptr;
            CHECK(p_pdhg_create(0, nullptr, &x) == PDHG_OK);
            for (const char *key : {"layout_a", "layout_at"}) CHECK(p_pdhg_set_tuning(x, key, 1) == PDHG_OK);
            CHECK(load(x, L) == PDHG_OK);
            pdhg_params p;
            p_pdhg_params_default(&p);
            CHECK(p_pdhg_configure(x, &p) == PDHG_OK);
            p.precision = PDHG_FP32;
            p.levels = &level;
            p.n_levels = 1;
            p.polish = 1;
            calls = 0;
            from = k < 0 ? LONG_MAX : k;
            const int rc = p_pdhg_configure(x, &p);
            const bool reached = calls > k;
            std::vector<double> in(L.n, 1.0), out(L.n);
            const int rs = p_pdhg_spmv(x, 1, 1, PDHG_FP32, in.data(), out.data(), PDHG_MEM_HOST);
            from = LONG_MAX;
            CHECK(rs == PDHG_OK || rs == PDHG_E_OOM);
            if (rc != PDHG_OK) {
                int status = 0;
                CHECK(rc == PDHG_E_OOM && p_pdhg_iterate(x, 1, &status) == PDHG_E_STATE);
            }
            CHECK(p_pdhg_configure(x, &p) == PDHG_OK);
            if (k < 0) full = used;
            CHECK(used == full);
            p_pdhg_destroy(x);
            CHECK(live.empty());
            if (k >= 0 && !reached) break;
        }
        std::printf("half a configure: %ld allocations\n", tried);
    }
    // products with the loaded values are as many launches in any layout
    {
        const Lp L = make_lp(3000, 7000, 5);
        std::vector<double> in(L.n, 1.0), out(L.n);
        long n[3];
        for (int layout = 0; layout < 3; ++layout) {
            pdhg_ctx *x = nullptr;
            CHECK(p_pdhg_create(0, nullptr, &x) == PDHG_OK);
            for (const char *key : {"layout_a", "layout_at"}) CHECK(p_pdhg_set_tuning(x, key, layout) == PDHG_OK);
            CHECK(load(x, L) == PDHG_OK);
            launches = 0;
            for (int which = 0; which < 2; ++which)
                for (int prec : {PDHG_FP64, PDHG_FP32})
                    CHECK(p_pdhg_spmv(x, which, 0, prec, in.data(), out.data(), PDHG_MEM_HOST) == PDHG_OK);
            n[layout] = launches;
            p_pdhg_destroy(x);
        }
        CHECK(n[0] > 0 && n[1] == n[0] && n[2] == n[0]);
        std::printf("loaded values: %ld launches\n", n[0]);
    }
    std::printf("done\n");
    return 0;
}
