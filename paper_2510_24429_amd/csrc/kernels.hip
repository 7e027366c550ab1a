// kernels.hip -- HIP kernels for gfx950 (CDNA4, wave64).
//
// All sparse products go through one row-block kernel: each workgroup takes
// a descriptor (a run of short rows, one long row, or one part of a split
// row) built on the host from the row lengths.  Multi-row blocks stream
// their nonzeros, fully coalesced, into LDS and sum each row with a group of
// lanes sized to the block's row count; single long rows are strided by the
// whole workgroup and reduced across its four waves.  The PDHG updates are
// epilogues of these products, so every iteration is two kernels.  No
// atomics: every sum has a fixed order for a given matrix, so repeated runs
// are bitwise identical.
#include <cmath>

#include <type_traits>

#include "control.h"
#include "internal.h"

namespace pdhg {

namespace {

constexpr int kFixThreads = 64;

// Loads of the streamed CSR arrays (indices and values, each read once per
// SpMV), plain or non-temporal.  Measured on MI355X: plain loads are faster
// while the gathered table fits comfortably in L2 (9.4M streamed pairs with
// one random gather each from a 1.6 MB table: 45.5 us plain, 54.6 us
// non-temporal; the power-law steps 7,120 -> 7,773 iterations/s), while
// non-temporal loads keep a 5 MB gather panel in L2 (multicommodity, FP32:
// 3,828 plain, 4,294 non-temporal).  Each matrix side picks one at load.
template <bool NT, typename T>
__device__ __forceinline__ T sload(const T *p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Four consecutive streamed entries starting at a multiple of 4, as 16-byte
// loads (index arrays and value arrays are padded to a multiple of 4).
template <bool NT>
__device__ __forceinline__ void ld4(const int32_t *p, int (&o)[4]) {
    const v4i v = sload<NT>((const v4i *)p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
template <bool NT>
__device__ __forceinline__ void ld4(const double *p, double (&o)[4]) {
    const v2d a = sload<NT>((const v2d *)p);
    const v2d b = sload<NT>((const v2d *)(p + 2));
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
}
template <bool NT>
__device__ __forceinline__ void ld4(const float *p, float (&o)[4]) {
    const v4f v = sload<NT>((const v4f *)p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}

// Sum over the 256 threads of a workgroup; every thread gets the result.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T *sred) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sred[w] = v;
    __syncthreads();
    return (sred[0] + sred[1]) + (sred[2] + sred[3]);
}

__device__ __forceinline__ double block_max(double v, double *sred) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sred[w] = v;
    __syncthreads();
    return fmax(fmax(sred[0], sred[1]), fmax(sred[2], sred[3]));
}

// ---------------------------------------------------------------- elements

// One nonzero's contribution v[p] * x[ci[p]].  fetch4() reads four streamed
// indices and values, apply() gathers x and multiplies; splitting the two
// lets a thread issue all of its index/value loads, then all of its gathers,
// before waiting on any of them.
// (The load kind is a template parameter: a runtime branch between the two
// kinds of otherwise identical loads was merged by the compiler into plain
// loads.)
template <typename MT, typename VT, typename Acc, bool NT>
struct SpmvElem {
    const int32_t *ci;
    const MT *v;
    const VT *x;
    // entries base..base+3 (base a multiple of 4)
    __device__ __forceinline__ void fetch4(int base, int (&j)[4],
                                           MT (&a)[4]) const {
        ld4<NT>(ci + base, j);
        ld4<NT>(v + base, a);
    }
    __device__ __forceinline__ Acc apply(int j, MT a) const {
        return (Acc)a * (Acc)x[j];
    }
};

// ---------------------------------------------------------------- epilogues

// An epilogue may split into pre(r), the loads of its own operands of row r,
// and fin(r, s, pre), the update with the row sum s; multi-row blocks then
// issue the loads at their start, ahead of the row sums (operator() is
// fin(r, s, pre(r))).  Epilogues without a Pre type run after the sums.
template <class Epi, class = void>
struct has_pre : std::false_type {};
template <class Epi>
struct has_pre<Epi, std::void_t<typename Epi::Pre>> : std::true_type {};
struct NoPre {};
template <class Epi, bool = has_pre<Epi>::value>
struct PreOf {
    using type = NoPre;
};
template <class Epi>
struct PreOf<Epi, true> {
    using type = typename Epi::Pre;
};

template <typename OutT, typename Acc>
struct StoreEpi {
    OutT *out;
    __device__ __forceinline__ bool begin() { return true; }
    __device__ __forceinline__ void operator()(int r, Acc s) const {
        out[r] = (OutT)s;
    }
};

// out = row sum / sqrt(*norm2), or the sum itself where that is not positive.
struct StoreNormedEpi {
    double *out;
    const double *norm2;
    double nrm;
    __device__ __forceinline__ bool begin() {
        nrm = sqrt(*norm2);
        if (!(nrm > 0.0)) nrm = 1.0;
        return true;
    }
    __device__ __forceinline__ void operator()(int r, double s) const { out[r] = s / nrm; }
};

// Panel pass: row r of the stacked panel matrix stores its partial sum; the
// wrapped epilogue's begin() still decides whether the pass runs at all.
template <class Epi, typename Acc>
struct PanelEpi {
    Epi e;
    Acc *q;
    __device__ __forceinline__ bool begin() { return e.begin(); }
    __device__ __forceinline__ void operator()(int r, Acc s) const { q[r] = s; }
};

// Fused primal step over a row j of A~^T:
//   x_j <- max(l_j, x_j - tau (c_j - g_j)),  xbar_j <- xbar_j + (x_j - xbar_j)/t
// (xin, the old x, may be x itself)
template <typename T, bool HAS_L, bool AVG>
struct PrimalEpi {
    T *x, *xbar;
    const T *xin, *c, *l;
    const State *st;
    int off;
    T tau;
    T t;
    __device__ __forceinline__ bool begin() {
        tau = (T)st->tau;
        t = (T)(double)(st->t_base + off + 1);
        return st->status == PDHG_RUNNING;
    }
    struct Pre {
        T x, c, l, xb;
    };
    __device__ __forceinline__ Pre pre(int j) const {
        return {xin[j], c[j], HAS_L ? l[j] : (T)0, AVG ? xbar[j] : (T)0};
    }
    __device__ __forceinline__ void fin(int j, T g, const Pre &p) const {
        const T v = p.x - tau * (p.c - g);
        const T xn = v < p.l ? p.l : v;
        x[j] = xn;
        if (AVG) xbar[j] = p.xb + (xn - p.xb) / t;
    }
    __device__ __forceinline__ void operator()(int j, T g) const { fin(j, g, pre(j)); }
};

// Fused extrapolated dual step over a row i of A~ (q = (A~ x_new)_i):
//   y_i <- y_i + sigma (b_i - (2 q - (A~ x_old)_i)),  (A~ x)_i <- q,  ybar
// (yin, the old y, may be y itself)
template <typename T, bool AVG>
struct DualEpi {
    T *y, *ybar, *ax;
    const T *yin, *b;
    const State *st;
    int off;
    T sigma;
    T t;
    __device__ __forceinline__ bool begin() {
        sigma = (T)st->sigma;
        t = (T)(double)(st->t_base + off + 1);
        return st->status == PDHG_RUNNING;
    }
    struct Pre {
        T y, b, a, yb;
    };
    __device__ __forceinline__ Pre pre(int i) const {
        return {yin[i], b[i], ax[i], AVG ? ybar[i] : (T)0};
    }
    __device__ __forceinline__ void fin(int i, T q, const Pre &p) const {
        const T yn = p.y + sigma * (p.b - ((q + q) - p.a));
        y[i] = yn;
        ax[i] = q;
        if (AVG) ybar[i] = p.yb + (yn - p.yb) / t;
    }
    __device__ __forceinline__ void operator()(int i, T q) const { fin(i, q, pre(i)); }
};

// Reflected Halpern step, primal part over a row j of A~^T:
//   x^_j = max(l_j, x_j - tau (c_j - g_j))   (kept for the dual part)
//   x_j <- lambda ((1 + rho) x^_j - rho x_j) + (1 - lambda) x0_j
// with lambda = t / (t + 1) for the t-th step since the anchor x0.
template <typename T, bool HAS_L>
struct PrimalHalpernEpi {
    T *x, *xh;
    const T *c, *l, *x0;
    const State *st;
    int off;
    T tau, lam, rho;
    __device__ __forceinline__ bool begin() {
        tau = (T)st->tau;
        const double t = (double)(st->t_base + off + 1);
        lam = (T)(t / (t + 1.0));
        rho = (T)st->reflect;
        return st->status == PDHG_RUNNING;
    }
    struct Pre {
        T x, c, l, x0;
    };
    __device__ __forceinline__ Pre pre(int j) const {
        return {x[j], c[j], HAS_L ? l[j] : (T)0, x0[j]};
    }
    __device__ __forceinline__ void fin(int j, T g, const Pre &p) const {
        const T v = p.x - tau * (p.c - g);
        const T xhv = v < p.l ? p.l : v;
        xh[j] = xhv;
        x[j] = lam * (((T)1 + rho) * xhv - rho * p.x) + ((T)1 - lam) * p.x0;
    }
    __device__ __forceinline__ void operator()(int j, T g) const { fin(j, g, pre(j)); }
};

// Reflected Halpern step, dual part over a row i of A~ (q = (A~ x^)_i):
//   y^_i = y_i + sigma (b_i - (2 q - (A~x)_i))
//   y_i  <- lambda ((1 + rho) y^_i - rho y_i) + (1 - lambda) y0_i
//   (A~x)_i <- lambda ((1 + rho) q - rho (A~x)_i) + (1 - lambda) (A~x0)_i
template <typename T>
struct DualHalpernEpi {
    T *y, *ax;
    const T *b, *y0, *ax0;
    const State *st;
    int off;
    T sigma, lam, rho;
    __device__ __forceinline__ bool begin() {
        sigma = (T)st->sigma;
        const double t = (double)(st->t_base + off + 1);
        lam = (T)(t / (t + 1.0));
        rho = (T)st->reflect;
        return st->status == PDHG_RUNNING;
    }
    struct Pre {
        T a, y, b, y0, a0;
    };
    __device__ __forceinline__ Pre pre(int i) const {
        return {ax[i], y[i], b[i], y0[i], ax0[i]};
    }
    __device__ __forceinline__ void fin(int i, T q, const Pre &p) const {
        const T yhv = p.y + sigma * (p.b - ((q + q) - p.a));
        y[i] = lam * (((T)1 + rho) * yhv - rho * p.y) + ((T)1 - lam) * p.y0;
        ax[i] = lam * (((T)1 + rho) * q - rho * p.a) + ((T)1 - lam) * p.a0;
    }
    __device__ __forceinline__ void operator()(int i, T q) const { fin(i, q, pre(i)); }
};

// Evaluation of T(z) in FP64 arithmetic (storage T): primal part over a row j
// of A~^T records A~^T y and x^ = max(l, x - tau (c - A~^T y)).
template <typename T, bool HAS_L>
struct PrimalEvalEpi {
    const T *x;
    const double *c, *l;
    T *xh;
    double *aty;
    const State *st;
    double tau;
    __device__ __forceinline__ bool begin() {
        tau = st->tau;
        return true;
    }
    __device__ __forceinline__ void operator()(int j, double g) const {
        aty[j] = g;
        const double v = (double)x[j] - tau * (c[j] - g);
        const double lj = HAS_L ? l[j] : 0.0;
        xh[j] = (T)(v < lj ? lj : v);
    }
};

// ... dual part over a row i of A~ (q = (A~ x^)_i) records A~ x^ and
// y^ = y + sigma (b - (2 q - A~x)).
template <typename T>
struct DualEvalEpi {
    const T *y;
    const double *axc, *b;
    T *yh;
    double *axh;
    const State *st;
    double sigma;
    __device__ __forceinline__ bool begin() {
        sigma = st->sigma;
        return true;
    }
    __device__ __forceinline__ void operator()(int i, double q) const {
        axh[i] = q;
        yh[i] = (T)((double)y[i] + sigma * (b[i] - ((q + q) - axc[i])));
    }
};

// The adjoint keeps, per row i and per column j, a line of 128 bytes with one
// pair for each of the last kAdjSteps<T> steps k: (tau y_k, sigma gy_{k+1}) and
// (gv_k, 2 x_{k+1} - x_k); dL/dA~ is updated from both lines once per line.
template <typename T>
constexpr int kAdjLine = 128 / (int)sizeof(T);
template <typename T>
__device__ __forceinline__ void adj_pair(T *lines, int r, int slot, T a, T b) {
    using V2 = T __attribute__((ext_vector_type(2)));
    *(V2 *)(lines + (int64_t)r * kAdjLine<T> + 2 * slot) = V2{a, b};
}

// Adjoint of the dual step, over a row j of A~^T (s = (A~^T gy_{k+1})_j):
//   gxbar = -sigma s;  g = gx_{k+1} + 2 gxbar;  gv = 1[x_{k+1} > l] g
//   gx_k = gv - gxbar;  gc -= tau gv
template <typename T, bool HAS_L>
struct AdjDualEpi {
    const T *gx_in, *x1, *x0, *l;
    T *gx_out, *gv, *gc, *lines;
    int slot;
    T tau, sigma;
    __device__ __forceinline__ bool begin() { return true; }
    struct Pre {
        T gx, x1, x0, l, gc;
    };
    __device__ __forceinline__ Pre pre(int j) const {
        return {gx_in[j], x1[j], x0[j], HAS_L ? l[j] : (T)0, gc[j]};
    }
    __device__ __forceinline__ void fin(int j, T s, const Pre &p) const {
        const T gxbar = -sigma * s;
        const T g = p.gx + (gxbar + gxbar);
        const T v = p.x1 > p.l ? g : (T)0;
        gv[j] = v;
        gx_out[j] = v - gxbar;
        gc[j] = p.gc - tau * v;
        adj_pair(lines, j, slot, v, (p.x1 + p.x1) - p.x0);
    }
    __device__ __forceinline__ void operator()(int j, T s) const { fin(j, s, pre(j)); }
};

// Adjoint of the primal step, over a row i of A~ (s = (A~ gv)_i):
//   gy_k = gy_{k+1} + tau s;  gb += sigma gy_{k+1}
template <typename T>
struct AdjPrimalEpi {
    const T *gy_in, *y0;
    T *gy_out, *gb, *lines;
    int slot;
    T tau, sigma;
    __device__ __forceinline__ bool begin() { return true; }
    struct Pre {
        T g, y0, gb;
    };
    __device__ __forceinline__ Pre pre(int i) const { return {gy_in[i], y0[i], gb[i]}; }
    __device__ __forceinline__ void fin(int i, T s, const Pre &p) const {
        gy_out[i] = p.g + tau * s;
        gb[i] = p.gb + sigma * p.g;
        adj_pair(lines, i, slot, tau * p.y0, sigma * p.g);
    }
    __device__ __forceinline__ void operator()(int i, T s) const { fin(i, s, pre(i)); }
};

// ---------------------------------------------------------------- kernels

template <typename Acc, int TILE, class Elem, class Epi>
__global__ __launch_bounds__(kWG) void k_rowblock(
    const RowBlock *__restrict__ blks, const int32_t *__restrict__ rp,
    Elem elem, Epi epi_in, Acc *__restrict__ part) {
    constexpr int U = TILE / kWG;     // nonzeros per thread in a full tile
    using MT = decltype(elem.v[0] + 0);
    __shared__ Acc s_prod[TILE];
    __shared__ Acc s_sum[kWG];
    __shared__ int s_rp[TILE + 1];
    __shared__ Acc s_red[4];
    Epi epi = epi_in;
    // the control state and the descriptor are loaded together, and a
    // multi-row block issues its streamed loads before it looks at the state:
    // one memory latency less in a chain of four, which is what a launch over
    // a small matrix costs
    const RowBlock b = blks[blockIdx.x];
    const bool live = epi.begin();
    if (b.r1 == b.r0) return;         // padding of an XCD queue
    const int tid = threadIdx.x;
    if (b.r1 - b.r0 == 1) {
        if (!live) return;
        // one row: the workgroup strides it in aligned groups of four
        // nonzeros per lane (16-byte index and value loads), two groups in
        // flight; entries outside [p0, p1) are masked and never gathered
        int p0 = b.p0, p1 = b.p1;
        if (b.nparts > 1) {
            const int chunk = (p1 - p0 + b.nparts - 1) / b.nparts;
            p0 = p0 + b.part * chunk;
            p1 = min(p1, p0 + chunk);
        }
        Acc s0 = (Acc)0, s1 = (Acc)0;
        int base = (p0 & ~3) + 4 * tid;
        for (; base + 4 * kWG < p1; base += 8 * kWG) {
            int j0[4], j1[4];
            MT a0[4], a1[4];
            elem.fetch4(base, j0, a0);
            elem.fetch4(base + 4 * kWG, j1, a1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = base + u;
                if (p >= p0) s0 += elem.apply(j0[u], a0[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = base + 4 * kWG + u;
                if (p < p1) s1 += elem.apply(j1[u], a1[u]);
            }
        }
        if (base < p1) {
            int j0[4];
            MT a0[4];
            elem.fetch4(base, j0, a0);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = base + u;
                if (p >= p0 && p < p1) s0 += elem.apply(j0[u], a0[u]);
            }
        }
        Acc s = block_sum(s0 + s1, s_red);
        if (tid == 0) {
            if (b.nparts > 1)
                part[b.slot + b.part] = s;
            else
                epi(b.r0, s);
        }
        return;
    }
    // several rows: stage their row pointers in LDS, stream their nonzeros
    // (contiguous, <= TILE - 3) into LDS in aligned groups of four per lane
    // (16-byte loads), index and value loads first, then the gathers
    const int R = b.r1 - b.r0;
    // the epilogue's own operands of this thread's row, loaded first
    typename PreOf<Epi>::type pre{};
    if constexpr (has_pre<Epi>::value)
        if (R <= kWG && tid < R) pre = epi.pre(b.r0 + tid);
    const int p0 = b.p0;
    const int nz = b.p1 - p0;
    for (int r = tid; r <= R; r += kWG) s_rp[r] = rp[b.r0 + r] - p0;
    {
        const int a0 = p0 & ~3;
        constexpr int G4 = U / 4;      // groups of four per lane
        int jj[G4][4];
        MT aa[G4][4];
#pragma unroll
        for (int g = 0; g < G4; ++g) {
            const int base = a0 + 4 * (tid + g * kWG);
            if (base < p0 + nz) elem.fetch4(base, jj[g], aa[g]);
        }
        if (!live) return;
#pragma unroll
        for (int g = 0; g < G4; ++g) {
            const int base = a0 + 4 * (tid + g * kWG);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = base + u - p0;
                if (q >= 0 && q < nz) s_prod[q] = elem.apply(jj[g][u], aa[g][u]);
            }
        }
    }
    __syncthreads();
    if (R <= kWG) {
        // a power-of-two group of lanes per row sums it from LDS
        int G = 64;
        while (G * R > kWG) G >>= 1;
        const int r = tid / G, lane = tid & (G - 1);
        Acc s = (Acc)0;
        if (r < R) {
            const int q1 = s_rp[r + 1];
            for (int q = s_rp[r] + lane; q < q1; q += G) s += s_prod[q];
        }
        for (int o = G >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (r < R && lane == 0) s_sum[r] = s;
        __syncthreads();
        // epilogue on consecutive rows by consecutive threads
        if (tid < R) {
            if constexpr (has_pre<Epi>::value)
                epi.fin(b.r0 + tid, s_sum[tid], pre);
            else
                epi(b.r0 + tid, s_sum[tid]);
        }
    } else {
        for (int r = tid; r < R; r += kWG) {
            const int q1 = s_rp[r + 1];
            Acc s = (Acc)0;
            for (int q = s_rp[r]; q < q1; ++q) s += s_prod[q];
            epi(b.r0 + r, s);
        }
    }
}

// Finish split rows: add the parts in order, then the epilogue.
template <typename Acc, class Epi>
__global__ __launch_bounds__(kFixThreads) void k_split_fix(
    const SplitRow *__restrict__ sp, int nsplit, const Acc *__restrict__ part,
    Epi epi_in) {
    Epi epi = epi_in;
    if (!epi.begin()) return;
    const int t = blockIdx.x * kFixThreads + threadIdx.x;
    if (t >= nsplit) return;
    Acc s = (Acc)0;
    const SplitRow r = sp[t];
    for (int q = 0; q < r.nparts; ++q) s += part[r.first + q];
    epi(r.row, s);
}

// Rows of a panelled matrix: the partial sums of row i (stacked rows
// p * rows + i) over the panels that hold entries of it (bits of mask[i];
// all panels when mask is null), added in panel order, then the epilogue.
// Partials of empty stacked rows are neither written nor read; skipping
// them drops only exact zeros.
template <typename Acc, class Epi>
__global__ __launch_bounds__(kWG) void k_panel_combine(
    const Acc *__restrict__ q, const uint8_t *__restrict__ mask, int P,
    int rows, Epi epi_in) {
    Epi epi = epi_in;
    if (!epi.begin()) return;
    for (int i = blockIdx.x * kWG + threadIdx.x; i < rows; i += gridDim.x * kWG) {
        const unsigned m = mask ? mask[i] : 0xffu;
        Acc s = (Acc)0;
        for (int p = 0; p < P; ++p)
            if (m & (1u << p)) s += q[(int64_t)p * rows + i];
        epi(i, s);
    }
}

// ----------------------------------------------------------------- buckets

// Streamed entries come in 16-byte units of values (2 FP64 or 4 FP32), one
// unit per lane, so that a wave's load or store covers whole lines in order;
// their indices and positions come in units of as many.  (Any: a unit that may
// start at any element.)
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
typedef unsigned short v4us __attribute__((ext_vector_type(4)));
template <typename T>
struct UnitOf;
template <>
struct UnitOf<double> {
    static constexpr int W = 2;
    using V = v2d;
    using Any = double __attribute__((ext_vector_type(2), aligned(8)));
    using H = v2us;
};
template <>
struct UnitOf<float> {
    static constexpr int W = 4;
    using V = v4f;
    using Any = float __attribute__((ext_vector_type(4), aligned(4)));
    using H = v4us;
};

// Push pass: each workgroup multiplies the quads of its item with their column
// block of x, which sits in LDS, into their buckets: 19 (FP64) or 11 (FP32)
// bytes a nonzero, at 4.9 to 5.8 TB/s with 117 MB of products, which fit the
// memory-side cache (15M nonzeros, 58 and 55 us), and 3.3 to 3.8 TB/s with 880
// MB, which do not (110M, 685 and 560 us).  x may start at any element: the
// iterates of an unrolled pass lie n or m elements apart.
template <typename MT, typename VT, typename Acc>
__global__ __launch_bounds__(kBktThreads) void k_bkt_push(
    const PushItem *__restrict__ items, const uint16_t *__restrict__ col,
    const MT *__restrict__ val, const int32_t *__restrict__ dest,
    const VT *__restrict__ x, int64_t cols, int width, Acc *__restrict__ prod) {
    __shared__ __align__(16) VT s_x[kBktCols];
    using Un = UnitOf<MT>;
    using X = UnitOf<VT>;
    using Out = Acc __attribute__((ext_vector_type(Un::W)));
    constexpr int U = 4, F = 4 / Un::W;       // F units per quad
    const int tid = threadIdx.x;
    struct Regs {
        typename Un::V a;
        typename Un::H j;
        int d;
    };
    auto fetch = [&](int64_t p, Regs &r) {
        r.a = __builtin_nontemporal_load((const typename Un::V *)val + p);
        r.j = __builtin_nontemporal_load((const typename Un::H *)col + p);
        r.d = __builtin_nontemporal_load(dest + p / F);
    };
    auto store = [&](int64_t p, const Regs &r) {
        Out o;
#pragma unroll
        for (int i = 0; i < Un::W; ++i) o[i] = (Acc)r.a[i] * (Acc)s_x[r.j[i]];
        *(Out *)(prod + 4 * (int64_t)r.d + Un::W * (p % F)) = o;
    };
    const PushItem it = items[blockIdx.x];
    if (it.q0 == it.q1) return;
    // whole rounds of U units per lane without a bound check, the next round's
    // loads issued ahead of this round's products; then the rest
    const int64_t end = (int64_t)F * it.q1;
    int64_t h = (int64_t)F * it.q0 + tid;
    const int rounds = (int)((end - (h - tid)) / (U * kBktThreads));
    Regs r[U];
    if (rounds > 0)
#pragma unroll
        for (int u = 0; u < U; ++u) fetch(h + u * kBktThreads, r[u]);
    const int64_t c0 = (int64_t)it.cb * width;
    const int nc = (int)(cols - c0 < width ? cols - c0 : width);
    for (int i = X::W * tid; i < nc; i += X::W * kBktThreads) {
        if (i + X::W <= nc) {
            *(typename X::V *)(s_x + i) = *(const typename X::Any *)(x + c0 + i);
        } else {
            for (int u = i; u < nc; ++u) s_x[u] = x[c0 + u];
        }
    }
    __syncthreads();
    for (int k = 1; k <= rounds; ++k, h += U * kBktThreads) {
        Regs n[U];
        if (k < rounds) {
#pragma unroll
            for (int u = 0; u < U; ++u) fetch(h + (U + u) * kBktThreads, n[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) store(h + u * kBktThreads, r[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = n[u];
    }
    for (; h < end; h += kBktThreads) {
        fetch(h, r[0]);
        store(h, r[0]);
    }
}

// Where a bucket's products come from: fetch() issues the streamed loads of
// one unit, mul() forms its products, place() has their CSR positions.
template <typename Acc>
struct PushedUnits {                  // written by the push pass
    static constexpr int W = UnitOf<Acc>::W, kCap = kBktCap;
    static constexpr int kWaves = sizeof(Acc) == 4 ? 8 : 4;   // per SIMD
    static constexpr int kDepth = kCap / W / kBktThreads;     // units per lane
    using H = typename UnitOf<Acc>::H;
    const Acc *prod;
    const uint16_t *pos;
    struct Regs {
        typename UnitOf<Acc>::V a;
        H j;
    };
    __device__ __forceinline__ void fetch(int64_t p, Regs &r) const {
        r.a = __builtin_nontemporal_load((const typename UnitOf<Acc>::V *)prod + p);
        r.j = __builtin_nontemporal_load((const H *)pos + p);
    }
    __device__ __forceinline__ Acc mul(const Regs &r, int i) const { return r.a[i]; }
    __device__ __forceinline__ int place(const Regs &r, int i) const { return r.j[i]; }
};
// Values times gathers of the vector.  Bound by streaming 12 (FP64) or 8 (FP32)
// bytes a nonzero and by the lines the gathers bring from L2 (0.5 a nonzero on
// 200,000 FP64 columns): 9M nonzeros in random columns take 46 us, in
// neighbouring ones 33; FP32 26 and 19.  Two FP32 tiles fit in a CU's LDS, and
// one's stream overlaps the other's gathers, if few registers hold loads
// ahead: power-law primal 38 us a step with one workgroup per CU, 36 with two
// and three units ahead, 31 with one.  In FP64 the depth makes no difference.
template <typename MT, typename VT, typename Acc>
struct GatheredUnits {
    static constexpr int W = 4, kCap = kTileCap;   // (a wave gathers 64 neighbours at a time)
    static constexpr int kWaves = sizeof(Acc) == 4 ? 8 : 4;
    static constexpr int kDepth = sizeof(Acc) == 4 ? 1 : 3;
    const int32_t *word, *base;
    const MT *val;
    const VT *x;
    struct Regs {
        MT a[4];
        int w[4], b;
    };
    __device__ __forceinline__ void fetch(int64_t p, Regs &r) const {
        ld4<false>(word + 4 * p, r.w);
        ld4<false>(val + 4 * p, r.a);
        // (a wave's units lie in one group)
        r.b = base[__builtin_amdgcn_readfirstlane((int)(p >> 6))];
    }
    __device__ __forceinline__ Acc mul(const Regs &r, int i) const {
        return (Acc)r.a[i] * (Acc)x[r.b + (int)((unsigned)r.w[i] >> kTilePos)];
    }
    __device__ __forceinline__ int place(const Regs &r, int i) const {
        return r.w[i] & ((1 << kTilePos) - 1);
    }
};

// Streamed loads of the units h, h + NT, ... (U of them; past the end the last
// one again, so that no branch separates them), and their products to their
// places in LDS.
template <int U, class Units>
struct UnitRegs {
    typename Units::Regs a[U];
};
template <int U, class Units>
__device__ __forceinline__ void bkt_fetch(const Units &units, int64_t h,
                                          int64_t end, UnitRegs<U, Units> &r) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = h + u * kBktThreads;
        units.fetch(p < end ? p : end - 1, r.a[u]);
    }
}
template <int U, class Units, typename Acc>
__device__ __forceinline__ void bkt_store(const Units &units,
                                          const UnitRegs<U, Units> &r,
                                          Acc *__restrict__ s_prod) {
    constexpr int W = Units::W;
    Acc o[U][W];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < W; ++i) o[u][i] = units.mul(r.a[u], i);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < W; ++i) s_prod[units.place(r.a[u], i)] = o[u][i];
}
// All units [h - tid, end) of a bucket, at most U per lane at a time and no
// more than there are.
template <int U, class Units, typename Acc>
__device__ __forceinline__ void bkt_fill(const Units &units,
                                         int64_t h, int64_t end,
                                         Acc *__restrict__ s_prod) {
    const int64_t tid = threadIdx.x;
    for (; end - (h - tid) > (U - 1) * kBktThreads; h += U * kBktThreads) {
        UnitRegs<U, Units> r;
        bkt_fetch(units, h, end, r);
        bkt_store(units, r, s_prod);
    }
    if constexpr (U > 1)
        if (h - tid < end) bkt_fill<U - 1>(units, h, end, s_prod);
}

// A lane's share of a row, s[p], s[p + G], .. below p1; from eight on in
// balanced sums of eight that are added in FP64.  (Row blocks give a row of
// thousands 256 lanes that multiply as they add, a bucket at most 64: added one
// by one, FP32 sums of 400 to 5,000 products had an rms error of 1.42e-7 of their
// size against 9.2e-8 in row blocks, and FP32 iterates of a power-law LP were 8%
// further from 64 bits; so it is 9.0e-8, at the same times.)
template <typename Acc>
__device__ __forceinline__ Acc lane_sum(const Acc *s, int p, int p1, int G) {
    double t = 0.0;
    for (; p + 7 * G < p1; p += 8 * G) {
        Acc a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = s[p + u * G];
        t += (double)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
    }
    Acc r = (Acc)0;
    for (; p < p1; p += G) r += s[p];
    return (Acc)(t + (double)r);
}

// Sum pass: a bucket's products go to their CSR positions in LDS, then a
// power-of-two group of lanes sums each row (one lane per row, several rows
// per lane, when there are more rows than lanes), then the epilogue.  LOOP: a
// workgroup takes every gridDim.x-th bucket and loads the next one while it
// sums this one.
template <typename Acc, bool LOOP, class Units, class Epi>
__global__ __launch_bounds__(kBktThreads, Units::kWaves) void k_bkt_sum(
    const Bucket *__restrict__ buckets, int nbuckets,
    const int32_t *__restrict__ rp, Units units, Acc *__restrict__ part, Epi epi_in) {
    constexpr int NT = kBktThreads;
    __shared__ Acc s_prod[Units::kCap + 1];
    __shared__ Acc s_sum[NT];
    constexpr int F = 4 / Units::W, KP = 3;
    constexpr int U = Units::kDepth;
    Epi epi = epi_in;
    int t = blockIdx.x;
    Bucket b = buckets[t];
    if (!epi.begin() || b.r0 == b.r1) return;
    const int tid = threadIdx.x;
    UnitRegs<LOOP ? U : 1, Units> regs;
    int64_t h = (int64_t)F * b.q0 + tid, end = (int64_t)F * b.q1;
    if (LOOP && b.q0 < b.q1) bkt_fetch(units, h, end, regs);
    for (;;) {
        const bool more = LOOP && t + (int)gridDim.x < nbuckets;
        t = more ? t + (int)gridDim.x : t;
        const Bucket nb = LOOP ? buckets[t] : b;
        const int R = b.r1 - b.r0, nz = b.p1 - b.p0;
        int rs[KP], re[KP], G = 64;
        if (R <= NT)
            while (G * R > NT) G >>= 1;
        else
            G = 1;
        const int r0 = tid / G, lane = tid & (G - 1);
        typename PreOf<Epi>::type pre[KP]{};
        if (R > 1) {
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const int r = r0 + k * NT;
                if (r < R) {
                    rs[k] = rp[b.r0 + r] - b.p0;
                    re[k] = rp[b.r0 + r + 1] - b.p0;
                }
                if constexpr (has_pre<Epi>::value)
                    if (tid + k * NT < R) pre[k] = epi.pre(b.r0 + tid + k * NT);
            }
        }
        if constexpr (LOOP) {
            if (b.q0 < b.q1) {
                bkt_store(units, regs, s_prod);
                // units beyond the registers (the padding of short runs)
                bkt_fill<1>(units, h + U * NT, end, s_prod);
            }
            h = (int64_t)F * nb.q0 + tid;
            end = (int64_t)F * nb.q1;
            if (more && nb.q0 < nb.q1) bkt_fetch(units, h, end, regs);
        } else {
            bkt_fill<U>(units, h, end, s_prod);
        }
        __syncthreads();
        if (R == 1) {
            Acc s = wave_sum(lane_sum(s_prod, tid, nz, NT));
            if ((tid & 63) == 0) s_sum[tid >> 6] = s;
            __syncthreads();
            if (tid == 0) {
                double t = s_sum[0];
                for (int w = 1; w < NT / 64; ++w) t += s_sum[w];
                s = (Acc)t;
                if (b.slot >= 0)
                    part[b.slot + b.part] = s;
                else
                    epi(b.r0, s);
            }
        } else if (R <= NT) {
            Acc s = (Acc)0;
            if (r0 < R) s = lane_sum(s_prod, rs[0] + lane, re[0], G);
            for (int o = G >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o);
            if (r0 < R && lane == 0) s_sum[r0] = s;
            __syncthreads();
            if (tid < R) {
                if constexpr (has_pre<Epi>::value)
                    epi.fin(b.r0 + tid, s_sum[tid], pre[0]);
                else
                    epi(b.r0 + tid, s_sum[tid]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const int r = tid + k * NT;
                if (r < R) {
                    const Acc s = lane_sum(s_prod, rs[k], re[k], 1);
                    if constexpr (has_pre<Epi>::value)
                        epi.fin(b.r0 + r, s, pre[k]);
                    else
                        epi(b.r0 + r, s);
                }
            }
            for (int r = tid + KP * NT; r < R; r += NT) {
                epi(b.r0 + r, lane_sum(s_prod, rp[b.r0 + r] - b.p0, rp[b.r0 + r + 1] - b.p0, 1));
            }
        }
        if (!more) break;
        b = nb;
        __syncthreads();
    }
}

template <typename Acc, class Units, class Epi>
void run_sum(const DevCsr &M, const Units &units, Epi e, hipStream_t s) {
    const DevBuckets &K = *M.bkt;
    Acc *part = (Acc *)K.part;
    // FP64 products fill a CU's LDS with one bucket: workgroups that stay and
    // load ahead (multicommodity iteration 247 -> 237 us).  Two buckets fit in
    // FP32, which overlap by themselves (139 us against 145).
    constexpr bool loop = std::is_same<Units, PushedUnits<double>>::value;
    constexpr int kCus = 256;
    if (K.nbuckets > 0)
        hipLaunchKernelGGL((k_bkt_sum<Acc, loop, Units, Epi>),
                           dim3(loop && K.nbuckets > kCus ? kCus : K.nbuckets),
                           dim3(kBktThreads), 0, s, K.buckets, K.nbuckets, M.rp,
                           units, part, e);
    if (K.nsplit > 0)
        hipLaunchKernelGGL((k_split_fix<Acc, Epi>),
                           dim3((K.nsplit + kFixThreads - 1) / kFixThreads),
                           dim3(kFixThreads), 0, s, K.split, K.nsplit, part,
                           e);
}

template <typename Acc, typename MT, typename VT, class Epi>
void run_buckets(const DevCsr &M, const MT *vals, const VT *in, Epi e,
                 hipStream_t s) {
    const DevBuckets &K = *M.bkt;
    if (K.word) {
        run_sum<Acc>(M, GatheredUnits<MT, VT, Acc>{K.word, K.base, vals, in}, e, s);
        return;
    }
    Acc *prod = (Acc *)K.prod;
    if (K.nitems > 0)
        hipLaunchKernelGGL((k_bkt_push<MT, VT, Acc>), dim3(K.nitems),
                           dim3(kBktThreads), 0, s, K.items, K.col, vals, K.dest,
                           in, M.cols, K.width, prod);
    run_sum<Acc>(M, PushedUnits<Acc>{prod, K.pos}, e, s);
}

template <typename Acc, int TILE, class Elem, class Epi>
void run_rowblock(const RowBlock *blk, int nblk, const SplitRow *split,
                  int nsplit, Acc *part, const int32_t *rp,
                  Elem elem, Epi epi, hipStream_t s) {
    if (nblk > 0)
        hipLaunchKernelGGL((k_rowblock<Acc, TILE, Elem, Epi>), dim3(nblk),
                           dim3(kWG), 0, s, blk, rp, elem, epi, part);
    if (nsplit > 0)
        hipLaunchKernelGGL((k_split_fix<Acc, Epi>),
                           dim3((nsplit + kFixThreads - 1) / kFixThreads),
                           dim3(kFixThreads), 0, s, split, nsplit, part,
                           epi);
}

int grid_for(int64_t k, int per = kWG, int cap = 8192) {
    int64_t g = (k + per - 1) / per;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// FP64 accumulation always uses the FP64 bins; FP32 accumulation the FP32
// bins (twice the nonzeros per tile for the same LDS bytes).
template <typename Acc, class Elem, class Epi>
void run_bins(const DevCsr &M, Elem e, Epi p, hipStream_t s) {
    if constexpr (std::is_same<Acc, double>::value)
        run_rowblock<double, kTile64>(M.blk64, M.nblk64, M.split64, M.nsplit64,
                                      M.part64, M.rp, e, p, s);
    else
        run_rowblock<float, kTile32>(M.blk32, M.nblk32, M.split32, M.nsplit32,
                                     M.part32, M.rp, e, p, s);
}

// out-row r of M x epilogue, with M's values `vals` (its scaled FP64 or FP32
// values, or others).  The scaled values of an M with buckets run through
// these, a panelled M's through the panel twin (XCD-dealt panel pass, in tiles
// or row blocks, then the combine with the epilogue); any other value array
// takes the plain bins, and without `buckets` every one does.
template <typename Acc, typename MT, typename VT, class Epi>
void rb_spmv(const DevCsr &M, const MT *vals, const VT *in, Epi e,
             hipStream_t s, bool buckets = true) {
    if (buckets && M.bkt) {
        if constexpr (std::is_same<MT, double>::value) {
            if (vals == M.v64 && M.bkt->f64) return run_buckets<Acc>(M, (const MT *)M.bkt->v64, in, e, s);
        } else {
            if (vals == M.v32) return run_buckets<Acc>(M, (const MT *)M.bkt->v32, in, e, s);
        }
    }
    const MT *tv = nullptr;
    if (M.pan) {
        if constexpr (std::is_same<MT, double>::value) {
            if (vals == M.v64) tv = M.pan->v64;
        } else {
            if (vals == M.v32) tv = M.pan->v32;
        }
    }
    if (!tv) {
        if (M.stream_nt)
            run_bins<Acc>(M, SpmvElem<MT, VT, Acc, true>{M.ci, vals, in}, e, s);
        else
            run_bins<Acc>(M, SpmvElem<MT, VT, Acc, false>{M.ci, vals, in}, e, s);
        return;
    }
    Acc *q;
    if constexpr (std::is_same<Acc, double>::value)
        q = M.q64;
    else
        q = M.q32;
    if (buckets && M.pan->bkt && (M.pan->bkt->f64 || std::is_same<MT, float>::value)) {
        const MT *kv;
        if constexpr (std::is_same<MT, double>::value)
            kv = M.pan->bkt->v64;
        else
            kv = M.pan->bkt->v32;
        run_buckets<Acc>(*M.pan, kv, in, PanelEpi<Epi, Acc>{e, q}, s);
    } else if (M.stream_nt)
        run_bins<Acc>(*M.pan, SpmvElem<MT, VT, Acc, true>{M.pan->ci, tv, in},
                      PanelEpi<Epi, Acc>{e, q}, s);
    else
        run_bins<Acc>(*M.pan, SpmvElem<MT, VT, Acc, false>{M.pan->ci, tv, in},
                      PanelEpi<Epi, Acc>{e, q}, s);
    hipLaunchKernelGGL((k_panel_combine<Acc, Epi>),
                       dim3(grid_for(M.rows, kWG, 4096)), dim3(kWG), 0, s, q,
                       M.pan_mask, M.P, (int)M.rows, e);
}

}  // namespace

// ======================================================================= SpMV

void spmv_f64(const DevCsr &M, const double *vals, const double *in,
              double *out, hipStream_t s) {
    rb_spmv<double>(M, vals, in, StoreEpi<double, double>{out}, s);
}

void spmv_f64_normed(const DevCsr &M, const double *in, const double *norm2,
                     double *out, hipStream_t s) {
    rb_spmv<double>(M, (const double *)M.v64, in, StoreNormedEpi{out, norm2, 1.0}, s);
}

void spmv_f64_in32(const DevCsr &M, const double *vals, const float *in,
                   double *out, hipStream_t s) {
    rb_spmv<double>(M, vals, in, StoreEpi<double, double>{out}, s);
}

void spmv_f32(const DevCsr &M, const float *in, float *out, hipStream_t s,
              bool buckets) {
    rb_spmv<float>(M, (const float *)M.v32, in, StoreEpi<float, float>{out}, s, buckets);
}

// ============================================================ PDHG iteration

template <typename T, class Epi>
static void rbT(const DevCsr &M, const T *in, Epi e, hipStream_t s) {
    if constexpr (sizeof(T) == 8)
        rb_spmv<double>(M, (const double *)M.v64, in, e, s);
    else
        rb_spmv<float>(M, (const float *)M.v32, in, e, s);
}

template <typename T>
void launch_primal(const DevCsr &At, const Iter<T> &v, bool has_l,
                   const State *st, int off, hipStream_t s) {
    if (has_l)
        rbT<T>(At, v.y, PrimalEpi<T, true, true>{v.x, v.xbar, v.x, v.cs, v.ls, st, off}, s);
    else
        rbT<T>(At, v.y, PrimalEpi<T, false, true>{v.x, v.xbar, v.x, v.cs, v.ls, st, off}, s);
}

template <typename T>
void launch_dual(const DevCsr &A, const Iter<T> &v, const State *st, int off,
                 hipStream_t s) {
    rbT<T>(A, v.x, DualEpi<T, true>{v.y, v.ybar, v.ax, v.y, v.bs, st, off}, s);
}

template <typename T>
void launch_primal_halpern(const DevCsr &At, const Iter<T> &v, bool has_l,
                           const State *st, int off, hipStream_t s) {
    if (has_l)
        rbT<T>(At, v.y, PrimalHalpernEpi<T, true>{v.x, v.xbar, v.cs, v.ls, v.xl, st, off}, s);
    else
        rbT<T>(At, v.y, PrimalHalpernEpi<T, false>{v.x, v.xbar, v.cs, v.ls, v.xl, st, off}, s);
}

template <typename T>
void launch_dual_halpern(const DevCsr &A, const Iter<T> &v, const State *st,
                         int off, hipStream_t s) {
    rbT<T>(A, (const T *)v.xbar, DualHalpernEpi<T>{v.y, v.ax, v.bs, v.yl, v.ax0, st, off}, s);
}

template <typename T>
void launch_eval_T(const DevCsr &A, const DevCsr &At, const Iter<T> &v,
                   bool has_l, const double *cs, const double *bs,
                   const double *ls, const State *st, double *aty,
                   double *axh, const double *axc, hipStream_t s) {
    const double *atv = At.v64, *av = A.v64;
    if (has_l)
        rb_spmv<double>(At, atv, (const T *)v.y,
                        PrimalEvalEpi<T, true>{v.x, cs, ls, v.xbar, aty, st}, s);
    else
        rb_spmv<double>(At, atv, (const T *)v.y,
                        PrimalEvalEpi<T, false>{v.x, cs, ls, v.xbar, aty, st}, s);
    rb_spmv<double>(A, av, (const T *)v.xbar,
                    DualEvalEpi<T>{v.y, axc, bs, v.ybar, axh, st}, s);
}

// ------------------------------------------------------------ small LPs

namespace {

template <typename T>
struct SmallSide {
    const int32_t *off, *row;
    const uint16_t *col;
    const T *val;
    int G, K, rows;
};

template <typename T>
struct SmallArgs {
    SmallSide<T> at, a;
    Iter<T> v;
    const State *st;
    int off, count;
    T *tx, *ty;
};

// NP consecutive pairs of steps of one slice.
template <typename T, int NP>
struct SmallPairs {
    T a[NP][2];
    v2us j[NP];
    // pairs t.. of a slice that ends at pair t1
    __device__ __forceinline__ void load(const SmallSide<T> &s, int t, int t1) {
        using V2 = T __attribute__((ext_vector_type(2)));
        // uniform bases and one lane offset: addresses take few registers
        const unsigned l = threadIdx.x & 63;
        const V2 *val = (const V2 *)s.val + (int64_t)t * 64;
        const v2us *col = (const v2us *)s.col + (int64_t)t * 64;
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (t + u < t1) {
                const V2 v = (val + u * 64)[l];
                a[u][0] = v.x;
                a[u][1] = v.y;
                j[u] = (col + u * 64)[l];
            }
    }
    __device__ __forceinline__ T dot(const T *s_x, int t, int t1, T acc) const {
        T x[NP][2];
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (t + u < t1) {
                x[u][0] = s_x[j[u].x];
                x[u][1] = s_x[j[u].y];
            }
#pragma unroll
        for (int u = 0; u < NP; ++u)
            if (t + u < t1) acc += a[u][0] * x[u][0] + a[u][1] * x[u][1];
        return acc;
    }
};

// Sum of this lane's row in the slice [t, t1), whose first pairs are given.
template <typename T, int NP>
__device__ __forceinline__ T small_row(const SmallSide<T> &s, const T *s_x,
                                       const SmallPairs<T, NP> &first, int t,
                                       int t1) {
    T acc = first.dot(s_x, t, t1, (T)0);
    for (t += NP; t < t1; t += 2) {
        SmallPairs<T, 2> p;
        p.load(s, t, t1);
        acc = p.dot(s_x, t, t1, acc);
    }
    for (int o = s.G >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    return acc;
}

// `count` iterations in one workgroup.  On an LP of a few thousand nonzeros an
// iteration of two launches is all latency; here the gathered vectors stay in
// LDS, a row's other operands and the first NP pairs of its nonzeros with its
// lane (the rest streams from L2), and one barrier ends each half.
template <typename T, int MODE, int KX, int KY, int NP>
__global__ __launch_bounds__(kSmallThreads) void k_small(SmallArgs<T> g) {
    constexpr int NT = kSmallThreads;
    __shared__ T s_x[KX * NT + 1];
    __shared__ T s_y[KY * NT + 1];
    if (g.st->status != PDHG_RUNNING) return;
    const T tau = (T)g.st->tau, sigma = (T)g.st->sigma, rho = (T)g.st->reflect;
    const long long t0 = g.st->t_base + g.off;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = g.at.rows, m = g.a.rows;
    // this lane's columns and rows (-1: none; one lane of a row's G keeps it)
    // and their operands (xa, ya: average or anchor), and the wave's slices
    T x[KX], xa[KX], c[KX], l[KX], y[KY], ya[KY], b[KY], ax[KY], ax0[KY];
    int jx[KX], iy[KY], ex[KX], fx[KX], ey[KY], fy[KY];
#pragma unroll
    for (int k = 0; k < KX; ++k) {
        x[k] = xa[k] = c[k] = l[k] = (T)0;
        jx[k] = -1;
        ex[k] = fx[k] = 0;
        if (k < g.at.K) {
            ex[k] = g.at.off[k * kSmallWaves + w];
            fx[k] = g.at.off[k * kSmallWaves + w + 1];
            if (tid % g.at.G == 0) jx[k] = g.at.row[(k * NT + tid) / g.at.G];
        }
        const int j = jx[k];
        if (j >= 0) {
            x[k] = g.v.x[j];
            c[k] = g.v.cs[j];
            if (g.v.ls) l[k] = g.v.ls[j];
            if (MODE == SMALL_AVG) xa[k] = g.v.xbar[j];
            if (MODE == SMALL_HALPERN) xa[k] = g.v.xl[j];
        }
    }
#pragma unroll
    for (int k = 0; k < KY; ++k) {
        y[k] = ya[k] = b[k] = ax[k] = ax0[k] = (T)0;
        iy[k] = -1;
        ey[k] = fy[k] = 0;
        if (k < g.a.K) {
            ey[k] = g.a.off[k * kSmallWaves + w];
            fy[k] = g.a.off[k * kSmallWaves + w + 1];
            if (tid % g.a.G == 0) iy[k] = g.a.row[(k * NT + tid) / g.a.G];
        }
        const int i = iy[k];
        if (i >= 0) {
            y[k] = g.v.y[i];
            b[k] = g.v.bs[i];
            ax[k] = g.v.ax[i];
            if (MODE == SMALL_AVG) ya[k] = g.v.ybar[i];
            if (MODE == SMALL_HALPERN) {
                ya[k] = g.v.yl[i];
                ax0[k] = g.v.ax0[i];
            }
            s_y[i] = y[k];
        }
    }
    if (tid == 0) s_x[n] = s_y[m] = (T)0;      // what padding gathers
    SmallPairs<T, NP> px[KX], py[KY];
#pragma unroll
    for (int k = 0; k < KX; ++k) px[k].load(g.at, ex[k], fx[k]);
#pragma unroll
    for (int k = 0; k < KY; ++k) py[k].load(g.a, ey[k], fy[k]);
    __syncthreads();
    for (int it = 0; it < g.count; ++it) {
        const double td = (double)(t0 + it + 1);
        const T t = (T)td, lam = (T)(td / (td + 1.0));
#pragma unroll
        for (int k = 0; k < KX; ++k) {
            if (k >= g.at.K) break;
            const T s = small_row(g.at, s_y, px[k], ex[k], fx[k]);
            const int j = jx[k];
            if (j >= 0) {
                const T v = x[k] - tau * (c[k] - s);
                const T xn = v < l[k] ? l[k] : v;
                s_x[j] = xn;
                if (MODE == SMALL_HALPERN) {
                    x[k] = lam * (((T)1 + rho) * xn - rho * x[k]) + ((T)1 - lam) * xa[k];
                } else {
                    x[k] = xn;
                    if (MODE == SMALL_AVG) xa[k] = xa[k] + (xn - xa[k]) / t;
                    if (MODE == SMALL_PLAIN && g.tx) g.tx[(int64_t)it * n + j] = xn;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KY; ++k) {
            if (k >= g.a.K) break;
            const T q = small_row(g.a, s_x, py[k], ey[k], fy[k]);
            const int i = iy[k];
            if (i >= 0) {
                const T yh = y[k] + sigma * (b[k] - ((q + q) - ax[k]));
                if (MODE == SMALL_HALPERN) {
                    y[k] = lam * (((T)1 + rho) * yh - rho * y[k]) + ((T)1 - lam) * ya[k];
                    ax[k] = lam * (((T)1 + rho) * q - rho * ax[k]) + ((T)1 - lam) * ax0[k];
                } else {
                    y[k] = yh;
                    ax[k] = q;
                    if (MODE == SMALL_AVG) ya[k] = ya[k] + (yh - ya[k]) / t;
                    if (MODE == SMALL_PLAIN && g.ty) g.ty[(int64_t)it * m + i] = yh;
                }
                s_y[i] = y[k];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < KX; ++k)
        if (jx[k] >= 0) {
            g.v.x[jx[k]] = x[k];
            if (MODE == SMALL_AVG) g.v.xbar[jx[k]] = xa[k];
            if (MODE == SMALL_HALPERN) g.v.xbar[jx[k]] = s_x[jx[k]];
        }
#pragma unroll
    for (int k = 0; k < KY; ++k)
        if (iy[k] >= 0) {
            g.v.y[iy[k]] = y[k];
            g.v.ax[iy[k]] = ax[k];
            if (MODE == SMALL_AVG) g.v.ybar[iy[k]] = ya[k];
        }
}

// The reverse of steps [k0, k1), last first, in one workgroup: as k_small, with
// gy and gv as the gathered vectors.  X and Y hold the iterates of all steps.
template <typename T>
struct SmallAdjArgs {
    SmallSide<T> at, a;
    AdjVecs<T> v;
    const T *X, *Y, *ls;
    int k0, k1, slot0;
    T tau, sigma;
};
template <typename T, int KX, int KY, int NP>
__global__ __launch_bounds__(kSmallThreads) void k_small_adj(SmallAdjArgs<T> g) {
    constexpr int NT = kSmallThreads;
    __shared__ T s_gv[KX * NT + 1];
    __shared__ T s_gy[KY * NT + 1];
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = g.at.rows, m = g.a.rows;
    T gx[KX], gc[KX], l[KX], x1[KX], gy[KY], gb[KY];
    int jx[KX], iy[KY], ex[KX], fx[KX], ey[KY], fy[KY];
#pragma unroll
    for (int k = 0; k < KX; ++k) {
        gx[k] = gc[k] = l[k] = x1[k] = (T)0;
        jx[k] = -1;
        ex[k] = fx[k] = 0;
        if (k < g.at.K) {
            ex[k] = g.at.off[k * kSmallWaves + w];
            fx[k] = g.at.off[k * kSmallWaves + w + 1];
            if (tid % g.at.G == 0) jx[k] = g.at.row[(k * NT + tid) / g.at.G];
        }
        const int j = jx[k];
        if (j >= 0) {
            gx[k] = g.v.gx[j];
            gc[k] = g.v.gc[j];
            if (g.ls) l[k] = g.ls[j];
            x1[k] = g.X[(int64_t)g.k1 * n + j];
        }
    }
#pragma unroll
    for (int k = 0; k < KY; ++k) {
        gy[k] = gb[k] = (T)0;
        iy[k] = -1;
        ey[k] = fy[k] = 0;
        if (k < g.a.K) {
            ey[k] = g.a.off[k * kSmallWaves + w];
            fy[k] = g.a.off[k * kSmallWaves + w + 1];
            if (tid % g.a.G == 0) iy[k] = g.a.row[(k * NT + tid) / g.a.G];
        }
        const int i = iy[k];
        if (i >= 0) {
            gy[k] = g.v.gy[i];
            gb[k] = g.v.gb[i];
            s_gy[i] = gy[k];
        }
    }
    if (tid == 0) s_gv[n] = s_gy[m] = (T)0;    // what padding gathers
    SmallPairs<T, NP> px[KX], py[KY];
#pragma unroll
    for (int k = 0; k < KX; ++k) px[k].load(g.at, ex[k], fx[k]);
#pragma unroll
    for (int k = 0; k < KY; ++k) py[k].load(g.a, ey[k], fy[k]);
    __syncthreads();
    for (int st = g.k1 - 1, slot = g.slot0; st >= g.k0; --st, --slot) {
        T x0[KX], y0[KY];
#pragma unroll
        for (int k = 0; k < KX; ++k) x0[k] = jx[k] >= 0 ? g.X[(int64_t)st * n + jx[k]] : (T)0;
#pragma unroll
        for (int k = 0; k < KY; ++k) y0[k] = iy[k] >= 0 ? g.Y[(int64_t)st * m + iy[k]] : (T)0;
#pragma unroll
        for (int k = 0; k < KX; ++k) {
            if (k >= g.at.K) break;
            const T s = small_row(g.at, s_gy, px[k], ex[k], fx[k]);
            if (jx[k] >= 0) {
                const T gxbar = -g.sigma * s;
                const T q = gx[k] + (gxbar + gxbar);
                const T v = x1[k] > l[k] ? q : (T)0;
                s_gv[jx[k]] = v;
                gx[k] = v - gxbar;
                gc[k] = gc[k] - g.tau * v;
                adj_pair(g.v.lj, jx[k], slot, v, (x1[k] + x1[k]) - x0[k]);
                x1[k] = x0[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KY; ++k) {
            if (k >= g.a.K) break;
            const T s = small_row(g.a, s_gv, py[k], ey[k], fy[k]);
            if (iy[k] >= 0) {
                gb[k] = gb[k] + g.sigma * gy[k];
                adj_pair(g.v.li, iy[k], slot, g.tau * y0[k], g.sigma * gy[k]);
                gy[k] = gy[k] + g.tau * s;
                s_gy[iy[k]] = gy[k];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < KX; ++k)
        if (jx[k] >= 0) {
            g.v.gx[jx[k]] = gx[k];
            g.v.gc[jx[k]] = gc[k];
        }
#pragma unroll
    for (int k = 0; k < KY; ++k)
        if (iy[k] >= 0) {
            g.v.gy[iy[k]] = gy[k];
            g.v.gb[iy[k]] = gb[k];
        }
}

template <typename T>
SmallSide<T> small_side(const DevCsr &M) {
    const DevSmall &S = *M.small;
    const T *v;
    if constexpr (sizeof(T) == 8)
        v = S.v64;
    else
        v = S.v32;
    return {S.off, S.row, S.col, v, S.G, S.K, (int)M.rows};
}

// fn(columns per lane, rows per lane, resident pairs per slice) as constants:
// as many pairs as the registers of a lane (128) hold beside its rows.
template <typename T, class Fn>
void small_sized(int kx, int ky, Fn fn) {
    using std::integral_constant;
    constexpr bool d = sizeof(T) == 8;
    if (kx <= 1 && ky <= 1)
        fn(integral_constant<int, 1>(), integral_constant<int, 1>(), integral_constant<int, d ? 4 : 6>());
    else if (kx <= 2 && ky <= 1)
        fn(integral_constant<int, 2>(), integral_constant<int, 1>(), integral_constant<int, d ? 2 : 4>());
    else
        fn(integral_constant<int, 4>(), integral_constant<int, 2>(), integral_constant<int, d ? 1 : 2>());
}

}  // namespace

template <typename T>
void launch_small(const DevCsr &A, const DevCsr &At, const Iter<T> &v,
                  bool has_l, int mode, const State *st, int off, int count,
                  T *tx, T *ty, hipStream_t s) {
    SmallArgs<T> g{small_side<T>(At), small_side<T>(A), v, st, off, count, tx, ty};
    if (!has_l) g.v.ls = nullptr;
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(kSmallThreads), 0, s, g);
    };
    auto sized = [&](auto kx, auto ky, auto np) {
        constexpr int KX = decltype(kx)::value, KY = decltype(ky)::value,
                      NP = decltype(np)::value;
        if (mode == SMALL_HALPERN)
            run(k_small<T, SMALL_HALPERN, KX, KY, NP>);
        else if (mode == SMALL_AVG)
            run(k_small<T, SMALL_AVG, KX, KY, NP>);
        else
            run(k_small<T, SMALL_PLAIN, KX, KY, NP>);
    };
    small_sized<T>(g.at.K, g.a.K, sized);
}

template <typename T>
void launch_small_adj(const DevCsr &A, const DevCsr &At, const AdjVecs<T> &v,
                      const T *X, const T *Y, bool has_l, int k0, int k1,
                      int slot0, double tau, double sigma, hipStream_t s) {
    const SmallAdjArgs<T> g{small_side<T>(At), small_side<T>(A), v, X, Y,
                            has_l ? v.ls : nullptr, k0, k1, slot0, (T)tau, (T)sigma};
    small_sized<T>(g.at.K, g.a.K, [&](auto kx, auto ky, auto np) {
        constexpr int KX = decltype(kx)::value, KY = decltype(ky)::value,
                      NP = decltype(np)::value;
        hipLaunchKernelGGL((k_small_adj<T, KX, KY, NP>), dim3(1),
                           dim3(kSmallThreads), 0, s, g);
    });
}
template void launch_small_adj<double>(const DevCsr &, const DevCsr &,
                                       const AdjVecs<double> &, const double *,
                                       const double *, bool, int, int, int,
                                       double, double, hipStream_t);
template void launch_small_adj<float>(const DevCsr &, const DevCsr &,
                                      const AdjVecs<float> &, const float *,
                                      const float *, bool, int, int, int,
                                      double, double, hipStream_t);
template void launch_small<double>(const DevCsr &, const DevCsr &,
                                   const Iter<double> &, bool, int,
                                   const State *, int, int, double *, double *,
                                   hipStream_t);
template void launch_small<float>(const DevCsr &, const DevCsr &,
                                  const Iter<float> &, bool, int, const State *,
                                  int, int, float *, float *, hipStream_t);

#define INST_HALPERN(T)                                                        \
    template void launch_primal_halpern<T>(const DevCsr &, const Iter<T> &,   \
                                           bool, const State *, int,          \
                                           hipStream_t);                      \
    template void launch_dual_halpern<T>(const DevCsr &, const Iter<T> &,     \
                                         const State *, int, hipStream_t);    \
    template void launch_eval_T<T>(const DevCsr &, const DevCsr &,            \
                                   const Iter<T> &, bool, const double *,     \
                                   const double *, const double *,            \
                                   const State *, double *, double *,         \
                                   const double *, hipStream_t);
INST_HALPERN(double)
INST_HALPERN(float)
#undef INST_HALPERN

template void launch_primal<double>(const DevCsr &, const Iter<double> &, bool,
                                   const State *, int, hipStream_t);
template void launch_primal<float>(const DevCsr &, const Iter<float> &, bool,
                                   const State *, int, hipStream_t);
template void launch_dual<double>(const DevCsr &, const Iter<double> &,
                                 const State *, int, hipStream_t);
template void launch_dual<float>(const DevCsr &, const Iter<float> &,
                                 const State *, int, hipStream_t);

// ============================================================ adjoint

// One plain step from (x0, y0) to (v.x, v.y), A~x in v.ax.
template <typename T>
void launch_plain_step(const DevCsr &A, const DevCsr &At, const Iter<T> &v,
                       const T *x0, const T *y0, bool has_l, const State *st,
                       hipStream_t s) {
    if (has_l)
        rbT<T>(At, y0, PrimalEpi<T, true, false>{v.x, nullptr, x0, v.cs, v.ls, st, 0}, s);
    else
        rbT<T>(At, y0, PrimalEpi<T, false, false>{v.x, nullptr, x0, v.cs, v.ls, st, 0}, s);
    rbT<T>(A, (const T *)v.x, DualEpi<T, false>{v.y, nullptr, v.ax, y0, v.bs, st, 0}, s);
}

// The reverse of one step k (slot: its place in the lines).
template <typename T>
void launch_adj_step(const DevCsr &A, const DevCsr &At, const AdjVecs<T> &v,
                     const T *x0, const T *x1, const T *y0, bool has_l,
                     int slot, double tau, double sigma, hipStream_t s) {
    if (has_l)
        rbT<T>(At, (const T *)v.gy,
               AdjDualEpi<T, true>{v.gx, x1, x0, v.ls, v.gx, v.gv, v.gc, v.lj, slot, (T)tau, (T)sigma}, s);
    else
        rbT<T>(At, (const T *)v.gy,
               AdjDualEpi<T, false>{v.gx, x1, x0, v.ls, v.gx, v.gv, v.gc, v.lj, slot, (T)tau, (T)sigma}, s);
    rbT<T>(A, (const T *)v.gv,
           AdjPrimalEpi<T>{v.gy, y0, v.gy, v.gb, v.li, slot, (T)tau, (T)sigma}, s);
}

// dA~_p += sum over the slots below cnt of tau y_k,i gv_j - sigma gy_{k+1},i
// (2 x_{k+1},j - x_k,j), p = (i, j).  Eight lanes read the two lines of a
// nonzero, 16 bytes each, so a random access brings a line that is used whole.
// (One update per step, with five 8-byte gathers a nonzero, took 15 us a step
// at 800k nonzeros.)
template <typename T>
__global__ __launch_bounds__(kWG) void k_adj_gA(
    const int32_t *__restrict__ rowidx, const int32_t *__restrict__ ci,
    int64_t nnz, const T *__restrict__ li, const T *__restrict__ lj, int cnt,
    T *__restrict__ gA) {
    using Un = UnitOf<T>;
    constexpr int U = 4, W = Un::W;
    const int sub = threadIdx.x & 7;
    const int64_t step = (int64_t)gridDim.x * (kWG / 8);
    for (int64_t p0 = (int64_t)blockIdx.x * (kWG / 8) + (threadIdx.x >> 3);
         p0 < nnz; p0 += U * step) {
        typename Un::V a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int64_t p = p0 + u * step;
            if (p >= nnz) p = p0;
            a[u] = *((const typename Un::V *)(li + (int64_t)rowidx[p] * kAdjLine<T>) + sub);
            b[u] = *((const typename Un::V *)(lj + (int64_t)ci[p] * kAdjLine<T>) + sub);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            T d = (T)0;
#pragma unroll
            for (int i = 0; i < W; i += 2)
                if (W / 2 * sub + i / 2 < cnt) d += a[u][i] * b[u][i] - a[u][i + 1] * b[u][i + 1];
            for (int o = 4; o > 0; o >>= 1) d += __shfl_xor(d, o);
            const int64_t p = p0 + u * step;
            if (sub == 0 && p < nnz) gA[p] += d;
        }
    }
}

template <typename T>
void launch_adj_gA(const DevCsr &A, const int32_t *rowidx, const AdjVecs<T> &v,
                   int cnt, T *gA, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_gA<T>, dim3(grid_for(A.nnz, 32 * 4, 16384)),
                       dim3(kWG), 0, s, rowidx, A.ci, A.nnz, (const T *)v.li,
                       (const T *)v.lj, cnt, gA);
}

#define INST_ADJ(T)                                                          \
    template void launch_plain_step<T>(const DevCsr &, const DevCsr &,      \
                                       const Iter<T> &, const T *,          \
                                       const T *, bool, const State *,      \
                                       hipStream_t);                        \
    template void launch_adj_step<T>(const DevCsr &, const DevCsr &,        \
                                     const AdjVecs<T> &, const T *,         \
                                     const T *, const T *, bool, int,       \
                                     double, double, hipStream_t);          \
    template void launch_adj_gA<T>(const DevCsr &, const int32_t *,         \
                                   const AdjVecs<T> &, int, T *, hipStream_t);
INST_ADJ(double)
INST_ADJ(float)
#undef INST_ADJ

// ============================================================ KKT evaluation

namespace {

template <typename T>
struct KktArgs {
    const T *x[2], *y[2], *xl, *yl;
    const double *ax[2], *aty[2];
    const double *bs, *cs, *ls, *dr, *dc;
    int64_t m, n;
};

// Two consecutive entries of a vector as one load (the vectors are whole
// allocations, so even entries are aligned); past the end the second is 0.
typedef float v2f __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ void ld_pair(const T *p, int64_t i, bool both,
                                        double (&o)[2]) {
    if (both) {
        if constexpr (sizeof(T) == 8) {
            const v2d v = *(const v2d *)(p + i);
            o[0] = v.x; o[1] = v.y;
        } else {
            const v2f v = *(const v2f *)(p + i);
            o[0] = (double)v.x; o[1] = (double)v.y;
        }
    } else {
        o[0] = (double)p[i];
        o[1] = 0.0;
    }
}

// Sums / maxima over the workgroup of NQ quantities of NC candidates, written
// to partial[(c * Q_NQ + ids[q]) * kRedBlocks + blk].  Each wave reduces its
// quantities by shuffles; one pass through LDS joins the four waves.
template <int NC, int NQ>
__device__ __forceinline__ void kkt_finish(const double (&acc)[NC][NQ],
                                           const int (&ids)[NQ], int blk,
                                           double *__restrict__ partial) {
    __shared__ double s_w[4][NC * NQ];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const bool mx = ids[q] == Q_RPMAX || ids[q] == Q_RDMAX;
            const double v = mx ? wave_max(acc[c][q]) : wave_sum(acc[c][q]);
            if (l == 0) s_w[w][c * NQ + q] = v;
        }
    __syncthreads();
    if (threadIdx.x < NC * NQ) {
        const int c = threadIdx.x / NQ, q = threadIdx.x % NQ;
        int id = 0;
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            if (i == q) id = ids[i];
        const double a = s_w[0][threadIdx.x], b = s_w[1][threadIdx.x],
                     d = s_w[2][threadIdx.x], e = s_w[3][threadIdx.x];
        partial[(c * Q_NQ + id) * kRedBlocks + blk] =
            (id == Q_RPMAX || id == Q_RDMAX) ? fmax(fmax(a, b), fmax(d, e))
                                             : (a + b) + (d + e);
    }
}

// Blocks [0, nbr) reduce over rows, [nbr, nbr + nbc) over columns, each of
// the quantities of its side.  Bound by streaming 7 vectors per side and
// candidate pair: two entries per lane and load, and enough blocks to keep
// every CU's loads in flight.  Reducing the quantities one block reduction
// after the other, over 512 blocks a side however small the LP, took 29 us on
// a 500 x 1000 LP and 252 us on the 1.35M x 4.95M one (1.4 TB/s).
template <typename T, int NC>
__global__ __launch_bounds__(kWG) void k_kkt(KktArgs<T> a, int nbr, int nbc,
                                            double *__restrict__ partial) {
    if ((int)blockIdx.x < nbr) {
        constexpr int ids[6] = {Q_RP2, Q_RPMAX, Q_SRP2, Q_BY, Q_DY2, Q_FY2};
        double acc[NC][6] = {};
        for (int64_t i = 2 * ((int64_t)blockIdx.x * kWG + threadIdx.x); i < a.m;
             i += 2 * (int64_t)nbr * kWG) {
            const bool both = i + 1 < a.m;
            double b[2], dr[2], yl[2], ax[NC][2], y[NC][2];
            ld_pair(a.bs, i, both, b);
            ld_pair(a.dr, i, both, dr);
            ld_pair(a.yl, i, both, yl);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                ld_pair(a.ax[c], i, both, ax[c]);
                ld_pair(a.y[c], i, both, y[c]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (u && !both) break;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const double rs = b[u] - ax[c][u];
                    const double ru = rs / dr[u];
                    acc[c][0] += ru * ru;
                    acc[c][1] = fmax(acc[c][1], fabs(ru));
                    acc[c][2] += rs * rs;
                    acc[c][3] += b[u] * y[c][u];
                    const double dy = y[c][u] - yl[u];
                    acc[c][4] += dy * dy;
                }
                if (NC > 1) {
                    const double f = y[NC - 1][u] - y[0][u];
                    acc[NC - 1][5] += f * f;
                }
            }
        }
        kkt_finish<NC, 6>(acc, ids, blockIdx.x, partial);
    } else {
        constexpr int ids[7] = {Q_RD2, Q_RDMAX, Q_SRD2, Q_CX, Q_LZ, Q_DX2, Q_FX2};
        const int blk = (int)blockIdx.x - nbr;
        double acc[NC][7] = {};
        for (int64_t j = 2 * ((int64_t)blk * kWG + threadIdx.x); j < a.n;
             j += 2 * (int64_t)nbc * kWG) {
            const bool both = j + 1 < a.n;
            double cj[2], dc[2], xl[2], lj[2] = {0.0, 0.0}, g[NC][2], x[NC][2];
            ld_pair(a.cs, j, both, cj);
            ld_pair(a.dc, j, both, dc);
            ld_pair(a.xl, j, both, xl);
            if (a.ls) ld_pair(a.ls, j, both, lj);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                ld_pair(a.aty[c], j, both, g[c]);
                ld_pair(a.x[c], j, both, x[c]);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (u && !both) break;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const double ds = cj[u] - g[c][u];
                    const double zs = ds > 0.0 ? ds : 0.0;
                    const double rds = zs - ds;
                    const double du = ds / dc[u];
                    const double zu = du > 0.0 ? du : 0.0;
                    const double rdu = zu - du;
                    acc[c][0] += rdu * rdu;
                    acc[c][1] = fmax(acc[c][1], fabs(rdu));
                    acc[c][2] += rds * rds;
                    acc[c][3] += cj[u] * x[c][u];
                    acc[c][4] += lj[u] * zs;
                    const double dx = x[c][u] - xl[u];
                    acc[c][5] += dx * dx;
                }
                if (NC > 1) {
                    const double f = x[NC - 1][u] - x[0][u];
                    acc[NC - 1][6] += f * f;
                }
            }
        }
        kkt_finish<NC, 7>(acc, ids, blk, partial);
    }
}

// One evaluation's decisions: a fixed-order finish of the partial sums in one
// workgroup (a wave per quantity), then control_decide (control.h) on thread
// 0.  The control state is decided on in LDS and written back at the end:
// latency of dependent accesses is all that this kernel costs.  With a tree of
// barriers per quantity and the state in global memory it took 54-59 us per
// evaluation.
constexpr int kCtlThreads = 1024;
__global__ __launch_bounds__(kCtlThreads) void k_control(
    State *st, const double *__restrict__ partial, int nbr, int nbc, int ncand,
    int batch, int initial, double *elog) {
    __shared__ double tot[2][Q_NQ];
    __shared__ State s;
    static_assert(sizeof(State) % sizeof(uint32_t) == 0, "copied by words");
    constexpr int kWords = sizeof(State) / sizeof(uint32_t);
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    for (int i = tid; i < kWords; i += kCtlThreads)
        ((uint32_t *)&s)[i] = ((const uint32_t *)st)[i];
    for (int p = w; p < ncand * Q_NQ; p += kCtlThreads / 64) {
        const int q = p % Q_NQ;
        const bool mx = q == Q_RPMAX || q == Q_RDMAX;
        const int nb = (q <= Q_DY2 || q == Q_FY2) ? nbr : nbc;
        double v = 0.0;
#pragma unroll 4
        for (int b = l; b < nb; b += 64) {
            const double t = partial[p * kRedBlocks + b];
            v = mx ? fmax(v, t) : v + t;
        }
        v = mx ? wave_max(v) : wave_sum(v);
        if (l == 0) tot[p / Q_NQ][q] = v;
    }
    __syncthreads();
    if (tid == 0) {
        if (s.status == PDHG_RUNNING) {
            control_decide(&s, tot, ncand, batch, initial, elog);
        } else {
            s.copy_pending = 0;
            s.snap_n = 0;
        }
    }
    __syncthreads();
    for (int i = tid; i < kWords; i += kCtlThreads)
        ((uint32_t *)st)[i] = ((const uint32_t *)&s)[i];
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_polish_stash(
    const State *st, const T *x0, const T *y0, const T *x1, const T *y1,
    const double *dr, const double *dc, double *xs, double *ys, int64_t m,
    int64_t n) {
    if (!st->polish_due) return;
    const T *x = st->polish_cand ? x1 : x0;
    const T *y = st->polish_cand ? y1 : y0;
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride)
        xs[j] = dc[j] * (double)x[j];
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
        ys[i] = dr[i] * (double)y[i];
}

__global__ void k_advance(State *st, int batch) {
    if (threadIdx.x == 0 && st->status == PDHG_RUNNING) {
        st->k += batch;
        st->t_base += batch;
        st->copy_pending = 0;
        st->snap_n = 0;
    }
}

__global__ void k_set_status(State *st, int status) {
    if (threadIdx.x == 0 && st->status == PDHG_RUNNING) {
        st->status = status;
        st->copy_pending = 0;
        st->snap_n = 0;
    }
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_restart_apply(
    const State *__restrict__ st, T *x, T *y, T *ax, T *xbar, T *ybar,
    const double *ax_avg, T *xl, T *yl, T *ax0, int64_t m, int64_t n) {
    if (!st->copy_pending) return;
    const bool avg = st->copy_avg != 0, last = st->set_last != 0;
    const int64_t stride = (int64_t)gridDim.x * kWG;
    // a restart also starts the averages afresh (from zero, so that the first
    // average after it is exactly the first iterate)
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        const T v = avg ? xbar[j] : x[j];
        if (avg) x[j] = v;
        if (last) {
            xl[j] = v;
            xbar[j] = (T)0;
        }
    }
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride) {
        const T v = avg ? ybar[i] : y[i];
        if (avg) {
            y[i] = v;
            ax[i] = (T)ax_avg[i];
        }
        if (last) {
            yl[i] = v;
            ybar[i] = (T)0;
            if (ax0) ax0[i] = avg ? (T)ax_avg[i] : ax[i];
        }
    }
}

// Unscaled snapshot of candidate snap_cand into slot snap_first:
// x = D_c x~, y = D_r y~, z = max(0, (c~ - A~^T y~) / D_c).
template <typename T>
__global__ __launch_bounds__(kWG) void k_snapshot_pack(
    const State *__restrict__ st, const T *x0, const T *y0, const T *x1,
    const T *y1, const double *aty0, const double *aty1, const double *cs,
    const double *dr, const double *dc, const int32_t *pr, const int32_t *pc,
    double *slots, int64_t m, int64_t n) {
    if (st->snap_n == 0) return;
    const int c = st->snap_cand;
    const T *x = c ? x1 : x0;
    const T *y = c ? y1 : y0;
    const double *aty = c ? aty1 : aty0;
    double *base = slots + (int64_t)st->snap_first * (2 * n + m);
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        const int64_t o = pc[j];
        base[o] = dc[j] * (double)x[j];
        const double d = (cs[j] - aty[j]) / dc[j];
        base[n + m + o] = d > 0.0 ? d : 0.0;
    }
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
        base[n + pr[i]] = dr[i] * (double)y[i];
}

}  // namespace

void launch_kkt_reduce(int ncand, const void *x0, const void *y0,
                       const void *x1, const void *y1, bool f32,
                       const double *ax0, const double *aty0,
                       const double *ax1, const double *aty1, const void *xl,
                       const void *yl, const double *bs, const double *cs,
                       const double *ls, const double *dr, const double *dc,
                       int64_t m, int64_t n, double *partial, hipStream_t s) {
    const int nbr = red_blocks(m), nbc = red_blocks(n);
    auto run = [&](auto zero) {
        using T = decltype(zero);
        const KktArgs<T> a{{(const T *)x0, (const T *)x1},
                           {(const T *)y0, (const T *)y1},
                           (const T *)xl, (const T *)yl,
                           {ax0, ax1}, {aty0, aty1}, bs, cs, ls, dr, dc, m, n};
        if (ncand > 1)
            hipLaunchKernelGGL((k_kkt<T, 2>), dim3(nbr + nbc), dim3(kWG), 0, s,
                               a, nbr, nbc, partial);
        else
            hipLaunchKernelGGL((k_kkt<T, 1>), dim3(nbr + nbc), dim3(kWG), 0, s,
                               a, nbr, nbc, partial);
    };
    if (f32)
        run(0.0f);
    else
        run(0.0);
}

void launch_control(State *st, const double *partial, int64_t m, int64_t n,
                    int ncand, int batch, int initial, double *log,
                    hipStream_t s) {
    hipLaunchKernelGGL(k_control, dim3(1), dim3(kCtlThreads), 0, s, st, partial,
                       red_blocks(m), red_blocks(n), ncand, batch, initial, log);
}

void launch_polish_stash(const State *st, bool f32, const void *x0,
                         const void *y0, const void *x1, const void *y1,
                         const double *dr, const double *dc, double *xs,
                         double *ys, int64_t m, int64_t n, hipStream_t s) {
    const int g = grid_for(n > m ? n : m, kWG, 4096);
    if (f32)
        hipLaunchKernelGGL(k_polish_stash<float>, dim3(g), dim3(kWG), 0, s, st,
                           (const float *)x0, (const float *)y0, (const float *)x1,
                           (const float *)y1, dr, dc, xs, ys, m, n);
    else
        hipLaunchKernelGGL(k_polish_stash<double>, dim3(g), dim3(kWG), 0, s, st,
                           (const double *)x0, (const double *)y0,
                           (const double *)x1, (const double *)y1, dr, dc, xs,
                           ys, m, n);
}

void launch_advance(State *st, int batch, hipStream_t s) {
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, st, batch);
}

void launch_set_status(State *st, int status, hipStream_t s) {
    hipLaunchKernelGGL(k_set_status, dim3(1), dim3(64), 0, s, st, status);
}

void launch_restart_apply(State *st, bool f32, void *x, void *y, void *ax,
                          void *xbar, void *ybar, const double *ax_avg,
                          void *xl, void *yl, void *ax0, int64_t m, int64_t n,
                          hipStream_t s) {
    const int g = grid_for(n > m ? n : m, kWG, 4096);
    if (f32)
        hipLaunchKernelGGL(k_restart_apply<float>, dim3(g), dim3(kWG), 0, s,
                           st, (float *)x, (float *)y, (float *)ax,
                           (float *)xbar, (float *)ybar, ax_avg,
                           (float *)xl, (float *)yl, (float *)ax0, m, n);
    else
        hipLaunchKernelGGL(k_restart_apply<double>, dim3(g), dim3(kWG), 0, s,
                           st, (double *)x, (double *)y, (double *)ax,
                           (double *)xbar, (double *)ybar, ax_avg,
                           (double *)xl, (double *)yl, (double *)ax0, m, n);
}

void launch_snapshot_pack(const State *st, bool f32, const void *x0,
                          const void *y0, const void *x1, const void *y1,
                          const double *aty0, const double *aty1,
                          const double *cs, const double *dr, const double *dc,
                          const int32_t *pr, const int32_t *pc, double *slots,
                          int64_t m, int64_t n, hipStream_t s) {
    const int g = grid_for(n > m ? n : m, kWG, 4096);
    if (f32)
        hipLaunchKernelGGL(k_snapshot_pack<float>, dim3(g), dim3(kWG), 0, s,
                           st, (const float *)x0, (const float *)y0,
                           (const float *)x1, (const float *)y1, aty0, aty1,
                           cs, dr, dc, pr, pc, slots, m, n);
    else
        hipLaunchKernelGGL(k_snapshot_pack<double>, dim3(g), dim3(kWG), 0, s,
                           st, (const double *)x0, (const double *)y0,
                           (const double *)x1, (const double *)y1, aty0, aty1,
                           cs, dr, dc, pr, pc, slots, m, n);
}

// ============================================================ Ruiz scaling

namespace {

// rho_r = max over row r of |(D_r,i a_ij) D_c,j|, over the row blocks: for the
// rows of A (TR false) the row's factor comes first, so values and gathered
// factors are staged and combined row by row; for the rows of A^T the
// gathered factor comes first and the row's can multiply the maximum
// (rounding is monotone).  Bound by the gathers, as the steps are.  (A group
// of lanes per row, sized to the mean length, left skewed rows to few lanes:
// 145 us a pass on the power-law columns, 4.7M nonzeros, and 3.2 ms on the
// coupled LP's 55M.)
template <bool TR>
__global__ __launch_bounds__(kWG) void k_ruiz_rowmax(
    const RowBlock *__restrict__ blks, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ ci, const double *__restrict__ v,
    const double *__restrict__ d_row, const double *__restrict__ d_col,
    double *__restrict__ rho, double *__restrict__ part) {
    constexpr int U = kTile64 / kWG;
    __shared__ double s_v[kTile64];
    __shared__ double s_d[TR ? 1 : kTile64];
    __shared__ double s_red[4];
    const RowBlock b = blks[blockIdx.x];
    const int tid = threadIdx.x, R = b.r1 - b.r0;
    if (R == 1) {
        int p0 = b.p0, p1 = b.p1;
        if (b.nparts > 1) {
            const int chunk = (p1 - p0 + b.nparts - 1) / b.nparts;
            p0 = p0 + b.part * chunk;
            p1 = min(p1, p0 + chunk);
        }
        const double dr = d_row[b.r0];
        double mx = 0.0;
#pragma unroll 4
        for (int p = p0 + tid; p < p1; p += kWG) {
            const double a = TR ? (d_col[ci[p]] * v[p]) * dr : (dr * v[p]) * d_col[ci[p]];
            mx = fmax(mx, fabs(a));
        }
        mx = wave_max(mx);
        if ((tid & 63) == 0) s_red[tid >> 6] = mx;
        __syncthreads();
        if (tid == 0) {
            mx = fmax(fmax(s_red[0], s_red[1]), fmax(s_red[2], s_red[3]));
            if (b.nparts > 1)
                part[b.slot + b.part] = mx;
            else
                rho[b.r0] = mx;
        }
        return;
    }
    const int nz = b.p1 - b.p0;
    {
        int j[U];
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = tid + u * kWG;
            if (q < nz) {
                j[u] = ci[b.p0 + q];
                a[u] = v[b.p0 + q];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = tid + u * kWG;
            if (q < nz) {
                if (TR) {
                    s_v[q] = d_col[j[u]] * a[u];
                } else {
                    s_v[q] = a[u];
                    s_d[q] = d_col[j[u]];
                }
            }
        }
    }
    int G = 64;
    while (G > 1 && G * R > kWG) G >>= 1;
    const int lane = tid & (G - 1);
    __syncthreads();
    for (int r0 = 0; r0 < R; r0 += kWG / G) {
        const int r = r0 + tid / G;
        double mx = 0.0;
        if (r < R) {
            const double dr = d_row[b.r0 + r];
            const int q1 = rp[b.r0 + r + 1] - b.p0;
            for (int q = rp[b.r0 + r] - b.p0 + lane; q < q1; q += G)
                mx = fmax(mx, TR ? fabs(s_v[q]) : fabs((dr * s_v[q]) * s_d[q]));
            if (TR) mx = fmax(0.0, mx * dr);
        }
        for (int o = G >> 1; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        if (r < R && lane == 0) rho[b.r0 + r] = mx;
    }
}

// Rows split over several workgroups: the maximum of their parts.
__global__ __launch_bounds__(kFixThreads) void k_split_max(
    const SplitRow *__restrict__ sp, int nsplit, const double *__restrict__ part,
    double *__restrict__ rho) {
    const int t = blockIdx.x * kFixThreads + threadIdx.x;
    if (t >= nsplit) return;
    double mx = 0.0;
    const SplitRow r = sp[t];
    for (int q = 0; q < r.nparts; ++q) mx = fmax(mx, part[r.first + q]);
    rho[r.row] = mx;
}

__global__ __launch_bounds__(kWG) void k_ruiz_update(double *d,
                                                     const double *rho,
                                                     int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG) {
        double r = rho[i];
        if (r == 0.0) r = 1.0;
        d[i] = d[i] / sqrt(r);
    }
}

// out[p] = (D_r,i v[p]) * D_c,j over the row blocks (out32: its FP32 copy); an
// entry's row comes from a search of the block's row pointers in LDS.
template <bool TR>
__global__ __launch_bounds__(kWG) void k_scale_values(
    const RowBlock *__restrict__ blks, const int32_t *__restrict__ rp,
    const int32_t *__restrict__ ci, const double *__restrict__ v,
    const double *__restrict__ d_row, const double *__restrict__ d_col,
    double *__restrict__ out, float *__restrict__ out32) {
    __shared__ int s_rp[kTile64 + 1];
    __shared__ double s_dr[kTile64];
    const RowBlock b = blks[blockIdx.x];
    const int tid = threadIdx.x, R = b.r1 - b.r0;
    int p0 = b.p0, p1 = b.p1;
    if (b.nparts > 1) {
        const int chunk = (p1 - p0 + b.nparts - 1) / b.nparts;
        p0 = p0 + b.part * chunk;
        p1 = min(p1, p0 + chunk);
    }
    for (int r = tid; r < R; r += kWG) {
        s_rp[r + 1] = rp[b.r0 + r + 1];
        s_dr[r] = d_row[b.r0 + r];
    }
    __syncthreads();
    for (int p = p0 + tid; p < p1; p += kWG) {
        // the first row that ends beyond p
        int lo = 0, hi = R - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_rp[mid + 1] > p) hi = mid; else lo = mid + 1;
        }
        const double dr = s_dr[lo], dc = d_col[ci[p]];
        const double a = TR ? (dc * v[p]) * dr : (dr * v[p]) * dc;
        out[p] = a;
        if (out32) out32[p] = (float)a;
    }
}

}  // namespace

void launch_ruiz_rowmax(const DevCsr &M, const double *d_row,
                        const double *d_col, int transposed, double *rho,
                        hipStream_t s) {
    if (M.nblk64 > 0) {
        auto run = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(M.nblk64), dim3(kWG), 0, s, M.blk64,
                               M.rp, M.ci, M.v_orig, d_row, d_col, rho,
                               M.part64);
        };
        if (transposed)
            run(k_ruiz_rowmax<true>);
        else
            run(k_ruiz_rowmax<false>);
    }
    if (M.nsplit64 > 0)
        hipLaunchKernelGGL(k_split_max,
                           dim3((M.nsplit64 + kFixThreads - 1) / kFixThreads),
                           dim3(kFixThreads), 0, s, M.split64, M.nsplit64,
                           M.part64, rho);
}

void launch_ruiz_update(double *d, const double *rho, int64_t k,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_ruiz_update, dim3(grid_for(k, kWG, 4096)), dim3(kWG),
                       0, s, d, rho, k);
}

void launch_scale_values(const DevCsr &M, const double *v, const double *d_row,
                         const double *d_col, int transposed, double *out,
                         float *out32, hipStream_t s) {
    if (M.nblk64 == 0) return;
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(M.nblk64), dim3(kWG), 0, s, M.blk64, M.rp,
                           M.ci, v, d_row, d_col, out, out32);
    };
    if (transposed)
        run(k_scale_values<true>);
    else
        run(k_scale_values<false>);
}

// ============================================================ vector kernels

namespace {

__global__ __launch_bounds__(kWG) void k_dot_partial(const double *a,
                                                     const double *b,
                                                     int64_t k,
                                                     double *partial) {
    __shared__ double s_red[4];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG)
        acc += a[i] * b[i];
    acc = block_sum(acc, s_red);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// mode 0: sum of partials; mode 1: max of partials
__global__ __launch_bounds__(kWG) void k_finish(const double *partial, int np,
                                                double *result, int mode) {
    __shared__ double s_red[4];
    double v = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < np; b += kWG) {
        const double p = partial[b];
        v = mode ? fmax(v, p) : v + p;
    }
    v = mode ? wave_max(v) : wave_sum(v);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        *result = mode ? fmax(fmax(s_red[0], s_red[1]), fmax(s_red[2], s_red[3]))
                       : (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_fill(T *p, T v, int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG)
        p[i] = v;
}

template <typename D, typename S>
__global__ __launch_bounds__(kWG) void k_convert(D *dst, const S *src,
                                                 int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG)
        dst[i] = (D)src[i];
}

// The start of a solve from the scaled pair (xs, ys): iterate and restart point
// take it, the averages start at zero.  One launch for what small LPs pay for
// as eight fills and four copies (about 70 us of a 3.6 ms solve).
template <typename T>
__global__ __launch_bounds__(kWG) void k_start(const double *__restrict__ xs,
                                               const double *__restrict__ ys,
                                               int64_t n, int64_t m, Iter<T> v) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n + m;
         i += (int64_t)gridDim.x * kWG) {
        if (i < n) {
            v.x[i] = v.xl[i] = (T)xs[i];
            v.xbar[i] = (T)0;
        } else {
            v.y[i - n] = v.yl[i - n] = (T)ys[i - n];
            v.ybar[i - n] = (T)0;
        }
    }
}

__global__ __launch_bounds__(kWG) void k_ew(double *out, const double *a,
                                            const double *b, int64_t k,
                                            int mode) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG) {
        if (mode == 0)
            out[i] = a[i] * b[i];
        else if (mode == 1)
            out[i] = a[i] / b[i];
        else
            out[i] = a[i] * b[0];
    }
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_unscale_xyz(
    const T *xs, const T *ys, const double *aty, const double *cs,
    const double *dr, const double *dc, const int32_t *pr, const int32_t *pc,
    double *x, double *y, double *z, int64_t m, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        const int64_t o = pc[j];
        if (x) x[o] = dc[j] * (double)xs[j];
        if (z) {
            const double d = (cs[j] - aty[j]) / dc[j];
            z[o] = d > 0.0 ? d : 0.0;
        }
    }
    if (y)
        for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
            y[pr[i]] = dr[i] * (double)ys[i];
}

__global__ __launch_bounds__(kWG) void k_gather(double *dst,
                                                const double *src,
                                                const int32_t *idx,
                                                int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG)
        dst[i] = src[idx[i]];
}

__global__ __launch_bounds__(kWG) void k_permute(double *dst,
                                                 const double *src,
                                                 const int32_t *perm,
                                                 int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG)
        dst[perm[i]] = src[i];
}

// Correction LP data in the scaled space: b^ = DP (b~ - A~x~),
// c^ = DD (c~ - A~^T y~), l^ = -DP x~.
__global__ __launch_bounds__(kWG) void k_refine_rhs(
    const double *bs, const double *ax, const double *cs, const double *aty,
    const double *xs, const double *ls, double DP, double DD, double *bh,
    double *ch, double *lh, int64_t m, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
        bh[i] = DP * (bs[i] - ax[i]);
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        ch[j] = DD * (cs[j] - aty[j]);
        lh[j] = DP * ((ls ? ls[j] : 0.0) - xs[j]);
    }
}

// Per block: max |r_P,i| and max (l_j - x_j)^+ (unscaled) into
// partial[0][b], max (-d_j)^+ into partial[1][b].
__global__ __launch_bounds__(kWG) void k_refine_delta(
    const double *bs, const double *ax, const double *cs, const double *aty,
    const double *xs, const double *ls, const double *dr, const double *dc,
    int64_t m, int64_t n, double *partial) {
    __shared__ double s_red[4];
    double dp = 0.0, dd = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
        dp = fmax(dp, fabs((bs[i] - ax[i]) / dr[i]));
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        dp = fmax(dp, dc[j] * ((ls ? ls[j] : 0.0) - xs[j]));
        dd = fmax(dd, -((cs[j] - aty[j]) / dc[j]));
    }
    dp = block_max(dp, s_red);
    dd = block_max(dd, s_red);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = dp;
        partial[gridDim.x + blockIdx.x] = dd;
    }
}

template <typename T>
__global__ __launch_bounds__(kWG) void k_refine_update(
    double *xs, double *ys, const T *xh, const T *yh, const double *ls,
    double invP, double invD, int64_t m, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t j = (int64_t)blockIdx.x * kWG + threadIdx.x; j < n; j += stride) {
        const double v = xs[j] + (double)xh[j] * invP;
        const double lj = ls ? ls[j] : 0.0;
        xs[j] = v < lj ? lj : v;
    }
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < m; i += stride)
        ys[i] = ys[i] + (double)yh[i] * invD;
}

__global__ __launch_bounds__(kWG) void k_norm_unscaled_partial(
    const double *vs, const double *d, int64_t k, double *partial) {
    __shared__ double s_red[4];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG) {
        const double u = vs[i] / d[i];
        acc += u * u;
    }
    acc = block_sum(acc, s_red);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

}  // namespace

void launch_dot(const double *a, const double *b, int64_t k, double *partial,
                double *result, hipStream_t s) {
    hipLaunchKernelGGL(k_dot_partial, dim3(red_blocks(k)), dim3(kWG), 0, s, a, b,
                       k, partial);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kWG), 0, s, partial,
                       red_blocks(k), result, 0);
}

void launch_norm_unscaled(const double *vs, const double *d, int64_t k,
                          double *partial, double *result, hipStream_t s) {
    hipLaunchKernelGGL(k_norm_unscaled_partial, dim3(red_blocks(k)), dim3(kWG),
                       0, s, vs, d, k, partial);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kWG), 0, s, partial,
                       red_blocks(k), result, 0);
}

void launch_fill(double *p, double v, int64_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_fill<double>, dim3(grid_for(k, kWG, 4096)),
                       dim3(kWG), 0, s, p, v, k);
}

void launch_fill32(float *p, float v, int64_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_fill<float>, dim3(grid_for(k, kWG, 4096)), dim3(kWG),
                       0, s, p, v, k);
}

template <typename T>
void launch_start(const double *xs, const double *ys, int64_t n, int64_t m,
                  const Iter<T> &v, hipStream_t s) {
    hipLaunchKernelGGL(k_start<T>, dim3(grid_for(n + m, kWG, 4096)), dim3(kWG),
                       0, s, xs, ys, n, m, v);
}
template void launch_start<double>(const double *, const double *, int64_t,
                                   int64_t, const Iter<double> &, hipStream_t);
template void launch_start<float>(const double *, const double *, int64_t,
                                  int64_t, const Iter<float> &, hipStream_t);

void launch_to_f32(float *dst, const double *src, int64_t k, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<float, double>), dim3(grid_for(k, kWG, 4096)),
                       dim3(kWG), 0, s, dst, src, k);
}

void launch_to_f64(double *dst, const float *src, int64_t k, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<double, float>), dim3(grid_for(k, kWG, 4096)),
                       dim3(kWG), 0, s, dst, src, k);
}

void launch_ew(double *out, const double *a, const double *b, int64_t k,
               int mode, hipStream_t s) {
    hipLaunchKernelGGL(k_ew, dim3(grid_for(k, kWG, 4096)), dim3(kWG), 0, s,
                       out, a, b, k, mode);
}

void launch_unscale_xyz(const double *xs, const double *ys, const double *aty,
                        const double *cs, const double *dr, const double *dc,
                        const int32_t *pr, const int32_t *pc, double *x,
                        double *y, double *z, int64_t m, int64_t n,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_unscale_xyz<double>,
                       dim3(grid_for(n > m ? n : m, kWG, 4096)), dim3(kWG), 0,
                       s, xs, ys, aty, cs, dr, dc, pr, pc, x, y, z, m, n);
}

void launch_unscale_xyz32(const float *xs, const float *ys, const double *aty,
                          const double *cs, const double *dr,
                          const double *dc, const int32_t *pr,
                          const int32_t *pc, double *x, double *y, double *z,
                          int64_t m, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_unscale_xyz<float>,
                       dim3(grid_for(n > m ? n : m, kWG, 4096)), dim3(kWG), 0,
                       s, xs, ys, aty, cs, dr, dc, pr, pc, x, y, z, m, n);
}

void launch_permute(double *dst, const double *src, const int32_t *perm,
                    int64_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_permute, dim3(grid_for(k, kWG, 16384)), dim3(kWG), 0,
                       s, dst, src, perm, k);
}

namespace {
__global__ __launch_bounds__(kWG) void k_gather_pad(
    double *__restrict__ dst, float *__restrict__ dst32,
    const double *__restrict__ src, const int32_t *__restrict__ idx, int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG) {
        const int p = idx[i];
        const double v = p < 0 ? 0.0 : src[p];
        dst[i] = v;
        dst32[i] = (float)v;
    }
}
}  // namespace

void launch_gather_pad(double *dst, float *dst32, const double *src,
                       const int32_t *idx, int64_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_gather_pad, dim3(grid_for(k, kWG, 16384)), dim3(kWG),
                       0, s, dst, dst32, src, idx, k);
}

// As k_gather_pad, of tiles (dst null: FP32 alone): an entry's place in the CSR is
// its position in the tile beyond the tile's first.
static __global__ __launch_bounds__(kWG) void k_gather_tiles(
    double *__restrict__ dst, float *__restrict__ dst32,
    const double *__restrict__ src, const int32_t *__restrict__ word,
    const int32_t *__restrict__ first, int64_t k) {
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < k;
         i += (int64_t)gridDim.x * kWG) {
        const double v = src[first[i >> 8] + (word[i] & ((1 << kTilePos) - 1))];
        if (dst) dst[i] = v;
        dst32[i] = (float)v;
    }
}

void launch_fill_buckets(const DevCsr &M, hipStream_t s) {
    const DevBuckets &K = *M.bkt;
    const int64_t k = 4 * K.quads;
    if (K.word)
        hipLaunchKernelGGL(k_gather_tiles, dim3(grid_for(k, kWG, 16384)), dim3(kWG),
                           0, s, K.v64, K.v32, M.v64, K.word, K.first, k);
    else
        launch_gather_pad(K.v64, K.v32, M.v64, K.src, k, s);
}

void launch_gather(double *dst, const double *src, const int32_t *idx,
                   int64_t k, hipStream_t s) {
    hipLaunchKernelGGL(k_gather, dim3(grid_for(k, kWG, 16384)), dim3(kWG), 0,
                       s, dst, src, idx, k);
}

void launch_refine_rhs(const double *bs, const double *ax, const double *cs,
                       const double *aty, const double *xs, const double *ls,
                       double DP, double DD, double *bh, double *ch,
                       double *lh, int64_t m, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_refine_rhs, dim3(grid_for(n > m ? n : m, kWG, 4096)),
                       dim3(kWG), 0, s, bs, ax, cs, aty, xs, ls, DP, DD, bh,
                       ch, lh, m, n);
}

void launch_refine_delta(const double *bs, const double *ax, const double *cs,
                         const double *aty, const double *xs,
                         const double *ls, const double *dr, const double *dc,
                         int64_t m, int64_t n, double *partial, double *out2,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_refine_delta, dim3(kRedBlocks), dim3(kWG), 0, s, bs,
                       ax, cs, aty, xs, ls, dr, dc, m, n, partial);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kWG), 0, s, partial,
                       kRedBlocks, out2, 1);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kWG), 0, s,
                       partial + kRedBlocks, kRedBlocks, out2 + 1, 1);
}

template <typename T>
void launch_refine_update(double *xs, double *ys, const T *xh, const T *yh,
                          const double *ls, double DP, double DD, int64_t m,
                          int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_refine_update<T>,
                       dim3(grid_for(n > m ? n : m, kWG, 4096)), dim3(kWG), 0,
                       s, xs, ys, xh, yh, ls, 1.0 / DP, 1.0 / DD, m, n);
}
template void launch_refine_update<float>(double *, double *, const float *,
                                          const float *, const double *,
                                          double, double, int64_t, int64_t,
                                          hipStream_t);
template void launch_refine_update<double>(double *, double *, const double *,
                                           const double *, const double *,
                                           double, double, int64_t, int64_t,
                                           hipStream_t);

// ============================================================ gather probe

namespace {

// splitmix64 finaliser (Steele, Lea and Flood's SplitMix generator): a
// counter-based hash giving the probe its random indices.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Indices of the probe's stream: entry i belongs to workgroup i / chunk,
// which gathers only from its panel (w % 8) % P of the table, as the row
// blocks of a panelled SpMV side do (workgroup w runs on XCD w % 8).
__global__ __launch_bounds__(kWG) void k_probe_fill(int32_t *idx, int64_t n,
                                                    int64_t chunk,
                                                    int64_t table, int P,
                                                    uint64_t seed) {
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n; i += stride) {
        const int64_t w = i / chunk;
        const int p = (int)((w % 8) % P);
        const int64_t lo = table * p / P, hi = table * (p + 1) / P;
        idx[i] = (int32_t)(lo + (int64_t)(mix64(seed + (uint64_t)i) % (uint64_t)(hi - lo)));
    }
}

// The SpMV's memory pattern without the row structure: workgroup w streams
// the (index, value) pairs [w chunk, (w + 1) chunk) with 16-byte loads, four
// per thread at a time, gathers table[index] for each and sums the products.
template <typename T, bool NT>
__global__ __launch_bounds__(kWG) void k_gather_probe(const int32_t *idx,
                                                      const T *val,
                                                      const T *table,
                                                      int64_t chunk,
                                                      int64_t n, T *out) {
    __shared__ T sred[4];
    const int64_t b0 = (int64_t)blockIdx.x * chunk;
    const int64_t b1 = b0 + chunk < n ? b0 + chunk : n;
    T acc = 0;
    for (int64_t p = b0 + 4 * (int64_t)threadIdx.x; p < b1; p += 4 * kWG) {
        int j[4];
        T a[4];
        ld4<NT>(idx + p, j);
        ld4<NT>(val + p, a);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (p + q < b1) acc += a[q] * table[j[q]];
    }
    acc = block_sum(acc, sred);
    if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

}  // namespace

void launch_probe_fill(int32_t *idx, int64_t n, int64_t chunk, int64_t table,
                       int P, uint64_t seed, hipStream_t s) {
    hipLaunchKernelGGL(k_probe_fill, dim3(grid_for(n, kWG, 16384)), dim3(kWG),
                       0, s, idx, n, chunk, table, P, seed);
}

template <typename T>
void launch_gather_probe(const int32_t *idx, const T *val, const T *table,
                         int64_t chunk, int64_t n, bool nt, T *out,
                         hipStream_t s) {
    const int g = (int)((n + chunk - 1) / chunk);
    if (nt)
        hipLaunchKernelGGL((k_gather_probe<T, true>), dim3(g), dim3(kWG), 0, s,
                           idx, val, table, chunk, n, out);
    else
        hipLaunchKernelGGL((k_gather_probe<T, false>), dim3(g), dim3(kWG), 0, s,
                           idx, val, table, chunk, n, out);
}
template void launch_gather_probe<double>(const int32_t *, const double *,
                                          const double *, int64_t, int64_t,
                                          bool, double *, hipStream_t);
template void launch_gather_probe<float>(const int32_t *, const float *,
                                         const float *, int64_t, int64_t,
                                         bool, float *, hipStream_t);

}  // namespace pdhg
