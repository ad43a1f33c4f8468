// bsde_host.cpp -- C ABI of libbsde.so: problem set-up (index set, grid,
// derivative channel matrices on the host; the Chebyshev basis matrix and
// its rank-checked pseudo-inverse R^{-1} Q' by CholeskyQR2 on the device),
// device buffers, the Picard loop that launches the HIP kernels, and the
// price/delta read-out.
//
// The method is Algorithm "algodetail" of Labart & Lelong (arXiv:1102.4666,
// Section 4.1); the least-squares extrapolating operator is that of
// Section 4.2 (eq. lspb) with polynomials centred and normalised to
// [-1, 1]^{d+1}; the model is Section 5 (eq. 4) with the correlation of
// Section 6.2.
#include "bsde_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <tuple>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

namespace bsde {
bool kernel_exists(int d, int eta, int q10);
int index_table(int d, int eta, int q10, int8_t *nu, int cap);
// ev0/ev1 (may be null): start and end times of the path-kernel dispatch
hipError_t launch_path(int d, int eta, int q10, bool fp32, int blocks, hipStream_t s,
                       const PathParams &prm, const double *pts,
                       const void *gamma, double *partial,
                       hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t launch_update(int n, int groups, int M, int ppg, int p, int nnz,
                         hipStream_t s, const double *partial, double *c,
                         double *var, const double *W, double *beta,
                         const double *alpha_in, double *alpha_out,
                         const int *rowptr, const int *cols, const double *vals,
                         double *g64, float *g32, hipEvent_t *ev);
hipError_t launch_channels(int p, int nnz, hipStream_t s, const double *alpha,
                           const int *rowptr, const int *cols, const double *vals,
                           double *g64, float *g32);
hipError_t launch_batch(int d, int eta, int q10, bool fp32, int vol, int blocks,
                        hipStream_t s, const BatchTileDesc *probs, int nprob,
                        const long long *tile_begin, unsigned int *counter);
int batch_occupancy(int d, int eta, int q10, bool fp32, int vol);
bool variant_exists(int d, int eta, int q10, bool fp32, int vol);
hipError_t launch_batch_update(int nprob, int max_n, int max_p, int max_cb,
                               hipStream_t s, const BatchUpdateDesc *d);
hipError_t launch_batch_channels(int nprob, int max_cb, hipStream_t s,
                                 const BatchUpdateDesc *d);
hipError_t launch_reset_counters(unsigned int *c, int n, hipStream_t s);
hipError_t launch_basis_matrix(const double *pts, int n, int ld, int dp,
                               const int8_t *nu, int pa, int pap, int eta,
                               const double *mid, const double *scale,
                               double T, double *B, hipStream_t s);
hipError_t launch_gram(const double *A, int ld, int pap, int rows_per_chunk,
                       int chunks, const int2 *pairs, int npairs,
                       double *partial, int pa, double *G, bool beside, hipStream_t s);
hipError_t launch_gemm_ax(const double *A, int ld, const double *X, int pap, bool upper,
                          double *Y, int ldy, int nrows, const int *colmap,
                          int ncols, hipStream_t s, const int *skip);
size_t factor_workspace(int pap);
hipError_t launch_factor(const double *G, int pa, int pap, double rel_tol, int stage,
                         double *X1, double *Xp, double *work, int *status, bool beside,
                         hipStream_t s);
hipError_t launch_project(const double *W, const double *c, int n, int p, double *beta,
                          hipStream_t s);
bool kernel_op_exists(int d, int vol);
hipError_t launch_kernel_path(int d, bool fp32, int blocks, hipStream_t s,
                              const PathParams &prm, const double *pts,
                              const void *table, double *partial,
                              hipEvent_t ev0, hipEvent_t ev1);
hipError_t launch_kernel_update(const PathParams &prm, int d, const double *pts,
                                const double *yprev, const double *c, double *ynew,
                                void *table, int fp32, hipStream_t s);
hipError_t launch_finalize(const double *partial, int n, int groups, int M,
                           int ppg, double *c, double *var, hipStream_t s);
} // namespace bsde

using namespace bsde;

static thread_local std::string g_last_error;

// ---------------------------------------------------------------------------
// Caching device allocator: buffers of released problems are kept per
// (device, size class) and handed to later problems, so that creating and
// destroying problems does not go through hipMalloc / hipFree each time.
// Size classes are powers of two from 256 bytes.  Thread-safe.
// ---------------------------------------------------------------------------
namespace {
struct DevicePool {
    std::mutex mu;
    std::map<std::pair<int, size_t>, std::vector<void *>> free_lists;
    std::map<void *, std::pair<int, size_t>> live;
    size_t cached_bytes = 0;
};
DevicePool &pool()
{
    static DevicePool *p = new DevicePool(); // never destroyed: buffers live
    return *p;                               // until the process ends
}
size_t size_class(size_t bytes)
{
    size_t c = 256;
    while (c < bytes) c <<= 1;
    return c;
}
hipError_t pool_alloc(void **ptr, size_t bytes)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t cls = size_class(bytes);
    DevicePool &P = pool();
    {
        std::lock_guard<std::mutex> g(P.mu);
        auto &fl = P.free_lists[{dev, cls}];
        if (!fl.empty()) {
            *ptr = fl.back();
            fl.pop_back();
            P.cached_bytes -= cls;
            P.live[*ptr] = {dev, cls};
            return hipSuccess;
        }
    }
    e = hipMalloc(ptr, cls);
    if (e == hipErrorOutOfMemory) {
        // release the cache of this device and retry once
        std::lock_guard<std::mutex> g(P.mu);
        for (auto &kv : P.free_lists)
            if (kv.first.first == dev) {
                for (void *q : kv.second) (void)hipFree(q);
                P.cached_bytes -= kv.first.second * kv.second.size();
                kv.second.clear();
            }
        e = hipMalloc(ptr, cls);
    }
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> g(P.mu);
    P.live[*ptr] = {dev, cls};
    return hipSuccess;
}
void pool_free(void *ptr)
{
    if (!ptr) return;
    DevicePool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    auto it = P.live.find(ptr);
    if (it == P.live.end()) return;
    P.free_lists[it->second].push_back(ptr);
    P.cached_bytes += it->second.second;
    P.live.erase(it);
}

// HIP events are reused across solves for the kernel timings.
std::mutex g_ev_mu;
std::vector<hipEvent_t> g_events;
hipError_t event_get(hipEvent_t *e)
{
    {
        std::lock_guard<std::mutex> g(g_ev_mu);
        if (!g_events.empty()) {
            *e = g_events.back();
            g_events.pop_back();
            return hipSuccess;
        }
    }
    return hipEventCreate(e);
}
void event_put(hipEvent_t e)
{
    std::lock_guard<std::mutex> g(g_ev_mu);
    g_events.push_back(e);
}

// Side streams of a device for the parallel branches of a batched solve
// (default priority, non-blocking), with the events that fork them from and
// join them back to the caller's stream.  Created once per device; the
// batched solves of one device take turns on them.
struct SideStreams {
    static constexpr int kCount = 3; // with the caller's stream, four queues
    hipStream_t s[kCount] = {};
    hipEvent_t fork = nullptr, join[kCount] = {};
    std::mutex mu;
};
std::mutex g_side_mu;
std::map<int, SideStreams *> g_side;
hipError_t side_streams(SideStreams **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> g(g_side_mu);
    auto it = g_side.find(dev);
    if (it != g_side.end()) {
        *out = it->second;
        return hipSuccess;
    }
    auto *ss = new SideStreams(); // kept until the process ends
    for (int k = 0; k < SideStreams::kCount && e == hipSuccess; ++k) {
        e = hipStreamCreateWithFlags(&ss->s[k], hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ss->join[k], hipEventDisableTiming);
    }
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ss->fork, hipEventDisableTiming);
    if (e != hipSuccess) return e; // (the partial set is not reused)
    g_side[dev] = ss;
    *out = ss;
    return hipSuccess;
}

// The instantiated graph of the last captured batched solve of a device,
// with the descriptor tables it reads and the launch plan it was captured
// from (a later batch with the same tables and plan replays it).
struct GraphCache {
    std::vector<char> blob;
    std::vector<long long> launches;
    char *dblob = nullptr;
    hipGraphExec_t exec = nullptr;
    void release()
    {
        if (exec) (void)hipGraphExecDestroy(exec);
        exec = nullptr;
        pool_free(dblob);
        dblob = nullptr;
        blob.clear();
        launches.clear();
    }
};
std::mutex g_graph_mu;
std::map<int, GraphCache> g_graph_cache;
} // namespace

bsde_status bsde::fail(bsde_status s, const std::string &msg)
{
    g_last_error = msg;
    return s;
}

// ---------------------------------------------------------------------------
// Set-up helpers
// ---------------------------------------------------------------------------
static bool cholesky(int d, double rho, double *L)
{
    for (int j = 0; j < kMaxD * kMaxD; ++j) L[j] = 0.0;
    for (int j = 0; j < d; ++j)
        for (int k = 0; k <= j; ++k) {
            double s = (j == k) ? 1.0 : rho;
            for (int l = 0; l < k; ++l) s -= L[j * kMaxD + l] * L[k * kMaxD + l];
            if (j == k) {
                if (!(s > 0.0)) return false;
                L[j * kMaxD + j] = std::sqrt(s);
            } else {
                L[j * kMaxD + k] = s / L[k * kMaxD + k];
            }
        }
    return true;
}

static double cheb_value(int a, double z)
{
    double t0 = 1.0, t1 = z;
    if (a == 0) return t0;
    for (int k = 1; k < a; ++k) {
        double t2 = 2.0 * z * t1 - t0;
        t0 = t1;
        t1 = t2;
    }
    return t1;
}

// coefficient of T_b in the derivative of T_a
static double cheb_deriv_coef(int a, int b)
{
    if (b >= a || ((a - b) & 1) == 0) return 0.0;
    return b == 0 ? (double)a : 2.0 * a;
}

// q in tenths when a kernel of that hyperbolic set is built for (d, eta),
// else 10 (the total-degree kernel, used with a mask for q < 1)
static int kernel_q10(int d, int eta, double q)
{
    const double q10 = q * 10.0;
    const int r = (int)std::lround(q10);
    if (r >= 1 && r < 10 && std::fabs(q10 - r) < 1e-9 && kernel_exists(d, eta, r)) return r;
    return 10;
}

// Set-up streams (non-blocking, one per concurrent set-up, reused)
namespace {
std::mutex g_stream_mu;
std::map<int, std::vector<hipStream_t>> g_setup_streams;
hipError_t setup_stream_get(hipStream_t *s)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> g(g_stream_mu);
        auto &v = g_setup_streams[dev];
        if (!v.empty()) {
            *s = v.back();
            v.pop_back();
            return hipSuccess;
        }
    }
    return hipStreamCreateWithFlags(s, hipStreamNonBlocking);
}
void setup_stream_put(hipStream_t s)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    std::lock_guard<std::mutex> g(g_stream_mu);
    g_setup_streams[dev].push_back(s);
}
} // namespace

// The rows of a problem's table in the cubic form (bsde_common.h) as
// combinations of the Chebyshev coefficients, in table order: put(row,
// factor) takes one entry.
template <typename Put>
static void cubic_rows(int d, bool fp32, int kind,
                       const std::map<std::vector<int8_t>, int> &pos, Put &&put)
{
    using Row = std::map<int, double>;
    const int dp = d + 1;
    // monomial coefficients of u, those of T_0 .. T_5 being
    static const double cheb[6][6] = {{1, 0, 0, 0, 0, 0},   {0, 1, 0, 0, 0, 0},
                                      {-1, 0, 2, 0, 0, 0},  {0, -3, 0, 4, 0, 0},
                                      {1, 0, -8, 0, 8, 0},  {0, 5, 0, -20, 0, 16}};
    std::map<std::vector<int8_t>, Row> mono; // at tau
    for (const auto &f : pos) {
        std::vector<std::pair<std::vector<int8_t>, double>> terms(
            1, {std::vector<int8_t>(dp, 0), 1.0});
        for (int v = 0; v < dp; ++v) {
            const int a = f.first[v];
            if (a == 0) continue;
            std::vector<std::pair<std::vector<int8_t>, double>> next;
            for (const auto &t : terms)
                for (int b = a & 1; b <= a; b += 2) {
                    next.push_back(t);
                    next.back().first[v] = (int8_t)b;
                    next.back().second *= cheb[a][b];
                }
            terms.swap(next);
        }
        for (const auto &t : terms) mono[t.first][f.second] += t.second;
    }
    std::map<std::vector<int8_t>, Row> mono_t; // at T: z_0 = 1
    for (const auto &m : mono) {
        std::vector<int8_t> mu = m.first;
        mu[0] = 0;
        Row &r = mono_t[mu];
        for (const auto &x : m.second) r[x.first] += x.second;
    }
    // the derivative at 0 along the variates of `by`: the monomial's
    // coefficient times the factorials of its exponents
    auto at0 = [&](std::map<std::vector<int8_t>, Row> &m, std::initializer_list<int> by,
                   double f) -> std::pair<const Row *, double> {
        std::vector<int8_t> mu(dp, 0);
        for (int v : by) f *= ++mu[v]; // 1, then 2, then 3 of the same variate
        return {&m[mu], f};
    };
    auto put_row = [&](std::pair<const Row *, double> e) {
        put(std::vector<std::pair<int, double>>(e.first->begin(), e.first->end()), e.second);
    };
    const CubicLayout lay(d, fp32, kind);
    auto row_tau = [&](int r, int k) { // coefficient k (0: constant) of row r
        if (r < lay.pairs) {
            const int v = hess_j(dp, r), w = hess_k(dp, r);
            return k == 0 ? at0(mono, {v, w}, 1.0) : at0(mono, {v, w, k - 1}, 1.0);
        }
        if (r < lay.pairs + dp) {
            const int v = r - lay.pairs;
            return k == 0 ? at0(mono, {v}, 1.0) : at0(mono, {v, k - 1}, 0.5);
        }
        return k == 0 ? at0(mono, {}, 1.0) : at0(mono, {k - 1}, 1.0 / 3.0);
    };
    auto row_t = [&](int r, int k) {
        if (r < lay.pairs_t) {
            const int v = 1 + hess_j(d, r), w = 1 + hess_k(d, r);
            const double f = v == w ? 1.0 : 2.0;
            return k == 0 ? at0(mono_t, {v, w}, f / 2.0) : at0(mono_t, {v, w, k}, f / 6.0);
        }
        return k == 0 ? at0(mono_t, {}, 1.0) : at0(mono_t, {k}, 1.0);
    };
    static const Row empty;
    const std::pair<const Row *, double> none{&empty, 0.0};
    if (fp32) {
        int e = 0;
        for (int part = 0; part < 2; ++part) {
            const int rows = part ? lay.rows_t : lay.rows, nk = part ? lay.kt : lay.ka;
            for (int g = 0; g < CubicLayout::groups(rows); ++g)
                for (int k = 0; k < nk; ++k)
                    for (int r = 4 * g; r < 4 * g + 4; ++r, ++e)
                        put_row(r >= rows ? none : part ? row_t(r, k) : row_tau(r, k));
        }
        for (; e < lay.off_q; ++e) put_row(none);
    }
    for (int r = 0; r < lay.rows && !fp32; ++r)
        for (int k = 0; k < lay.ka; ++k) put_row(row_tau(r, k));
    // coefficients of the monomials themselves
    auto coef = [&](std::map<std::vector<int8_t>, Row> &m, std::initializer_list<int> by) {
        std::vector<int8_t> mu(dp, 0);
        for (int v : by) ++mu[v];
        return std::pair<const Row *, double>{&m[mu], 1.0};
    };
    if (!fp32) {
        put_row(coef(mono_t, {}));
        for (int j = 1; j <= d; ++j) {
            put_row(coef(mono_t, {j}));
            for (int k = j; k <= d; ++k) {
                put_row(coef(mono_t, {j, k}));
                for (int l = k; l <= d; ++l) put_row(coef(mono_t, {j, k, l}));
            }
        }
    }
    for (int v = 0; v <= d && kind == 2; ++v) {
        put_row(coef(mono, {v, v, v, v}));
        put_row(coef(mono, {v, v, v, v, v}));
    }
}

// The points of Picard iteration k.  Uniform kind: n points uniform over
// [0, T] x D.  Otherwise time-major (point i = a n_spatial + b):
// time nodes a T / (n_t - 1); tensor grid digits equispaced in [-1, 1]; or
// Philox-uniform spatial points from the counter (b, 0, k', 2 << 24 |
// block) with k' = k when the points are redrawn every iteration, else 0.
// One counter serves four words and the spatial points are drawn once, not
// per time node: 0.35 ms for 81 920 points at d = 10, 4 ms less than with a
// draw for every coordinate of every point.
static void make_points(const bsde_problem_s *h, int k, std::vector<double> &pts)
{
    const int d = h->d, dp = d + 1;
    const long ns = h->n_spatial;
    const uint64_t seed = h->base.seed;
    const uint32_t kdraw = (h->redraw && h->grid_kind != BSDE_GRID_TENSOR) ? (uint32_t)k : 0u;
    pts.resize((size_t)h->n * dp);
    // the first `count` uniforms in (0, 1) of the counter (i, 0, k', sub << 24 |
    // block), four words a block
    auto uniforms = [&](uint32_t i, uint32_t sub, int count, double *u) {
        for (int q = 0; q < count; q += 4) {
            const u32x4 w = philox10(i, 0, kdraw, (sub << 24) | (uint32_t)(q / 4),
                                     (uint32_t)seed, (uint32_t)(seed >> 32));
            const uint32_t word[4] = {w.x, w.y, w.z, w.w};
            for (int c = 0; c < 4 && q + c < count; ++c)
                u[q + c] = ((double)word[c] + 0.5) * 0x1p-32;
        }
    };
    double u[kMaxD + 1];
    if (h->grid_kind == BSDE_GRID_UNIFORM) {
        // point i: word q of the counter (i, 0, k', 3 << 24 | q / 4) gives
        // t (q = 0) and x_j (q = 1 + j), uniform on [0, T] and [lo_j, hi_j]
        for (int i = 0; i < h->n; ++i) {
            double *row = &pts[(size_t)i * dp];
            uniforms((uint32_t)i, 3, dp, u);
            row[0] = h->base.T * u[0];
            for (int j = 0; j < d; ++j) row[1 + j] = h->lo[j] + u[1 + j] * (h->hi[j] - h->lo[j]);
        }
        return;
    }
    // the spatial points, in the rows of the first time node
    for (long s = 0; s < ns; ++s) {
        double *row = &pts[(size_t)s * dp];
        if (h->grid_kind != BSDE_GRID_TENSOR) uniforms((uint32_t)s, 2, d, u);
        long rest = s;
        for (int j = 0; j < d; ++j) {
            double z;
            if (h->grid_kind == BSDE_GRID_TENSOR) {
                long digit = rest % h->n_x;
                rest /= h->n_x;
                z = h->n_x > 1 ? -1.0 + 2.0 * digit / (h->n_x - 1) : 0.0;
            } else {
                z = 2.0 * u[j] - 1.0;
            }
            row[1 + j] = h->lo[j] + 0.5 * (z + 1.0) * (h->hi[j] - h->lo[j]);
        }
    }
    for (int a = 0; a < h->n_t; ++a) {
        // (the last is T itself, which the product can miss by its rounding)
        const double t = a == h->n_t - 1 ? h->base.T : a * h->base.T / (h->n_t - 1);
        double *rows = &pts[(size_t)a * ns * dp];
        if (a) std::memcpy(rows, pts.data(), sizeof(double) * (size_t)ns * dp);
        for (long s = 0; s < ns; ++s) rows[(size_t)s * dp] = t;
    }
}

// Shapes of the set-up: the leading dimension of the n x pap point matrices
// and the row chunks of the Gram kernel
static void setup_shape(int n, int pap, int &ld, int &rpc, int &chunks)
{
    // an odd multiple of 64 rows: columns a power of two of rows apart would
    // fall on the same memory channels
    ld = (((n + 63) / 64) | 1) * 64;
    const int nb = (pap + 63) / 64;
    // about 2048 single-wave workgroups over the block pairs and chunks,
    // at least 64 rows a chunk (a chunk's loads are a dependent chain, so
    // small problems want many short chunks)
    const int want = std::max(1, 2048 / (nb * (nb + 1) / 2));
    rpc = std::max(64, ((ld + want - 1) / want + 15) & ~15);
    chunks = (ld + rpc - 1) / rpc;
}

// Pinned host staging buffers for uploads: size classes of powers of two,
// reused, held until the process ends (like the device pool).
namespace {
std::mutex g_pin_mu;
std::multimap<size_t, void *> g_pin_free;
constexpr size_t kPinnedMax = size_t(16) << 20; // larger uploads stage in HIP
} // namespace
static void *pinned_get(size_t bytes, size_t *cap)
{
    size_t c = 4096;
    while (c < bytes) c <<= 1;
    *cap = c;
    {
        std::lock_guard<std::mutex> g(g_pin_mu);
        auto it = g_pin_free.find(c);
        if (it != g_pin_free.end()) {
            void *p = it->second;
            g_pin_free.erase(it);
            return p;
        }
    }
    void *p = nullptr;
    if (hipHostMalloc(&p, c, hipHostMallocDefault) != hipSuccess) return nullptr;
    return p;
}
static void pinned_put(void *p, size_t cap)
{
    if (!p) return;
    std::lock_guard<std::mutex> g(g_pin_mu);
    g_pin_free.emplace(cap, p);
}

// A pinned buffer of one call; get() is null when the size is not worth
// pinning or no memory could be pinned
namespace {
class PinnedBuffer {
public:
    explicit PinnedBuffer(size_t bytes)
        : p_(bytes <= kPinnedMax ? pinned_get(bytes, &cap_) : nullptr)
    {
    }
    PinnedBuffer(const PinnedBuffer &) = delete;
    PinnedBuffer &operator=(const PinnedBuffer &) = delete;
    ~PinnedBuffer() { pinned_put(p_, cap_); }
    void *get() { return p_; }

private:
    size_t cap_ = 0;
    void *p_;
};
} // namespace

// Pseudo-inverse W = B^+ (p x n, row-major; rows of inactive multi-indices
// zero) of the basis matrix of the grid by CholeskyQR2 on the device: the
// basis matrix from the device copy of the points, the Gram matrices, the
// factorisations and the products.  init allocates the workspace and uploads
// the small inputs, enqueue runs everything stream-ordered on s (the points
// must be uploaded on s or before) and ends with the copy of the status to
// host memory: 0, or not when B is numerically rank deficient (a Cholesky
// pivot of B'B below 1e-7 of the largest, i.e. a condition number beyond
// ~1e7); W is then left as it was.  The workspace goes back to the pool with
// the object, so s must be synchronized before.
namespace {
class PseudoInverse {
public:
    explicit PseudoInverse(const bsde_problem_s *h) : h_(h) {}
    PseudoInverse(const PseudoInverse &) = delete;
    PseudoInverse &operator=(const PseudoInverse &) = delete;
    ~PseudoInverse()
    {
        for (void *q : {(void *)dB_, (void *)dQ_, (void *)dPart_, (void *)dG_, (void *)dSmall_})
            pool_free(q);
        if (stage_pageable_.empty()) pinned_put(stage_, pin_cap_);
    }

    hipError_t init(hipStream_t s)
    {
        const std::vector<int> &act = h_->act;
        const int dp = h_->d + 1;
        pa_ = (int)act.size();
        pap_ = pad16(pa_);
        setup_shape(h_->n, pap_, ld_, rpc_, chunks_);
        std::vector<int2> pairs;
        const int nb = (pap_ + 63) / 64;
        for (int bi = 0; bi < nb; ++bi)
            for (int bj = bi; bj < nb; ++bj) pairs.push_back(make_int2(bi, bj));
        npairs_ = (int)pairs.size();
        // the small inputs of the set-up kernels travel in one upload:
        // index set | domain map | Gram block pairs | active columns | status
        auto al8 = [](size_t b) { return (b + 7) & ~(size_t)7; };
        o_ms_ = al8((size_t)pa_ * dp);
        o_pairs_ = o_ms_ + sizeof(double) * 2 * kMaxD;
        o_map_ = o_pairs_ + sizeof(int2) * pairs.size();
        o_status_ = al8(o_map_ + sizeof(int) * pa_);
        const size_t n_small = o_status_ + 8;
        stage_ = (unsigned char *)pinned_get(n_small, &pin_cap_);
        if (!stage_) {
            stage_pageable_.resize(n_small);
            stage_ = stage_pageable_.data();
        }
        std::memset(stage_, 0, n_small);
        for (int c = 0; c < pa_; ++c)
            std::memcpy(stage_ + (size_t)c * dp, &h_->nu[(size_t)act[c] * dp], dp);
        std::memcpy(stage_ + o_ms_, h_->base.mid, sizeof(double) * h_->d);
        std::memcpy(stage_ + o_ms_ + sizeof(double) * kMaxD, h_->base.scale,
                    sizeof(double) * h_->d);
        std::memcpy(stage_ + o_pairs_, pairs.data(), sizeof(int2) * pairs.size());
        std::memcpy(stage_ + o_map_, act.data(), sizeof(int) * pa_);

        // two p x n point matrices, the Gram partials, and the p x p matrices
        // (G, the two right factors and the factorisation's own) in one block
        const size_t sq = (size_t)pap_ * pap_;
        hipError_t e = pool_alloc((void **)&dB_, sizeof(double) * ld_ * pap_);
        if (e == hipSuccess) e = pool_alloc((void **)&dQ_, sizeof(double) * ld_ * pap_);
        if (e == hipSuccess) e = pool_alloc((void **)&dPart_, sizeof(double) * chunks_ * sq);
        if (e == hipSuccess)
            e = pool_alloc((void **)&dG_, sizeof(double) * (3 * sq + factor_workspace(pap_)));
        if (e == hipSuccess) e = pool_alloc((void **)&dSmall_, n_small);
        if (e == hipSuccess)
            e = hipMemcpyAsync(dSmall_, stage_, n_small, hipMemcpyHostToDevice, s);
        return e;
    }

    // of the points pts into W, whose rows of inactive multi-indices it leaves
    // (the caller has made them zero); beside: a path kernel fills the GPU meanwhile
    hipError_t enqueue(hipStream_t s, int *status, const double *pts, double *W, bool beside)
    {
        const int n = h_->n;
        const size_t sq = (size_t)pap_ * pap_;
        double *dX1 = dG_ + sq, *dX = dG_ + 2 * sq, *dWork = dG_ + 3 * sq;
        const double *dMS = (const double *)(dSmall_ + o_ms_);
        const int2 *dPairs = (const int2 *)(dSmall_ + o_pairs_);
        int *dStatus = (int *)(dSmall_ + o_status_);
        hipError_t e = launch_basis_matrix(pts, n, ld_, h_->d + 1, (const int8_t *)dSmall_,
                                           pa_, pap_, h_->eta, dMS, dMS + kMaxD, h_->base.T, dB_,
                                           s);
        if (e == hipSuccess)
            e = launch_gram(dB_, ld_, pap_, rpc_, chunks_, dPairs, npairs_, dPart_, pa_, dG_, beside, s);
        // a failed rank test leaves its status, and the later steps do nothing
        if (e == hipSuccess) e = launch_factor(dG_, pa_, pap_, 1e-7, 1, dX1, dX, dWork, dStatus, beside, s);
        if (e == hipSuccess)
            e = launch_gemm_ax(dB_, ld_, dX1, pap_, true, dQ_, ld_, ld_, nullptr, pap_, s, dStatus);
        if (e == hipSuccess)
            e = launch_gram(dQ_, ld_, pap_, rpc_, chunks_, dPairs, npairs_, dPart_, pa_, dG_, beside, s);
        if (e == hipSuccess) e = launch_factor(dG_, pa_, pap_, 1e-3, 2, dX1, dX, dWork, dStatus, beside, s);
        if (e == hipSuccess)
            e = launch_gemm_ax(dQ_, ld_, dX, pap_, false, W, n, n,
                               (const int *)(dSmall_ + o_map_), pa_, s, dStatus);
        if (e == hipSuccess)
            e = hipMemcpyAsync(status, dStatus, sizeof(int), hipMemcpyDeviceToHost, s);
        return e;
    }

    // host memory of the object for one status
    int *own_status() { return (int *)(stage_ + o_status_); }

private:
    const bsde_problem_s *h_;
    int pa_ = 0, pap_ = 0, ld_ = 0, rpc_ = 0, chunks_ = 0, npairs_ = 0;
    size_t o_ms_ = 0, o_pairs_ = 0, o_map_ = 0, o_status_ = 0, pin_cap_ = 0;
    unsigned char *stage_ = nullptr, *dSmall_ = nullptr;
    std::vector<unsigned char> stage_pageable_;
    double *dB_ = nullptr, *dQ_ = nullptr, *dPart_ = nullptr, *dG_ = nullptr;
};
constexpr const char *kRankMessage = "basis matrix is numerically rank deficient on the grid";
} // namespace

// The redrawn points of one solve on stream s (Algorithm 1).  An iteration's
// points and their pseudo-inverse do not depend on the iterate, and the
// set-up is a chain of small kernels: it runs on a stream of the library's own
// while the iteration before it runs on s, into the other of two sets of
// buffers, the problem's own and one of the solve's (one set, and everything
// on s, when that cannot be allocated or the paths are few).  Time outside
// the path kernel an iteration: 0.30 -> 0.03 ms at d = 10, n = 1000, p = 221,
// M = 30 000; 0.59 -> 0.05 at n = 1800, p = 364; 0.13 -> 0.03 at d = 5, p = 84; in
// FP64 at d = 10, whose path kernel leaves no registers free, 0.60 -> 0.50.
// draw(k) sends iteration k's points up from one of two pinned slots and
// enqueues their pseudo-inverse, begin(k) makes s wait for them and gives their
// set, end(k) frees it; finish() brings the last iteration's points and
// pseudo-inverse into the problem's own buffers.  The rank tests are looked at
// without a wait: failed() knows those of the draws that have ended when
// draw() reuses their slot, so that a solve stops two iterations after a
// deficient one, and full_rank() all of them once s is synchronized.  After a
// failure restore() leaves the problem with the points and pseudo-inverse of
// the iteration before the deficient one, the last that ran.
namespace {
class RedrawWork {
public:
    struct Set {
        double *pts, *W;
    };
    RedrawWork(bsde_problem_s *h, hipStream_t s)
        : h_(h), s_(s), set_{{h->d_pts, h->d_W}, {}}, from_(h->pts_k)
    {
    }
    RedrawWork(const RedrawWork &) = delete;
    RedrawWork &operator=(const RedrawWork &) = delete;
    ~RedrawWork()
    {
        if (!pinv_) return;
        // also after an error: the buffers go back
        if (side_) {
            (void)hipStreamSynchronize(side_);
            setup_stream_put(side_);
        }
        (void)hipStreamSynchronize(s_);
        if (count_ > 0 && !finished_) h_->pts_k = -1; // the points on the device are not known
        for (Slot &q : slot_) {
            pinned_put(q.mem, q.cap);
            if (q.sent) event_put(q.sent);
        }
        for (hipEvent_t ev : {ready_[0], ready_[1], used_[0], used_[1]})
            if (ev) event_put(ev);
        pool_free(set_[1].pts);
        pool_free(set_[1].W);
        pinned_put(pinned_status_, status_cap_);
    }

    // after: an event on s before which the buffers may be in use
    hipError_t draw(int k, hipEvent_t after)
    {
        const size_t bytes = sizeof(double) * h_->pts.size();
        hipError_t e = hipSuccess;
        if (!pinv_) init_error_ = init(bytes, after);
        if (init_error_ != hipSuccess) return init_error_;
        const hipStream_t ws = side_ ? side_ : s_;
        const int t = target(k);
        Slot &q = slot_[count_ & 1];
        if (!q.mem) e = hipStreamSynchronize(ws); // h->pts is still being read
        else if (count_ >= 2) e = hipEventSynchronize(q.sent);
        if (e != hipSuccess) return e;
        // (the slot's draw is on ws after the one before it)
        ended_ = q.mem ? std::max(0, count_ - 2) : count_;
        if (count_++ == 0) first_drawn_ = k;
        make_points(h_, k, h_->pts);
        if (q.mem) std::memcpy(q.mem, h_->pts.data(), bytes);
        if (side_ && in_use_[t]) e = hipStreamWaitEvent(side_, used_[t], 0);
        if (e == hipSuccess)
            e = hipMemcpyAsync(set_[t].pts, q.mem ? q.mem : (void *)h_->pts.data(), bytes,
                               hipMemcpyHostToDevice, ws);
        if (e == hipSuccess) e = hipEventRecord(q.sent, ws);
        if (e == hipSuccess)
            e = pinv_->enqueue(ws, status() + count_ - 1, set_[t].pts, set_[t].W,
                               side_ && long_path_);
        if (e == hipSuccess && side_) e = hipEventRecord(ready_[t], side_);
        if (e != hipSuccess) return e;
        h_->pts_k = drawn_ = k;
        return hipSuccess;
    }
    // whether iteration k's points have been drawn here
    bool drawn(int k) const { return count_ > 0 && drawn_ >= k; }
    // whether the next draw may run beside the present iteration (after an
    // error it reports it); before the iteration's end, which it makes count
    bool ahead(hipEvent_t after)
    {
        if (!pinv_) init_error_ = init(sizeof(double) * h_->pts.size(), after);
        return side_ != nullptr || init_error_ != hipSuccess;
    }

    hipError_t begin(int k, Set &set)
    {
        const int t = target(k);
        set = set_[t];
        return side_ && drawn(k) ? hipStreamWaitEvent(s_, ready_[t], 0) : hipSuccess;
    }
    hipError_t end(int k)
    {
        last_ = k;
        if (!side_) return hipSuccess;
        in_use_[target(k)] = true;
        return hipEventRecord(used_[target(k)], s_);
    }
    hipError_t finish()
    {
        hipError_t e = hipSuccess;
        if (pinv_ && target(last_) == 1) {
            e = hipMemcpyAsync(h_->d_pts, set_[1].pts, sizeof(double) * h_->pts.size(),
                               hipMemcpyDeviceToDevice, s_);
            if (e == hipSuccess)
                e = hipMemcpyAsync(h_->d_W, set_[1].W, sizeof(double) * (size_t)h_->p * h_->n,
                                   hipMemcpyDeviceToDevice, s_);
        }
        finished_ = e == hipSuccess;
        return e;
    }

    bool failed() { return deficient(ended_) < ended_; }
    bool full_rank() { return deficient(count_) == count_; }
    void restore()
    {
        h_->pts_k = -1;
        if (side_ && hipStreamSynchronize(side_) != hipSuccess) return;
        const int i = deficient(count_), k = i == 0 ? from_ : first_drawn_ + i - 1;
        if (k < 0) return;
        make_points(h_, k, h_->pts);
        hipError_t e = hipMemcpyAsync(h_->d_pts, h_->pts.data(), sizeof(double) * h_->pts.size(),
                                      hipMemcpyHostToDevice, s_);
        if (e == hipSuccess) e = pinv_->enqueue(s_, status(), h_->d_pts, h_->d_W, false);
        const hipError_t se = hipStreamSynchronize(s_);
        if (e == hipSuccess && se == hipSuccess && status()[0] == 0) h_->pts_k = k;
    }

private:
    hipError_t init(size_t bytes, hipEvent_t after)
    {
        pinv_.reset(new PseudoInverse(h_));
        status_.assign((size_t)h_->K_it, 0);
        hipError_t e = hipSuccess;
        for (Slot &q : slot_) {
            // (too large to pin: the points then go up from h->pts)
            if (bytes <= kPinnedMax) q.mem = pinned_get(bytes, &q.cap);
            if ((e = event_get(&q.sent)) != hipSuccess) return e;
        }
        first_ = h_->k_done;
        // The second stream's events cost some 10 us an iteration: not below
        // 2e7 asset steps, a path kernel of 40 us (d = 3, n = 300, M = 1000,
        // N = 5: 0.38 ms without, 0.45 with it; d = 5, n = 1000: 1.06 and
        // 1.01).  From 1e9 on the path kernel (0.6 ms and more) outlasts the
        // set-up, whose kernels are then those that fit beside it.
        const double steps = (double)h_->n * h_->M * h_->base.N * h_->d;
        long_path_ = steps > 1e9;
        const size_t w_bytes = sizeof(double) * (size_t)h_->p * h_->n;
        bool two = steps > 2e7 &&
                   pool_alloc((void **)&set_[1].pts, bytes) == hipSuccess &&
                   pool_alloc((void **)&set_[1].W, w_bytes) == hipSuccess;
        for (hipEvent_t *ev : {&ready_[0], &ready_[1], &used_[0], &used_[1]})
            two = two && event_get(ev) == hipSuccess;
        if (two && setup_stream_get(&side_) != hipSuccess) side_ = nullptr;
        if (steps > 2e7 && !side_) (void)hipGetLastError(); // one set does
        if (side_) {
            if ((e = hipStreamWaitEvent(side_, after, 0)) != hipSuccess) return e;
            if (h_->act.size() < (size_t)h_->p)
                e = hipMemsetAsync(set_[1].W, 0, w_bytes, side_);
        }
        if (e == hipSuccess) e = pinv_->init(side_ ? side_ : s_);
        if (e != hipSuccess) return e;
        pinned_status_ = (int *)pinned_get(sizeof(int) * status_.size(), &status_cap_);
        return hipSuccess;
    }
    // the set of iteration k: the problem's own first
    int target(int k) const { return side_ ? (k - first_) & 1 : 0; }
    int *status() { return pinned_status_ ? pinned_status_ : status_.data(); }
    // the first of `count` draws whose rank test failed, or count
    int deficient(int count)
    {
        int i = 0;
        while (i < count && status()[i] == 0) ++i;
        return i;
    }
    struct Slot {
        void *mem = nullptr;
        size_t cap = 0;
        hipEvent_t sent = nullptr;
    };
    bsde_problem_s *h_;
    hipStream_t s_, side_ = nullptr;
    std::unique_ptr<PseudoInverse> pinv_;
    Set set_[2];
    hipEvent_t ready_[2] = {nullptr, nullptr}, used_[2] = {nullptr, nullptr};
    bool in_use_[2] = {false, false}, finished_ = false, long_path_ = false;
    hipError_t init_error_ = hipSuccess;
    Slot slot_[2];
    int *pinned_status_ = nullptr;
    std::vector<int> status_;
    size_t status_cap_ = 0;
    // draws begun, those of them known to have ended, the first one's
    // iteration; the iteration whose points the solve began with
    int count_ = 0, ended_ = 0, first_drawn_ = 0, from_;
    int first_ = 0, drawn_ = -1, last_ = 0;
};
} // namespace

// The pseudo-inverse of the problem's points; synchronizes s
static bsde_status device_pseudo_inverse(const bsde_problem_s *h, hipStream_t s)
{
    PseudoInverse pinv(h);
    hipError_t e = pinv.init(s);
    if (e == hipSuccess && h->act.size() < (size_t)h->p) // rows that stay zero
        e = hipMemsetAsync(h->d_W, 0, sizeof(double) * (size_t)h->p * h->n, s);
    if (e == hipSuccess) e = pinv.enqueue(s, pinv.own_status(), h->d_pts, h->d_W, false);
    const hipError_t se = hipStreamSynchronize(s);
    if (e == hipSuccess) e = se;
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? BSDE_ENOMEM : BSDE_EDEVICE,
                    std::string("least-squares set-up: ") + hipGetErrorString(e));
    if (*pinv.own_status() != 0) return fail(BSDE_ERANK, kRankMessage);
    return BSDE_OK;
}

// the channel tables: dense, then the live rows packed (bsde_common.h)
static size_t table_floats(const bsde_problem_s *h)
{
    if (h->kop) return 0; // the kernel operator reads its point table instead
    return (size_t)h->n_live;
}

static void free_device(bsde_problem_s *h)
{
    pool_free(h->d_block);
    pool_free(h->d_W);
    pool_free(h->d_beta);
    pool_free(h->d_partial);
    pool_free(h->d_c);
    pool_free(h->d_var);
    h->d_pts = h->d_W = h->d_vals = h->d_alpha = h->d_beta = h->d_g64 = nullptr;
    h->d_partial = h->d_c = h->d_var = nullptr;
    h->d_g32 = nullptr;
    h->d_rowptr = h->d_cols = nullptr;
    h->d_block = nullptr;
}



#define HIP_TRY(expr)                                                          \
    do {                                                                       \
        hipError_t e_ = (expr);                                                \
        if (e_ != hipSuccess)                                                  \
            return fail(BSDE_EDEVICE, std::string(#expr) + ": " +              \
                                          hipGetErrorString(e_));              \
    } while (0)

// Tilings chosen by bsde_autotune, keyed by kernel signature and size
// class; consulted when a problem is created.
namespace {
struct TuneKey {
    int d, eta, q10, prec, vol, M, N, nclass;
    bool operator<(const TuneKey &o) const
    {
        return std::tie(d, eta, q10, prec, vol, M, N, nclass) <
               std::tie(o.d, o.eta, o.q10, o.prec, o.vol, o.M, o.N, o.nclass);
    }
};
std::mutex g_tune_mu;
std::map<TuneKey, std::pair<int, int>> g_tuned;

TuneKey tune_key(const bsde_problem_s *h)
{
    int nclass = 0;
    while ((1 << nclass) < h->n) ++nclass;
    return {h->d, h->eta, h->q10, h->precision, h->base.vol_kind, h->M, h->N, nclass};
}
} // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

const char *bsde_status_string(bsde_status s)
{
    switch (s) {
    case BSDE_OK: return "ok";
    case BSDE_EINVAL: return "invalid argument";
    case BSDE_ENOMEM: return "out of memory";
    case BSDE_ERANK: return "rank-deficient least-squares problem";
    case BSDE_EDEVICE: return "HIP device error";
    case BSDE_ESTATE: return "invalid state";
    case BSDE_EUNSUPPORTED: return "no kernel for this (d, eta)";
    case BSDE_EBUSY: return "request not finished";
    }
    return "unknown status";
}

const char *bsde_last_error(void) { return g_last_error.c_str(); }

} // extern "C"

static bsde_status prepare_tiling(bsde_problem h, int &groups, int &ppl,
                                  bool allow_alloc = true);

// Points of a grid and how many of them are spatial ones; 0 when its numbers
// are out of range or the points more than the 2^26 a problem may have
static int grid_points(int d, const bsde_grid *grid, int *spatial)
{
    const long most = 1L << 26, n_t = grid->kind == BSDE_GRID_UNIFORM ? 1 : grid->n_t;
    if (grid->n_x < 1 || n_t < 1) return 0;
    long ns = grid->n_x;
    for (int j = 1; j < d && grid->kind == BSDE_GRID_TENSOR && ns <= most; ++j) ns *= grid->n_x;
    if (ns > most || ns * n_t > most) return 0;
    *spatial = (int)ns;
    return (int)(ns * n_t);
}

extern "C" {

bsde_status bsde_create_problem(int d, const bsde_sigma *sigma, double r,
                                const bsde_payoff *payoff,
                                const bsde_grid *grid, int M, int N,
                                int n_picard, double penalty,
                                unsigned long long seed, int precision,
                                bsde_problem *out)
{
    if (out) *out = nullptr;
    if (!out || !sigma || !payoff || !grid || !sigma->level || !payoff->S0)
        return fail(BSDE_EINVAL, "null argument");
    if (d < 1 || d > kMaxD) return fail(BSDE_EINVAL, "d must be in [1, 10]");
    if (M < 1 || N < 1 || n_picard < 1)
        return fail(BSDE_EINVAL, "M, N and n_picard must be >= 1");
    if (!(penalty >= 0.0) || !std::isfinite(r))
        return fail(BSDE_EINVAL, "penalty must be >= 0 and r finite");
    if (!(payoff->T > 0.0) || payoff->kind < 0 || payoff->kind > 5)
        return fail(BSDE_EINVAL, "bad payoff");
    if (sigma->kind != BSDE_VOL_CONST && sigma->kind != BSDE_VOL_BUMP &&
        sigma->kind != BSDE_VOL_DUPIRE)
        return fail(BSDE_EINVAL, "bad volatility kind");
    if (sigma->kind == BSDE_VOL_BUMP && !(sigma->bump_c > 0.0))
        return fail(BSDE_EINVAL, "bump centre must be > 0");
    if (grid->kind != BSDE_GRID_TENSOR && grid->kind != BSDE_GRID_RANDOM &&
        grid->kind != BSDE_GRID_UNIFORM)
        return fail(BSDE_EINVAL, "bad grid kind");
    if (grid->redraw != 0 && (grid->redraw != 1 || grid->kind == BSDE_GRID_TENSOR))
        return fail(BSDE_EINVAL, "redraw needs random or uniform points");
    if ((grid->kind != BSDE_GRID_UNIFORM && grid->n_t < 2) || grid->n_x < 1 ||
        !(grid->width > 0.0) ||
        grid->eta < 1 || !(grid->q > 0.0 && grid->q <= 1.0))
        return fail(BSDE_EINVAL, "bad grid (n_t >= 2, n_x >= 1, width > 0, "
                                 "eta >= 1, 0 < q <= 1)");
    if (precision != BSDE_FP64 && precision != BSDE_FP32_PATHS)
        return fail(BSDE_EINVAL, "bad precision");
    for (int j = 0; j < d; ++j)
        if (!(sigma->level[j] > 0.0) || !(payoff->S0[j] > 0.0))
            return fail(BSDE_EINVAL, "levels and spots must be > 0");
    // the kernel operator of Section 3.2 instead of least squares
    const bool kop = grid->kernel_bw != 0.0;
    if (kop) {
        if (!(grid->kernel_bw > 0.0) || !std::isfinite(grid->kernel_bw))
            return fail(BSDE_EINVAL, "kernel_bw must be 0 or a finite bandwidth > 0");
        if (grid->redraw)
            return fail(BSDE_EUNSUPPORTED, "the kernel operator takes fixed points");
        if (!kernel_op_exists(d, sigma->kind))
            return fail(BSDE_EUNSUPPORTED, "the kernel operator is built for d <= 2 "
                                           "with constant or bump volatility");
    }
    // a kernel of the hyperbolic set itself when one is built, else the
    // total-degree kernel with the entries outside the set kept at zero
    const int q10 = kernel_q10(d, grid->eta, grid->q);
    if (kop) {
        // no basis: eta and q are not used
    } else if (!kernel_exists(d, grid->eta, q10))
        return fail(BSDE_EUNSUPPORTED, "no kernel instantiated for d=" +
                                           std::to_string(d) + ", eta=" +
                                           std::to_string(grid->eta));
    if (!kop && !variant_exists(d, grid->eta, q10, precision == BSDE_FP32_PATHS, sigma->kind))
        return fail(BSDE_EUNSUPPORTED,
                    "no kernel instantiated for d=" + std::to_string(d) + ", eta=" +
                        std::to_string(grid->eta) + " with this precision and "
                        "volatility kind (d = 10: FP64 paths for total degree "
                        "only; the Dupire-type volatility: d=1 eta=4, d=2 "
                        "eta=3, d=5 eta=2,3)");
    double Lc[kMaxD * kMaxD];
    if (!cholesky(d, sigma->rho, Lc))
        return fail(BSDE_EINVAL, "correlation matrix not positive definite");

    auto *h = new (std::nothrow) bsde_problem_s();
    if (!h) return fail(BSDE_ENOMEM, "host allocation");
    h->d = d;
    h->eta = grid->eta;
    h->q = grid->q;
    h->M = M;
    h->N = N;
    h->K_it = n_picard;
    h->omega = penalty;
    h->precision = precision;
    PathParams &b = h->base;
    b.seed = seed;
    b.M = M;
    b.N = N;
    b.vol_kind = sigma->kind;
    b.payoff = payoff->kind;
    b.r = r;
    b.omega = penalty;
    b.K = payoff->K;
    b.T = payoff->T;
    b.bump_a = sigma->kind == BSDE_VOL_BUMP ? sigma->bump_a : 0.0;
    b.log_bump_c = sigma->kind == BSDE_VOL_BUMP ? std::log(sigma->bump_c) : 0.0;
    b.rho = sigma->rho;
    std::memcpy(b.L, Lc, sizeof(Lc));
    h->lo.resize(d);
    h->hi.resize(d);
    for (int j = 0; j < d; ++j) {
        b.level[j] = sigma->level[j];
        b.spot[j] = payoff->S0[j];
        b.div[j] = sigma->dividend ? sigma->dividend[j] : 0.0;
        double half = grid->width * sigma->level[j] * std::sqrt(payoff->T);
        h->lo[j] = std::log(payoff->S0[j]) - half;
        h->hi[j] = std::log(payoff->S0[j]) + half;
        b.mid[j] = 0.5 * (h->lo[j] + h->hi[j]);
        b.scale[j] = 2.0 / (h->hi[j] - h->lo[j]);
    }
    fill_asset_consts(b, d);
    h->kop = kop;
    b.kbw = kop ? grid->kernel_bw : 0.0;

    // index set in kernel order; hyperbolic subset marked active (a
    // one-function placeholder for the kernel operator)
    const int dp = d + 1;
    h->q10 = q10;
    h->p = kop ? 1 : index_table(d, grid->eta, q10, nullptr, 0);
    h->nu.assign((size_t)h->p * dp, 0);
    if (!kop) index_table(d, grid->eta, q10, h->nu.data(), h->p);
    h->active.assign(h->p, 1);
    if (!kop && grid->q < 1.0) {
        for (int l = 0; l < h->p; ++l) {
            double s = 0.0;
            for (int v = 0; v < dp; ++v)
                if (h->nu[(size_t)l * dp + v]) s += std::pow((double)h->nu[(size_t)l * dp + v], grid->q);
            h->active[l] = s <= std::pow((double)grid->eta, grid->q) * (1.0 + 1e-12);
        }
    }
    h->C = num_channels(d);

    // grid points (time-major); uniform points: n_x of them, no time nodes
    int ns = 0;
    const int n_t = grid->kind == BSDE_GRID_UNIFORM ? 1 : grid->n_t;
    h->n = grid_points(d, grid, &ns);
    if (h->n == 0) {
        delete h;
        return fail(BSDE_EINVAL, "too many points");
    }
    h->n_spatial = ns;
    h->grid_kind = grid->kind;
    h->n_t = n_t;
    h->n_x = grid->n_x;
    h->redraw = grid->redraw;
    b.kop_nt = kop && grid->kind != BSDE_GRID_UNIFORM && n_t <= kKopTimes ? n_t : 0;
    h->pts_k = 0;
    make_points(h, 0, h->pts);

    // basis matrix over the active multi-indices and its pseudo-inverse
    std::vector<int> &act = h->act;
    for (int l = 0; l < h->p; ++l)
        if (h->active[l]) act.push_back(l);
    const int pa = (int)act.size();
    if (h->n < pa) {
        delete h;
        return fail(BSDE_ERANK, "fewer points than basis functions");
    }

    // The derivative channels as sparse rows over the basis: the derivative
    // of T_a in one variate is a combination of the T_b, b < a, a - b odd
    // (cheb_deriv_coef), so row mu of d/dz_v holds the functions mu + k e_v of
    // the set, k odd; rows columns ascending.  Channel 1 is d_t (2/T d/dz_0),
    // channel 2 + j d_{x_j} (scale_j d/dz_{1+j}), then the second
    // derivatives, the products of two of those.
    std::map<std::vector<int8_t>, int> pos;
    for (int l = 0; l < h->p; ++l)
        pos[std::vector<int8_t>(&h->nu[(size_t)l * dp], &h->nu[(size_t)l * dp] + dp)] = l;
    using SRow = std::vector<std::pair<int, double>>;
    std::vector<std::vector<SRow>> Dv(dp, std::vector<SRow>(h->p));
    for (int v = 0; v < dp && !kop; ++v) {
        for (int l = 0; l < h->p; ++l) {
            std::vector<int8_t> e(&h->nu[(size_t)l * dp], &h->nu[(size_t)l * dp] + dp);
            const int a = e[v];
            for (int bb = 0; bb < a; ++bb) {
                const double cf = cheb_deriv_coef(a, bb);
                if (cf == 0.0) continue;
                std::vector<int8_t> mu = e;
                mu[v] = (int8_t)bb;
                Dv[v][pos[mu]].push_back({l, cf});
            }
        }
        for (auto &r : Dv[v]) std::sort(r.begin(), r.end());
    }
    const double tfac = 2.0 / payoff->T;
    h->Dx.assign(kop ? 0 : d, std::vector<SRow>(h->p));
    for (int j = 0; j < d && !kop; ++j)
        for (int l = 0; l < h->p; ++l)
            for (const auto &x : Dv[1 + j][l]) h->Dx[j][l].push_back({x.first, b.scale[j] * x.second});
    // the packed channel table (bsde_common.h) as a sparse matrix over the
    // coefficients, in the order the path kernels read it: channel 0; each
    // second derivative over its live rows; then row by row the time
    // derivative and the gradient; then u(T, x).  The kernel's index set is
    // the set of rows here.
    std::vector<int> csr_ptr(1, 0), csr_col;
    std::vector<double> csr_val;
    if (!kop) {
        auto in_set = [&](const int *mu) {
            std::vector<int8_t> key(dp);
            for (int v = 0; v < dp; ++v) key[v] = (int8_t)mu[v];
            return pos.count(key) > 0;
        };
        auto live = [&](int l, int c) {
            return channel_row_live<kMaxD + 1>(&h->nu[(size_t)l * dp], dp, c, in_set);
        };
        auto put = [&](const SRow &r, double f) {
            for (const auto &x : r) {
                csr_col.push_back(x.first);
                csr_val.push_back(f * x.second);
            }
            csr_ptr.push_back((int)csr_col.size());
        };
        const int kind = cubic_kind(
            [&](int l, int v) { return (int)h->nu[(size_t)l * dp + v]; }, h->p, dp);
        if (kind > 0) {
            cubic_rows(d, precision == BSDE_FP32_PATHS, kind, pos, put);
        } else {
            for (int l = 0; l < h->p; ++l) put(SRow{{l, 1.0}}, 1.0);
            for (int c = 2 + d; c < h->C; ++c) {
                const int j = hess_j(d, c - 2 - d), k = hess_k(d, c - 2 - d);
                for (int l = 0; l < h->p; ++l) {
                    if (!live(l, c)) continue;
                    // row l of (d/dx_j)(d/dx_k): sum over the middle function mm,
                    // in ascending order
                    std::map<int, double> acc;
                    for (const auto &x1 : h->Dx[j][l])
                        for (const auto &x2 : h->Dx[k][x1.first]) acc[x2.first] += x1.second * x2.second;
                    put(SRow(acc.begin(), acc.end()), 1.0);
                }
            }
            for (int l = 0; l < h->p; ++l)
                for (int c = 1; c < 2 + d; ++c)
                    if (live(l, c)) put(Dv[c - 1][l], c == 1 ? tfac : b.scale[c - 2]);
            // u(T, x): the functions of every time degree over each spatial one
            for (int l = 0; l < h->p; ++l) {
                if (h->nu[(size_t)l * dp] != 0) continue;
                std::vector<int8_t> mu(&h->nu[(size_t)l * dp], &h->nu[(size_t)l * dp] + dp);
                SRow r;
                for (; mu[0] <= grid->eta; ++mu[0]) {
                    const auto it = pos.find(mu);
                    if (it != pos.end()) r.push_back({it->second, 1.0});
                }
                put(r, 1.0);
            }
        }
        h->n_live = (int)csr_ptr.size() - 1;
    }

    if (kop) {
        // the coefficients of a kernel-operator problem are its point values
        h->p = h->n;
    }

    // device buffers
    hipError_t alloc_err = hipSuccess;
    auto dalloc = [&](void **ptr, size_t bytes) {
        alloc_err = pool_alloc(ptr, bytes == 0 ? 8 : bytes);
        return alloc_err == hipSuccess;
    };
    // points, channel matrices, coefficients and channel tables in one
    // block (256-byte aligned parts)
    auto al256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t real_size = precision == BSDE_FP32_PATHS ? sizeof(float) : sizeof(double);
    const size_t b_pts = sizeof(double) * h->pts.size(),
                 b_val = sizeof(double) * csr_val.size(),
                 b_alpha = sizeof(double) * (size_t)(h->K_it + 1) * h->p,
                 b_g64 = sizeof(double) * table_floats(h),
                 b_g32 = sizeof(float) * table_floats(h),
                 b_ptr = kop ? 0 : sizeof(int) * csr_ptr.size(),
                 b_col = sizeof(int) * csr_col.size(),
                 b_ktab = kop ? real_size * kop_entries(d, h->n, b.kop_nt) : 0;
    const size_t o_val = al256(b_pts), o_alpha = o_val + al256(b_val),
                 o_g64 = o_alpha + al256(b_alpha), o_g32 = o_g64 + al256(b_g64),
                 o_ptr = o_g32 + al256(b_g32), o_col = o_ptr + al256(b_ptr),
                 o_ktab = o_col + al256(b_col), n_block = o_ktab + al256(b_ktab);
    bool ok = dalloc(&h->d_block, n_block) &&
              (kop || dalloc((void **)&h->d_W, sizeof(double) * (size_t)h->p * h->n)) &&
              (kop || dalloc((void **)&h->d_beta,
                             sizeof(double) * h->p * (size_t)project_segments(h->n))) &&
              dalloc((void **)&h->d_c, sizeof(double) * (size_t)h->K_it * h->n) &&
              dalloc((void **)&h->d_var, sizeof(double) * (size_t)h->K_it * h->n);
    if (!ok) {
        free_device(h);
        delete h;
        if (alloc_err == hipErrorOutOfMemory)
            return fail(BSDE_ENOMEM, "device allocation failed");
        return fail(BSDE_EDEVICE, std::string("hipMalloc: ") + hipGetErrorString(alloc_err));
    }
    {
        char *b = (char *)h->d_block;
        h->d_pts = (double *)b;
        h->d_vals = (double *)(b + o_val);
        h->d_alpha = (double *)(b + o_alpha);
        h->d_g64 = (double *)(b + o_g64);
        h->d_g32 = (float *)(b + o_g32);
        h->d_rowptr = b_ptr ? (int *)(b + o_ptr) : nullptr;
        h->d_cols = b_ptr ? (int *)(b + o_col) : nullptr;
        h->d_ktab = kop ? (void *)(b + o_ktab) : nullptr;
    }
    // the kernel operator's table in the path precision (bsde_common.h), y = 0
    std::vector<unsigned char> ktab(b_ktab, 0);
    auto set_ktab = [&](size_t e, double v) {
        const float f = (float)v;
        if (real_size == sizeof(float)) std::memcpy(&ktab[e * sizeof(f)], &f, sizeof(f));
        else std::memcpy(&ktab[e * sizeof(v)], &v, sizeof(v));
    };
    for (int i = 0; kop && i < h->n; ++i) {
        double z[kMaxD + 1];
        z[0] = 2.0 * h->pts[(size_t)i * dp] / payoff->T - 1.0;
        for (int j = 0; j < d; ++j)
            z[1 + j] = (h->pts[(size_t)i * dp + 1 + j] - b.mid[j]) * b.scale[j];
        if (b.kop_nt == 0) {
            for (int v = 0; v <= d; ++v) set_ktab((size_t)i * kKernelRow + v, z[v]);
            continue;
        }
        if (i % h->n_spatial == 0) {
            const int a = i / h->n_spatial;
            set_ktab(2 * a, z[0]);
            set_ktab(2 * a + 1, std::exp(-(1.0 - z[0]) * (1.0 - z[0]) * 0.5 / (b.kbw * b.kbw)));
        }
        if (i < h->n_spatial)
            for (int j = 0; j < d; ++j)
                set_ktab(kop_value(d, h->n, b.kop_nt, i) - d + j, z[1 + j]);
    }
    // uploads and the set-up kernels go to a set-up stream of the library
    // (non-blocking: a problem created while another one solves does not
    // wait for it).  The block goes up in one copy from pinned staging
    // memory: points, the channel update's sparse rows and zeros for the
    // starting coefficients and the channel tables.
    hipStream_t us = nullptr;
    size_t pin_cap = 0;
    void *pin = n_block <= kPinnedMax ? pinned_get(n_block, &pin_cap) : nullptr;
    hipError_t e = setup_stream_get(&us);
    if (e == hipSuccess && pin) {
        std::memset(pin, 0, n_block);
        std::memcpy(pin, h->pts.data(), b_pts);
        if (b_val) std::memcpy((char *)pin + o_val, csr_val.data(), b_val);
        if (b_ptr) std::memcpy((char *)pin + o_ptr, csr_ptr.data(), b_ptr);
        if (b_col) std::memcpy((char *)pin + o_col, csr_col.data(), b_col);
        if (b_ktab) std::memcpy((char *)pin + o_ktab, ktab.data(), b_ktab);
        e = hipMemcpyAsync(h->d_block, pin, n_block, hipMemcpyHostToDevice, us);
    } else if (e == hipSuccess) {
        e = hipMemcpyAsync(h->d_pts, h->pts.data(), b_pts, hipMemcpyHostToDevice, us);
        if (e == hipSuccess && b_val)
            e = hipMemcpyAsync(h->d_vals, csr_val.data(), b_val, hipMemcpyHostToDevice, us);
        if (e == hipSuccess)
            e = hipMemsetAsync((char *)h->d_block + o_alpha, 0, o_ptr - o_alpha, us);
        if (e == hipSuccess && b_ptr)
            e = hipMemcpyAsync(h->d_rowptr, csr_ptr.data(), b_ptr, hipMemcpyHostToDevice, us);
        if (e == hipSuccess && b_col)
            e = hipMemcpyAsync(h->d_cols, csr_col.data(), b_col, hipMemcpyHostToDevice, us);
        if (e == hipSuccess && b_ktab)
            e = hipMemcpyAsync(h->d_ktab, ktab.data(), b_ktab, hipMemcpyHostToDevice, us);
    }
    if (e != hipSuccess) {
        if (us) {
            (void)hipStreamSynchronize(us);
            setup_stream_put(us);
        }
        pinned_put(pin, pin_cap);
        free_device(h);
        delete h;
        return fail(BSDE_EDEVICE, std::string("upload: ") + hipGetErrorString(e));
    }
    // pseudo-inverse of the basis matrix of the grid, on the device (it
    // synchronizes the set-up stream: the sparse rows and the points may go
    // out of scope)
    // (the kernel operator fits nothing: only the upload to wait for)
    bsde_status pst = BSDE_OK;
    if (!kop) {
        pst = device_pseudo_inverse(h, us);
    } else {
        const hipError_t se = hipStreamSynchronize(us);
        if (se != hipSuccess)
            pst = fail(BSDE_EDEVICE, std::string("upload: ") + hipGetErrorString(se));
    }
    setup_stream_put(us);
    pinned_put(pin, pin_cap);
    if (pst != BSDE_OK) {
        free_device(h);
        delete h;
        return pst; // the last error is already recorded
    }
    h->alpha_hist.assign((size_t)(h->K_it + 1) * h->p, 0.0);
    {
        std::lock_guard<std::mutex> g(g_tune_mu);
        auto it = g_tuned.find(tune_key(h));
        if (it != g_tuned.end()) {
            h->groups = it->second.first;
            h->ppl = it->second.second;
        }
    }
    // the per-group sum buffer of the tiling the problem starts with, so
    // that solving it allocates nothing more
    int groups0, ppl0;
    const bsde_status tst = prepare_tiling(h, groups0, ppl0);
    if (tst != BSDE_OK) {
        free_device(h);
        delete h;
        return tst;
    }
    *out = h;
    return BSDE_OK;
}

bsde_status bsde_set_tiling(bsde_problem h, int groups_per_point,
                            int paths_per_lane)
{
    if (!h || groups_per_point < 0 || paths_per_lane < 0)
        return fail(BSDE_EINVAL, "bad tiling");
    if ((groups_per_point == 0) != (paths_per_lane == 0))
        return fail(BSDE_EINVAL, "set both tiling values or neither");
    if (groups_per_point > 0 &&
        (long)groups_per_point * paths_per_lane * kBlock < h->M)
        return fail(BSDE_EINVAL, "tiling covers fewer than M paths");
    h->groups = groups_per_point;
    h->ppl = paths_per_lane;
    return BSDE_OK;
}

// Tiling of a solve and the per-group sum buffer it needs (grown from the
// pool unless allow_alloc is false: then a buffer too small is an error).
static bsde_status prepare_tiling(bsde_problem h, int &groups, int &ppl,
                                  bool allow_alloc)
{
    groups = h->groups;
    ppl = h->ppl;
    if (groups == 0) auto_tiling(h->n, h->M, h->N, h->d, groups, ppl);
    const size_t need = (size_t)h->n * groups * 2;
    if (need > h->partial_cap) {
        if (!allow_alloc)
            return fail(BSDE_ESTATE, "the problem's tiling needs a larger per-group sum "
                                     "buffer than it was created with (solve it once with "
                                     "an allocating entry point first)");
        pool_free(h->d_partial);
        h->d_partial = nullptr;
        h->partial_cap = 0;
        HIP_TRY(pool_alloc((void **)&h->d_partial, sizeof(double) * need));
        h->partial_cap = need;
    }
    return BSDE_OK;
}

// the Monte Carlo path kernel of h's operator (least squares: the channel
// table; kernel operator: the point table)
// at the points pts
static hipError_t launch_problem_path(const bsde_problem_s *h, int blocks, hipStream_t s,
                                      const PathParams &prm, const double *pts,
                                      hipEvent_t ev0, hipEvent_t ev1)
{
    const bool fp32 = h->precision == BSDE_FP32_PATHS;
    if (h->kop)
        return launch_kernel_path(h->d, fp32, blocks, s, prm, pts, h->d_ktab,
                                  h->d_partial, ev0, ev1);
    return launch_path(h->d, h->eta, h->q10, fp32, blocks, s, prm, pts,
                       fp32 ? (const void *)h->d_g32 : (const void *)h->d_g64,
                       h->d_partial, ev0, ev1);
}

bsde_status bsde_solve(bsde_problem h, void *hip_stream)
{
    if (!h) return fail(BSDE_EINVAL, "null handle");
    hipStream_t s = (hipStream_t)hip_stream;
    int groups, ppl;
    bsde_status st = prepare_tiling(h, groups, ppl);
    if (st != BSDE_OK) return st;
    const bool fp32 = h->precision == BSDE_FP32_PATHS;
    const int iters = h->K_it - h->k_done;
    // events: start, end, and per iteration (timing level 1) the start and
    // end of the path-kernel dispatch (taken by the dispatch itself, no
    // marker packets), (level 2) also after the reduction, the projection
    // and the channel update
    const int lvl = h->timing;
    const int per = lvl >= 2 ? 5 : (lvl == 1 ? 2 : 0);
    std::vector<hipEvent_t> ev(2 + (size_t)per * iters);
    for (auto &x : ev) HIP_TRY(event_get(&x));
    struct Release {
        std::vector<hipEvent_t> &v;
        ~Release() { for (auto &x : v) event_put(x); }
    } release_events{ev};
    RedrawWork redraw(h, s);
    HIP_TRY(hipEventRecord(ev[0], s));
    // channel table of the starting coefficients (the kernel operator's
    // table already holds the current point values)
    if (!h->kop)
        HIP_TRY(launch_channels(h->p, h->n_live, s, h->d_alpha + (size_t)h->k_done * h->p,
                                h->d_rowptr, h->d_cols, h->d_vals, h->d_g64, h->d_g32));
    for (int it = 0; it < iters; ++it) {
        const int k = h->k_done + it;
        hipEvent_t *e = per ? &ev[2 + (size_t)per * it] : nullptr;
        // Algorithm 1: new points for this iteration, and the pseudo-inverse
        // of their basis matrix
        auto draw = [&](int kk) {
            const hipError_t re = redraw.draw(kk, ev[0]);
            if (re == hipSuccess) return BSDE_OK;
            return fail(re == hipErrorOutOfMemory ? BSDE_ENOMEM : BSDE_EDEVICE,
                        std::string("redrawn points: ") + hipGetErrorString(re));
        };
        RedrawWork::Set set{h->d_pts, h->d_W};
        if (h->redraw) {
            if (!redraw.drawn(k) && h->pts_k != k && (st = draw(k)) != BSDE_OK) return st;
            if (redraw.failed()) break;
            HIP_TRY(redraw.begin(k, set));
        }
        PathParams prm = h->base;
        prm.k = (uint32_t)k;
        prm.groups = groups;
        prm.paths_per_lane = ppl;
        prm.n = h->n;
        HIP_TRY(launch_problem_path(h, h->n * groups, s, prm, set.pts, e ? e[0] : nullptr,
                                    e ? e[1] : nullptr));
        if (h->kop) {
            // c^k, then y^k = u^k(points) + c^k with u^k = h[y^{k-1}]
            // (alpha row k; row 0 = 0 is u^0 = 0) into row k + 1 and the table
            double *ck = h->d_c + (size_t)k * h->n;
            HIP_TRY(launch_finalize(h->d_partial, h->n, groups, h->M, kBlock * ppl, ck,
                                    h->d_var + (size_t)k * h->n, s));
            if (per == 5) HIP_TRY(hipEventRecord(e[2], s));
            HIP_TRY(launch_kernel_update(prm, h->d, h->d_pts,
                                         k ? h->d_alpha + (size_t)k * h->p : nullptr, ck,
                                         h->d_alpha + (size_t)(k + 1) * h->p, h->d_ktab,
                                         fp32 ? 1 : 0, s));
            if (per == 5) {
                HIP_TRY(hipEventRecord(e[3], s));
                HIP_TRY(hipEventRecord(e[4], s));
            }
            continue;
        }
        HIP_TRY(launch_update(h->n, groups, h->M, kBlock * ppl, h->p, h->n_live, s,
                              h->d_partial, h->d_c + (size_t)k * h->n,
                              h->d_var + (size_t)k * h->n, set.W, h->d_beta,
                              h->d_alpha + (size_t)k * h->p,
                              h->d_alpha + (size_t)(k + 1) * h->p, h->d_rowptr, h->d_cols,
                              h->d_vals, h->d_g64, h->d_g32,
                              per == 5 ? e + 2 : nullptr)); // records e[2..4]
        if (h->redraw) {
            const bool ahead = it + 1 < iters && redraw.ahead(ev[0]);
            HIP_TRY(redraw.end(k));
            if (ahead && (st = draw(k + 1)) != BSDE_OK) return st;
        }
    }
    if (h->redraw) HIP_TRY(redraw.finish());
    HIP_TRY(hipEventRecord(ev[1], s));
    // the coefficients come back with the end of the solve, one wait for both
    const size_t alpha_bytes = sizeof(double) * h->alpha_hist.size();
    PinnedBuffer alpha(alpha_bytes);
    HIP_TRY(hipMemcpyAsync(alpha.get() ? alpha.get() : (void *)h->alpha_hist.data(), h->d_alpha,
                           alpha_bytes, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (!redraw.full_rank()) {
        redraw.restore();
        return fail(BSDE_ERANK, kRankMessage);
    }
    double t_path = 0, t_fin = 0, t_proj = 0, t_chan = 0;
    for (int it = 0; it < iters && per; ++it) {
        hipEvent_t *e = &ev[2 + (size_t)per * it];
        float ms;
        hipEventElapsedTime(&ms, e[0], e[1]); t_path += ms;
        if (per == 5) {
            hipEventElapsedTime(&ms, e[1], e[2]); t_fin += ms;
            hipEventElapsedTime(&ms, e[2], e[3]); t_proj += ms;
            hipEventElapsedTime(&ms, e[3], e[4]); t_chan += ms;
        } else {
            // the rest of the iteration: up to the next path kernel (or
            // the end of the solve)
            hipEvent_t next = it + 1 < iters ? ev[2 + (size_t)per * (it + 1)] : ev[1];
            hipEventElapsedTime(&ms, e[1], next); t_fin += ms;
        }
    }
    float tot;
    hipEventElapsedTime(&tot, ev[0], ev[1]);
    if (alpha.get()) std::memcpy(h->alpha_hist.data(), alpha.get(), alpha_bytes);
    if (iters > 0) {
        h->timings[0] = t_path / iters;
        h->timings[1] = t_fin / iters;
        h->timings[2] = t_proj / iters;
        h->timings[3] = t_chan / iters;
        h->timings[4] = tot;
    }
    h->k_done = h->K_it;
    h->have_alpha = true;
    return BSDE_OK;
}

} // extern "C"

// ---------------------------------------------------------------------------
// Batched solve: all remaining iterations of many problems.  Per iteration
// step and kernel signature (d, eta, precision, volatility kind) one
// persistent launch drains the tiles of every active problem of that
// signature; one launch each then reduces, projects and updates all active
// problems.  With BSDE_BATCH_GRAPH the whole schedule is captured once as a
// hipGraph and replayed.
// ---------------------------------------------------------------------------
namespace {
struct Sig {
    int d, eta, q10;
    bool fp32;
    int vol;
    bool operator<(const Sig &o) const
    {
        return std::tie(d, eta, q10, fp32, vol) < std::tie(o.d, o.eta, o.q10, o.fp32, o.vol);
    }
};

int num_cus()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount,
                                  dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

BatchUpdateDesc update_desc(bsde_problem h, int k, int groups, int ppl, bool advance)
{
    BatchUpdateDesc u{};
    u.partial = h->d_partial;
    u.n = h->n;
    u.groups = groups;
    u.ppg = kBlock * ppl;
    u.M = h->M;
    u.p = h->p;
    u.nnz = h->n_live;
    u.c = h->d_c + (size_t)std::min(k, h->K_it - 1) * h->n;
    u.var = h->d_var + (size_t)std::min(k, h->K_it - 1) * h->n;
    u.W = h->d_W;
    u.beta = h->d_beta;
    u.alpha_in = h->d_alpha + (size_t)k * h->p;
    u.alpha_out = advance ? h->d_alpha + (size_t)(k + 1) * h->p : nullptr;
    u.rowptr = h->d_rowptr;
    u.cols = h->d_cols;
    u.vals = h->d_vals;
    u.g64 = h->d_g64;
    u.g32 = h->d_g32;
    return u;
}
} // namespace

// Runs `steps` iterations (at most the remaining ones) of every problem.
// Copies the coefficient histories back when copy_back is set.
bsde_status bsde::run_batch(bsde_problem *probs, int count, hipStream_t s,
                            int steps, bool graph, bool copy_back, double *ms,
                            const int *steps_each, void *workspace,
                            size_t workspace_bytes, bool parallel_branches,
                            int cu_reserve)
{
    std::vector<int> G(count), PPL(count), R(count);
    int S = 0;
    for (int q = 0; q < count; ++q) {
        bsde_status st = prepare_tiling(probs[q], G[q], PPL[q], workspace == nullptr);
        if (st != BSDE_OK) return st;
        // iterations problem q runs in this call
        R[q] = std::max(0, std::min(steps_each ? steps_each[q] : steps,
                                    probs[q]->K_it - probs[q]->k_done));
        S = std::max(S, R[q]);
    }
    std::map<Sig, std::vector<int>> sigs;
    for (int q = 0; q < count; ++q) {
        bsde_problem h = probs[q];
        sigs[{h->d, h->eta, h->q10, h->precision == BSDE_FP32_PATHS,
              h->base.vol_kind}].push_back(q);
    }
    // host-side descriptor tables, laid out in one byte buffer
    std::vector<char> blob;
    auto put = [&](const void *src, size_t bytes) {
        size_t off = (blob.size() + 255) & ~(size_t)255;
        blob.resize(off + bytes);
        std::memcpy(blob.data() + off, src, bytes);
        return off;
    };
    struct PathLaunch { Sig sig; size_t desc_off, begin_off; int nprob; long long tiles; int counter; };
    struct StepPlan { std::vector<PathLaunch> paths; size_t upd_off; int nact, max_n, max_p, max_cb; };
    std::vector<StepPlan> plan(S);
    int n_counters = 0;
    int max_cb_all = 0; // workgroups of the channel update (256 entries each)
    for (int step = 0; step < S; ++step) {
        std::vector<BatchUpdateDesc> upd;
        int max_n = 0, max_p = 0, max_cb = 0;
        for (auto &kv : sigs) {
            std::vector<int> act;
            for (int q : kv.second)
                if (step < R[q]) act.push_back(q);
            if (act.empty()) continue;
            // heaviest tiles first (paths per lane x Euler steps)
            std::stable_sort(act.begin(), act.end(), [&](int a, int b) {
                return (long long)PPL[a] * probs[a]->N > (long long)PPL[b] * probs[b]->N;
            });
            std::vector<BatchTileDesc> td;
            std::vector<long long> begin(1, 0);
            for (int q : act) {
                bsde_problem h = probs[q];
                BatchTileDesc t{};
                t.prm = h->base;
                t.prm.k = (uint32_t)(h->k_done + step);
                t.prm.groups = G[q];
                t.prm.paths_per_lane = PPL[q];
                t.prm.n = h->n;
                t.pts = h->d_pts;
                t.gamma = kv.first.fp32 ? (const void *)h->d_g32 : (const void *)h->d_g64;
                t.partial = h->d_partial;
                td.push_back(t);
                begin.push_back(begin.back() + (long long)h->n * G[q]);
                upd.push_back(update_desc(h, h->k_done + step, G[q], PPL[q], true));
                max_n = std::max(max_n, h->n);
                max_p = std::max(max_p, h->p);
                max_cb = std::max(max_cb, (h->n_live + 255) / 256);
            }
            PathLaunch pl{kv.first, put(td.data(), sizeof(BatchTileDesc) * td.size()),
                          put(begin.data(), sizeof(long long) * begin.size()),
                          (int)act.size(), begin.back(), n_counters++};
            plan[step].paths.push_back(pl);
        }
        plan[step].upd_off = put(upd.data(), sizeof(BatchUpdateDesc) * upd.size());
        plan[step].nact = (int)upd.size();
        plan[step].max_n = max_n;
        plan[step].max_p = max_p;
        plan[step].max_cb = max_cb;
        max_cb_all = std::max(max_cb_all, max_cb);
    }
    std::vector<BatchUpdateDesc> init;
    for (int q = 0; q < count; ++q) {
        init.push_back(update_desc(probs[q], probs[q]->k_done, G[q], PPL[q], false));
        max_cb_all = std::max(max_cb_all, (probs[q]->n_live + 255) / 256);
    }
    const size_t init_off = put(init.data(), sizeof(BatchUpdateDesc) * init.size());
    const size_t ctr_off = (blob.size() + 255) & ~(size_t)255;
    blob.resize(ctr_off + sizeof(unsigned int) * std::max(1, n_counters), 0);

    // the descriptor tables and tile counters: from the pool, or in the
    // caller's workspace
    char *dblob = nullptr;
    if (workspace) {
        if (blob.size() > workspace_bytes)
            return fail(BSDE_EINVAL, "the batch's descriptor tables need " +
                                         std::to_string(blob.size()) +
                                         " bytes, more than the workspace of " +
                                         std::to_string(workspace_bytes));
        dblob = (char *)workspace;
    } else {
        HIP_TRY(pool_alloc((void **)&dblob, blob.size()));
    }
    struct Release {
        char *p;
        ~Release() { pool_free(p); }
    } release{workspace ? nullptr : dblob};
    HIP_TRY(hipMemcpyAsync(dblob, blob.data(), blob.size(), hipMemcpyHostToDevice, s));
    unsigned int *counters = (unsigned int *)(dblob + ctr_off);

    // Launches of different kernel signatures in one step run as parallel
    // branches: the first on s, the others on the library's side streams of
    // this device (forked from s and joined back before the step's update),
    // so that the tiles of one signature fill the tail of another's launch.
    // The no-allocation form (and a caller that asks) keeps everything on s.
    const bool parallel = workspace == nullptr && parallel_branches;
    SideStreams *side = nullptr;
    std::unique_lock<std::mutex> side_lock; // held until the batch is done
    if (parallel) {
        bool fork_any = false;
        for (int step = 0; step < S; ++step) fork_any |= plan[step].paths.size() > 1;
        if (fork_any) {
            HIP_TRY(side_streams(&side));
            side_lock = std::unique_lock<std::mutex>(side->mu);
        }
    }
    auto enqueue = [&]() -> hipError_t {
        hipError_t e = launch_reset_counters(counters, std::max(1, n_counters), s);
        if (e != hipSuccess) return e;
        e = launch_batch_channels(count, max_cb_all, s,
                                  (const BatchUpdateDesc *)(dblob + init_off));
        if (e != hipSuccess) return e;
        for (int step = 0; step < S; ++step) {
            const int nl = (int)plan[step].paths.size();
            const int nside = side ? std::min(nl - 1, SideStreams::kCount) : 0;
            if (nside > 0) {
                e = hipEventRecord(side->fork, s);
                for (int k = 0; k < nside && e == hipSuccess; ++k)
                    e = hipStreamWaitEvent(side->s[k], side->fork, 0);
                if (e != hipSuccess) return e;
            }
            for (int j = 0; j < nl; ++j) {
                const PathLaunch &pl = plan[step].paths[j];
                hipStream_t ls = (j == 0 || nside == 0) ? s : side->s[(j - 1) % nside];
                const int occ = std::max(1, batch_occupancy(pl.sig.d, pl.sig.eta, pl.sig.q10,
                                                            pl.sig.fp32, pl.sig.vol));
                const long long cap = (long long)occ * std::max(1, num_cus() - cu_reserve);
                const int blocks = (int)std::max(1LL, std::min(pl.tiles, cap));
                e = launch_batch(pl.sig.d, pl.sig.eta, pl.sig.q10, pl.sig.fp32, pl.sig.vol, blocks, ls,
                                 (const BatchTileDesc *)(dblob + pl.desc_off), pl.nprob,
                                 (const long long *)(dblob + pl.begin_off),
                                 counters + pl.counter);
                if (e != hipSuccess) return e;
            }
            for (int k = 0; k < nside; ++k) {
                e = hipEventRecord(side->join[k], side->s[k]);
                if (e == hipSuccess) e = hipStreamWaitEvent(s, side->join[k], 0);
                if (e != hipSuccess) return e;
            }
            e = launch_batch_update(plan[step].nact, plan[step].max_n, plan[step].max_p,
                                    plan[step].max_cb, s,
                                    (const BatchUpdateDesc *)(dblob + plan[step].upd_off));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };

    // timing events only when the time is asked for
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ms) {
        HIP_TRY(event_get(&e0));
        HIP_TRY(event_get(&e1));
        HIP_TRY(hipEventRecord(e0, s));
    }
    if (graph) {
        // The instantiated graph of the last captured batch on this device
        // is kept with its descriptor tables; a batch whose tables and
        // launch plan are byte for byte the same (the same problems, from
        // the same iteration) replays it instead of capturing again.  The
        // tables hold every address and parameter the kernels read, so
        // equal tables mean the same work.
        std::vector<long long> launches;
        for (int step = 0; step < S; ++step) {
            for (const PathLaunch &pl : plan[step].paths)
                launches.insert(launches.end(), {pl.sig.d, pl.sig.eta, pl.sig.q10, pl.sig.fp32,
                                                 pl.sig.vol, (long long)pl.desc_off,
                                                 (long long)pl.begin_off, pl.nprob, pl.tiles,
                                                 pl.counter});
            launches.insert(launches.end(), {-1, (long long)plan[step].upd_off, plan[step].nact,
                                             plan[step].max_n, plan[step].max_p,
                                             plan[step].max_cb});
        }
        launches.insert(launches.end(), {count, max_cb_all, (long long)init_off, n_counters,
                                         (long long)(side != nullptr)});
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev));
        std::lock_guard<std::mutex> gl(g_graph_mu);
        GraphCache &gc = g_graph_cache[dev];
        const bool hit = gc.exec && gc.blob == blob && gc.launches == launches;
        if (!hit) {
            gc.release();
            // the cached graph owns its descriptor tables: move them out of
            // this call's release
            gc.dblob = dblob;
            release.p = nullptr;
            hipGraph_t g = nullptr;
            HIP_TRY(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
            hipError_t le = enqueue();
            hipError_t ce = hipStreamEndCapture(s, &g);
            if (le != hipSuccess || ce != hipSuccess) {
                if (g) (void)hipGraphDestroy(g);
                gc.release();
                return fail(BSDE_EDEVICE, std::string("graph capture: ") +
                                              hipGetErrorString(le != hipSuccess ? le : ce));
            }
            hipError_t ie = hipGraphInstantiate(&gc.exec, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            if (ie != hipSuccess) {
                gc.exec = nullptr;
                gc.release();
                return fail(BSDE_EDEVICE, std::string("graph instantiate: ") +
                                              hipGetErrorString(ie));
            }
            gc.blob = blob;
            gc.launches = launches;
        }
        hipError_t ie = hipGraphLaunch(gc.exec, s);
        if (ie == hipSuccess) ie = hipStreamSynchronize(s);
        if (ie != hipSuccess) {
            gc.release();
            return fail(BSDE_EDEVICE, std::string("graph launch: ") + hipGetErrorString(ie));
        }
    } else {
        HIP_TRY(enqueue());
    }
    if (ms) {
        HIP_TRY(hipEventRecord(e1, s));
        HIP_TRY(hipEventSynchronize(e1));
        float t = 0.f;
        (void)hipEventElapsedTime(&t, e0, e1);
        event_put(e0);
        event_put(e1);
        *ms = t;
    } else {
        HIP_TRY(hipStreamSynchronize(s));
    }
    for (int q = 0; q < count; ++q) {
        bsde_problem h = probs[q];
        h->k_done += R[q];
        h->have_alpha = true;
        if (copy_back) {
            HIP_TRY(hipMemcpyAsync(h->alpha_hist.data(), h->d_alpha,
                                   sizeof(double) * h->alpha_hist.size(),
                                   hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
        }
    }
    return BSDE_OK;
}

bsde_status bsde::fetch_coefficients(bsde_problem h)
{
    HIP_TRY(hipMemcpy(h->alpha_hist.data(), h->d_alpha,
                      sizeof(double) * h->alpha_hist.size(), hipMemcpyDeviceToHost));
    return BSDE_OK;
}

size_t bsde::problem_device_bytes(int d, const bsde_grid *grid, int M, int N, int K_it)
{
    // (what bsde_create_problem refuses takes no memory)
    if (d < 1 || d > kMaxD || !grid || M < 1 || N < 1 || K_it < 1) return 0;
    const int p = index_table(d, grid->eta, kernel_q10(d, grid->eta, grid->q), nullptr, 0);
    if (p == 0) return 0;
    int ns = 0;
    const size_t n = (size_t)grid_points(d, grid, &ns);
    if (n == 0) return 0;
    const size_t C = (size_t)num_channels(d);
    int groups, ppl;
    auto_tiling((int)n, M, N, d, groups, ppl);
    // the block of points, the channel update's sparse rows, coefficients
    // and tables (one allocation, 256-byte aligned parts), then the separate
    // buffers; at most p C table entries and 16 p C non-zeros of the update in
    // all (a row of the channels has at most 10, of a mixed second derivative at
    // eta = 8: one per pair of odd degree steps k1 + k2 <= eta; one of the cubic
    // form up to 36, and the form's rows are less than a fifth of p C)
    auto al256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t entries = table_entries(p, (int)C), nonzeros = 16 * entries;
    const size_t block = al256(n * (d + 1) * 8) + al256(nonzeros * 8) +
                         al256((size_t)(K_it + 1) * p * 8) + al256(entries * 8) +
                         al256(entries * 4) + al256((entries + 1) * 4) +
                         al256(nonzeros * 4);
    const size_t sizes[] = {block, (size_t)p * n * 8, (size_t)p * 8 * project_segments((int)n),
                            (size_t)K_it * n * 8,
                            (size_t)K_it * n * 8,
                            n * groups * 16};
    size_t total = 0;
    for (size_t b : sizes) total += size_class(b == 0 ? 8 : b);
    // transient set-up buffers (PseudoInverse): two point matrices, the Gram
    // partials, the p x p matrices and the small inputs
    int ld, rpc, chunks;
    const size_t pap = (size_t)pad16(p);
    setup_shape((int)n, (int)pap, ld, rpc, chunks);
    total += 2 * size_class((size_t)ld * pap * 8) + size_class((size_t)chunks * pap * pap * 8) +
             size_class((3 * pap * pap + factor_workspace((int)pap)) * 8) +
             size_class((size_t)p * (d + 1 + sizeof(int)) + 1024);
    return total;
}

extern "C" {

bsde_status bsde_solve_batch(bsde_problem *problems, int count,
                                        void *hip_stream, int flags, double *ms)
{
    if (!problems || count < 1) return fail(BSDE_EINVAL, "no problems");
    for (int q = 0; q < count; ++q) {
        if (!problems[q]) return fail(BSDE_EINVAL, "null handle in batch");
        for (int r = 0; r < q; ++r)
            if (problems[r] == problems[q]) return fail(BSDE_EINVAL, "duplicate handle in batch");
        if (problems[q]->redraw)
            return fail(BSDE_EUNSUPPORTED, "points redrawn every iteration: use bsde_solve");
        if (problems[q]->kop)
            return fail(BSDE_EUNSUPPORTED, "the kernel operator: use bsde_solve");
    }
    hipStream_t s = (hipStream_t)hip_stream;
    hipStream_t own = nullptr;
    const bool graph = (flags & BSDE_BATCH_GRAPH) != 0;
    if (graph && !s) { // capture needs a stream other than the null stream
        HIP_TRY(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
        s = own;
    }
    bsde_status st = run_batch(problems, count, s, 1 << 30, graph, true, ms);
    if (own) (void)hipStreamDestroy(own);
    return st;
}

} // extern "C"

// ---------------------------------------------------------------------------
// The no-allocation batched solve.  Its descriptor tables and tile counters
// live in this fixed array, one copy per device, held until the process
// ends.  In host code the array's name is not a device address: the
// address of the current device's copy comes from hipGetSymbolAddress on
// the first call on that device and is used everywhere after.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t kNoAllocBytes = size_t(4) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];
std::mutex g_scratch_mu;            // one call per device at a time
std::map<int, void *> g_scratch;    // device -> address of its copy
} // namespace

extern "C" {

bsde_status bsde_solve_batch_noalloc(bsde_problem *problems, int count,
                                     void *hip_stream)
{
    if (!problems || count < 1) return fail(BSDE_EINVAL, "no problems");
    for (int q = 0; q < count; ++q) {
        if (!problems[q]) return fail(BSDE_EINVAL, "null handle in batch");
        for (int r = 0; r < q; ++r)
            if (problems[r] == problems[q]) return fail(BSDE_EINVAL, "duplicate handle in batch");
        if (problems[q]->redraw)
            return fail(BSDE_EUNSUPPORTED, "points redrawn every iteration: use bsde_solve");
        if (problems[q]->kop)
            return fail(BSDE_EUNSUPPORTED, "the kernel operator: use bsde_solve");
    }
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> g(g_scratch_mu);
    auto it = g_scratch.find(dev);
    if (it == g_scratch.end()) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(BSDE_EDEVICE, std::string("workspace address: ") + hipGetErrorString(e));
        it = g_scratch.emplace(dev, ptr).first;
    }
    return run_batch(problems, count, (hipStream_t)hip_stream, 1 << 30, false, true,
                     nullptr, nullptr, it->second, kNoAllocBytes);
}

bsde_status bsde_autotune(bsde_problem h, void *hip_stream, int *groups_out,
                          int *ppl_out, double *ms_out)
{
    if (!h) return fail(BSDE_EINVAL, "null handle");
    hipStream_t s = (hipStream_t)hip_stream;
    // candidates: paths per lane in powers of two, groups to cover M
    std::vector<std::pair<int, int>> cand;
    for (int ppl = 1; ppl <= 64; ppl *= 2) {
        const int groups = (h->M + kBlock * ppl - 1) / (kBlock * ppl);
        if (groups < 1) continue;
        if (!cand.empty() && cand.back().first == groups) continue;
        cand.push_back({groups, ppl});
        if (groups == 1) break;
    }
    size_t need = 0;
    for (auto &c : cand) need = std::max(need, (size_t)h->n * c.first * 2);
    if (need > h->partial_cap) {
        pool_free(h->d_partial);
        h->d_partial = nullptr;
        h->partial_cap = 0;
        HIP_TRY(pool_alloc((void **)&h->d_partial, sizeof(double) * need));
        h->partial_cap = need;
    }
    const int k = std::min(h->k_done, h->K_it - 1);
    if (!h->kop)
        HIP_TRY(launch_channels(h->p, h->n_live, s, h->d_alpha + (size_t)h->k_done * h->p,
                                h->d_rowptr, h->d_cols, h->d_vals, h->d_g64, h->d_g32));
    hipEvent_t e0, e1;
    HIP_TRY(event_get(&e0));
    HIP_TRY(event_get(&e1));
    double best = 1e300;
    std::pair<int, int> pick = cand.front();
    for (auto &c : cand) {
        PathParams prm = h->base;
        prm.k = (uint32_t)k;
        prm.groups = c.first;
        prm.paths_per_lane = c.second;
        prm.n = h->n;
        double t_min = 1e300;
        for (int rep = 0; rep < 5; ++rep) { // first launch warms up
            HIP_TRY(launch_problem_path(h, h->n * c.first, s, prm, h->d_pts, e0, e1));
            HIP_TRY(hipEventSynchronize(e1));
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            if (rep > 0) t_min = std::min(t_min, (double)ms);
        }
        // a later candidate (fewer workgroups per point) must win by more
        // than timing noise, so that repeated tunings agree
        if (t_min < 0.98 * best) {
            best = t_min;
            pick = c;
        }
    }
    event_put(e0);
    event_put(e1);
    h->groups = pick.first;
    h->ppl = pick.second;
    {
        std::lock_guard<std::mutex> g(g_tune_mu);
        g_tuned[tune_key(h)] = pick;
    }
    if (groups_out) *groups_out = pick.first;
    if (ppl_out) *ppl_out = pick.second;
    if (ms_out) *ms_out = best;
    return BSDE_OK;
}

// Architecture name of the current device ("gfx950"), the key under which
// recorded tilings are saved: a tiling measured on one architecture says
// nothing about another.
static bsde_status device_arch(std::string &arch)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch.resize(colon);
    if (arch.empty()) return fail(BSDE_EDEVICE, "device reports no architecture name");
    return BSDE_OK;
}

bsde_status bsde_autotune_save(const char *path, int *count)
{
    if (!path) return fail(BSDE_EINVAL, "null path");
    std::string arch;
    const bsde_status st = device_arch(arch);
    if (st != BSDE_OK) return st;
    std::vector<std::pair<TuneKey, std::pair<int, int>>> rows;
    {
        std::lock_guard<std::mutex> g(g_tune_mu);
        rows.assign(g_tuned.begin(), g_tuned.end());
    }
    FILE *f = std::fopen(path, "w");
    if (!f) return fail(BSDE_EINVAL, std::string("cannot write ") + path);
    std::fprintf(f, "# bsde path tilings: arch d eta q10 precision vol M N size_class "
                    "groups_per_point paths_per_lane\n");
    for (const auto &r : rows) {
        const TuneKey &k = r.first;
        std::fprintf(f, "%s %d %d %d %d %d %d %d %d %d %d\n", arch.c_str(), k.d, k.eta,
                     k.q10, k.prec, k.vol, k.M, k.N, k.nclass, r.second.first,
                     r.second.second);
    }
    const bool ok = std::fclose(f) == 0;
    if (!ok) return fail(BSDE_EINVAL, std::string("cannot write ") + path);
    if (count) *count = (int)rows.size();
    return BSDE_OK;
}

bsde_status bsde_autotune_load(const char *path, int *count)
{
    if (!path) return fail(BSDE_EINVAL, "null path");
    std::string arch;
    const bsde_status st = device_arch(arch);
    if (st != BSDE_OK) return st;
    FILE *f = std::fopen(path, "r");
    if (!f) return fail(BSDE_EINVAL, std::string("cannot read ") + path);
    // parse every line first: a malformed file changes nothing
    std::vector<std::pair<TuneKey, std::pair<int, int>>> rows;
    char line[512];
    int lineno = 0;
    bool bad = false;
    while (std::fgets(line, sizeof line, f)) {
        ++lineno;
        const char *q = line;
        while (*q == ' ' || *q == '\t') ++q;
        if (*q == '#' || *q == '\n' || *q == '\0') continue;
        char a[64];
        TuneKey k;
        int groups = 0, ppl = 0;
        if (std::sscanf(q, "%63s %d %d %d %d %d %d %d %d %d %d", a, &k.d, &k.eta, &k.q10,
                        &k.prec, &k.vol, &k.M, &k.N, &k.nclass, &groups, &ppl) != 11 ||
            groups < 1 || ppl < 1 || k.M < 1 ||
            (long long)groups * ppl * kBlock < (long long)k.M) {
            bad = true;
            break;
        }
        if (arch == a) rows.push_back({k, {groups, ppl}});
    }
    std::fclose(f);
    if (bad)
        return fail(BSDE_EINVAL, std::string(path) + ": malformed tiling record on line " +
                                     std::to_string(lineno));
    {
        std::lock_guard<std::mutex> g(g_tune_mu);
        for (const auto &r : rows) g_tuned[r.first] = r.second;
    }
    if (count) *count = (int)rows.size();
    return BSDE_OK;
}

bsde_status bsde_get_tiling(bsde_problem h, int *groups_per_point, int *paths_per_lane)
{
    if (!h || !groups_per_point || !paths_per_lane) return fail(BSDE_EINVAL, "null argument");
    *groups_per_point = h->groups;
    *paths_per_lane = h->ppl;
    return BSDE_OK;
}

bsde_status bsde_set_timing(bsde_problem h, int level)
{
    if (!h) return fail(BSDE_EINVAL, "null handle");
    if (level < 0 || level > 2) return fail(BSDE_EINVAL, "timing level must be 0, 1 or 2");
    h->timing = level;
    return BSDE_OK;
}

bsde_status bsde_last_timings(bsde_problem h, double *ms5)
{
    if (!h || !ms5) return fail(BSDE_EINVAL, "null argument");
    for (int i = 0; i < 5; ++i) ms5[i] = h->timings[i];
    return BSDE_OK;
}

bsde_status bsde_problem_sizes(bsde_problem h, int *n, int *p, int *C)
{
    if (!h) return fail(BSDE_EINVAL, "null handle");
    if (n) *n = h->n;
    if (p) *p = h->p;
    if (C) *C = h->C;
    return BSDE_OK;
}

bsde_status bsde_get_points(bsde_problem h, double *pts)
{
    if (!h || !pts) return fail(BSDE_EINVAL, "null argument");
    std::memcpy(pts, h->pts.data(), sizeof(double) * h->pts.size());
    return BSDE_OK;
}

bsde_status bsde_get_coefficients(bsde_problem h, int k, double *alpha,
                                  int *k_done)
{
    if (!h || !alpha) return fail(BSDE_EINVAL, "null argument");
    if (k < 0) k = h->k_done;
    if (k > h->k_done) return fail(BSDE_ESTATE, "iteration not computed");
    std::memcpy(alpha, &h->alpha_hist[(size_t)k * h->p], sizeof(double) * h->p);
    if (k_done) *k_done = h->k_done;
    return BSDE_OK;
}

// on_device: they are there already
static bsde_status store_alpha(bsde_problem h, const double *alpha, int k_done,
                               bool on_device = false)
{
    for (int l = 0; l < h->p; ++l)
        h->alpha_hist[(size_t)k_done * h->p + l] = h->active[l] ? alpha[l] : 0.0;
    if (!on_device)
        HIP_TRY(hipMemcpy(h->d_alpha + (size_t)k_done * h->p,
                          &h->alpha_hist[(size_t)k_done * h->p],
                          sizeof(double) * h->p, hipMemcpyHostToDevice));
    h->k_done = k_done;
    h->have_alpha = true;
    return BSDE_OK;
}

bsde_status bsde_set_coefficients(bsde_problem h, const double *alpha,
                                  int k_done)
{
    if (!h || !alpha) return fail(BSDE_EINVAL, "null argument");
    if (k_done < 0 || k_done > h->K_it) return fail(BSDE_EINVAL, "bad k_done");
    if (h->kop) return fail(BSDE_EUNSUPPORTED, "the kernel operator runs whole solves");
    return store_alpha(h, alpha, k_done);
}

bsde_status bsde_fit_values(bsde_problem h, const double *y, int k_done)
{
    if (!h || !y) return fail(BSDE_EINVAL, "null argument");
    if (k_done < 0 || k_done > h->K_it) return fail(BSDE_EINVAL, "bad k_done");
    if (h->kop) return fail(BSDE_EUNSUPPORTED, "the kernel operator fits no basis");
    if (h->redraw && h->pts_k < 0) {
        // a solve ended in a device error, and W may not be that of the points
        hipStream_t s = nullptr;
        HIP_TRY(setup_stream_get(&s));
        hipError_t e = hipMemcpyAsync(h->d_pts, h->pts.data(), sizeof(double) * h->pts.size(),
                                      hipMemcpyHostToDevice, s);
        const bsde_status st = device_pseudo_inverse(h, s);
        setup_stream_put(s);
        HIP_TRY(e);
        if (st != BSDE_OK) return st;
    }
    // alpha = R^{-1} Q' y = W y on the device, without memory of its own: y goes to
    // the paths' moments, which every iteration writes anew (n = 10 933, p = 56:
    // 41 us; W copied back and multiplied on the host: 590).  Up to 16 384 entries
    // of W the kernel takes y from pinned memory and leaves its sums there, with
    // one wait and no copy (n = 9, p = 6: 19 us, 23 on the host; n = 512, p = 15: 22
    // and 35, and 41 with the copies).
    const int segs = project_segments(h->n);
    const size_t y_bytes = sizeof(double) * (size_t)h->n;
    std::vector<double> a((size_t)segs * h->p, 0.0);
    const size_t a_bytes = sizeof(double) * a.size();
    if (h->partial_cap < (size_t)h->n) {
        int groups, ppl;
        const bsde_status st = prepare_tiling(h, groups, ppl);
        if (st != BSDE_OK) return st;
    }
    PinnedBuffer pin(y_bytes + a_bytes);
    double *py = (double *)pin.get(), *pa = py ? py + h->n : nullptr;
    const bool direct = py && segs == 1 && (size_t)h->n * h->p <= 16384;
    // (with every function active the sums are the coefficients)
    const bool in_place = direct && h->act.size() == (size_t)h->p;
    if (py) std::memcpy(py, y, y_bytes);
    hipStream_t us = nullptr;
    hipError_t e = setup_stream_get(&us);
    if (e == hipSuccess && !direct)
        e = hipMemcpyAsync(h->d_partial, py ? py : y, y_bytes, hipMemcpyHostToDevice, us);
    if (e == hipSuccess)
        e = launch_project(h->d_W, direct ? py : h->d_partial, h->n, h->p, direct ? pa : h->d_beta,
                           us);
    if (e == hipSuccess && in_place)
        e = launch_project(h->d_W, py, h->n, h->p, h->d_alpha + (size_t)k_done * h->p, us);
    if (e == hipSuccess && !direct)
        e = hipMemcpyAsync(pa ? pa : a.data(), h->d_beta, a_bytes, hipMemcpyDeviceToHost, us);
    if (us) {
        const hipError_t se = hipStreamSynchronize(us);
        if (e == hipSuccess) e = se;
        setup_stream_put(us);
    }
    if (e != hipSuccess)
        return fail(BSDE_EDEVICE, std::string("fit: ") + hipGetErrorString(e));
    if (pa) std::memcpy(a.data(), pa, a_bytes);
    for (int q = 1; q < segs; ++q)
        for (int l = 0; l < h->p; ++l) a[l] += a[(size_t)q * h->p + l];
    return store_alpha(h, a.data(), k_done, in_place);
}

bsde_status bsde_get_corrections(bsde_problem h, int k, double *c, double *var)
{
    if (!h || !c) return fail(BSDE_EINVAL, "null argument");
    if (k < 0 || k >= h->k_done) return fail(BSDE_ESTATE, "iteration not computed");
    HIP_TRY(hipMemcpy(c, h->d_c + (size_t)k * h->n, sizeof(double) * h->n, hipMemcpyDeviceToHost));
    if (var)
        HIP_TRY(hipMemcpy(var, h->d_var + (size_t)k * h->n, sizeof(double) * h->n, hipMemcpyDeviceToHost));
    return BSDE_OK;
}

bsde_status bsde_query_price_delta(bsde_problem h, int nq, const double *t,
                                   const double *S, double *price,
                                   double *delta)
{
    if (!h || nq < 0 || (nq > 0 && (!t || !S || !price)))
        return fail(BSDE_EINVAL, "bad query arguments");
    if (!h->have_alpha) return fail(BSDE_ESTATE, "no coefficients yet");
    const int d = h->d, dp = d + 1, p = h->p;
    const double *alpha = &h->alpha_hist[(size_t)h->k_done * p];
    if (h->kop) {
        // u = h[y] = S1 / S0 and d_{x_j} u = scale_j (d_j S1 - u d_j S0) / S0
        // over the points (FP64, the clamped Gaussian weights)
        const double b2 = h->base.kbw * h->base.kbw;
        for (int qi = 0; qi < nq; ++qi) {
            double z[kMaxD + 1];
            z[0] = 2.0 * t[qi] / h->base.T - 1.0;
            for (int j = 0; j < d; ++j) {
                if (!(S[(size_t)qi * d + j] > 0.0)) return fail(BSDE_EINVAL, "price must be > 0");
                z[1 + j] = (std::log(S[(size_t)qi * d + j]) - h->base.mid[j]) * h->base.scale[j];
            }
            double S0 = 0.0, S1 = 0.0, D0[kMaxD] = {0}, D1[kMaxD] = {0};
            for (int i = 0; i < h->n; ++i) {
                double dz[kMaxD + 1], q = 0.0;
                dz[0] = z[0] - (2.0 * h->pts[(size_t)i * dp] / h->base.T - 1.0);
                q = dz[0] * dz[0];
                for (int j = 0; j < d; ++j) {
                    dz[1 + j] = z[1 + j] - (h->pts[(size_t)i * dp + 1 + j] - h->base.mid[j]) *
                                               h->base.scale[j];
                    q += dz[1 + j] * dz[1 + j];
                }
                const double e = q / (2.0 * b2);
                const bool flat = e > kKernelClamp;
                const double w = std::exp(-(flat ? kKernelClamp : e));
                S0 += w;
                S1 += alpha[i] * w;
                if (flat) continue;
                for (int j = 0; j < d; ++j) {
                    D0[j] += w * (-dz[1 + j] / b2);
                    D1[j] += alpha[i] * w * (-dz[1 + j] / b2);
                }
            }
            const double u = S1 / S0;
            price[qi] = u;
            if (delta)
                for (int j = 0; j < d; ++j)
                    delta[(size_t)qi * d + j] =
                        (D1[j] - u * D0[j]) / S0 * h->base.scale[j] / S[(size_t)qi * d + j];
        }
        return BSDE_OK;
    }
    std::vector<double> g((size_t)d * p, 0.0); // d_{x_j} coefficients
    for (int j = 0; j < d; ++j)
        for (int l = 0; l < p; ++l) {
            double s = 0.0;
            for (const auto &x : h->Dx[j][l]) s += x.second * alpha[x.first];
            g[(size_t)j * p + l] = s;
        }
    for (int qi = 0; qi < nq; ++qi) {
        double z[kMaxD + 1];
        z[0] = 2.0 * t[qi] / h->base.T - 1.0;
        for (int j = 0; j < d; ++j) {
            if (!(S[(size_t)qi * d + j] > 0.0)) return fail(BSDE_EINVAL, "price must be > 0");
            z[1 + j] = (std::log(S[(size_t)qi * d + j]) - h->base.mid[j]) * h->base.scale[j];
        }
        double u = 0.0, du[kMaxD] = {0};
        for (int l = 0; l < p; ++l) {
            double bv = 1.0;
            for (int w = 0; w < dp; ++w) bv *= cheb_value(h->nu[(size_t)l * dp + w], z[w]);
            u += alpha[l] * bv;
            for (int j = 0; j < d; ++j) du[j] += g[(size_t)j * p + l] * bv;
        }
        price[qi] = u;
        if (delta)
            for (int j = 0; j < d; ++j) delta[(size_t)qi * d + j] = du[j] / S[(size_t)qi * d + j];
    }
    return BSDE_OK;
}

void bsde_destroy(bsde_problem h)
{
    if (!h) return;
    free_device(h);
    delete h;
}

} // extern "C"
