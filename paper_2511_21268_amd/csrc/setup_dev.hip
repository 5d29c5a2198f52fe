// Device execution of the hierarchy set-up (Sec. 3.1): the test vector by
// relaxation on K w = 0, the compatible weighted matching, the pairwise
// prolongator and the Galerkin product, with the same bits as the host
// set-up in host_setup.cpp.  Built without FMA contraction; every sum runs in
// the host's order.
//
//  * Matching: rounds of locally dominant edges.  In each round every free
//    vertex points to its best eligible free neighbour in the strict order
//    (c descending, smaller end ascending, larger end ascending) and mutual
//    pointers are matched.  The best remaining edge is always mutual, so every
//    round with a candidate matches at least one pair (at most n/2 rounds), and
//    an edge matched this way is never preceded in the order by an edge that
//    could take one of its ends: the result is the greedy matching.
//  * Galerkin product for a one-entry-per-row prolongator: the contribution of
//    stored entry e (row i, column j) is (pc_i k_e) pc_j at coarse position
//    (agg_i, agg_j); the host adds the contributions of a position in
//    ascending e.  Entry indices are sorted by position with a stable radix
//    sort, and one thread per position sums its run in that order from +0.0.
#include "setup_dev.h"
#include "grid.h"

#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <new>
#include <stdexcept>
#include <vector>

namespace amgiga {
namespace {

#pragma clang fp contract(off)

struct HipError : std::runtime_error {
    using std::runtime_error::runtime_error;
};
struct OutOfMemory : HipError {
    using HipError::HipError;
};
struct InputError : std::runtime_error {
    using std::runtime_error::runtime_error;
};

[[noreturn]] void fail(hipError_t e)
{
    const std::string m = std::string("HIP error in set-up: ") + hipGetErrorString(e);
    if (e == hipErrorOutOfMemory) throw OutOfMemory(m);
    throw HipError(m);
}

#define DCHK(x)                                                                                      \
    do {                                                                                             \
        hipError_t e_ = (x);                                                                         \
        if (e_ != hipSuccess) fail(e_);                                                              \
    } while (0)

// hipMalloc whose failure is in its result alone: the runtime also keeps it for
// the next hipGetLastError, where a launch that succeeded (of this library, after
// a way round the failure, or of its caller) would find it.
hipError_t device_malloc(void **p, size_t bytes)
{
    const hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

// Device memory of one set-up call: a released block serves the next request
// of the call that fits it (all work of the call is in one stream, so the next
// use is ordered behind the last), the rest goes back when the call ends.
// hipMalloc and hipFree (which waits for the device) took 32 ms of the 96 ms
// of a set-up of 10.5M entries.
struct Block { void *p; size_t bytes; };
struct Pool {
    std::vector<Block> idle, used;
    void *take(size_t bytes)
    {
        bytes = (bytes + 255) / 256 * 256;
        idle.reserve(idle.size() + used.size() + 1);   // give() does not allocate
        used.reserve(used.size() + 1);
        // the smallest that fits, at most a quarter larger (small ones: 1 MB)
        size_t best = idle.size();
        for (size_t k = 0; k < idle.size(); k++)
            if (idle[k].bytes >= bytes && idle[k].bytes <= std::max(bytes + bytes / 4, size_t(1) << 20) &&
                (best == idle.size() || idle[k].bytes < idle[best].bytes))
                best = k;
        if (best < idle.size()) {
            used.push_back(idle[best]);
            idle.erase(idle.begin() + best);
            return used.back().p;
        }
        void *p = nullptr;
        hipError_t e = device_malloc(&p, bytes);
        if (e == hipErrorOutOfMemory && !idle.empty()) {
            trim();
            e = device_malloc(&p, bytes);
        }
        DCHK(e);
        used.push_back({p, bytes});
        return p;
    }
    bool give(void *p)
    {
        for (size_t k = used.size(); k-- > 0;)
            if (used[k].p == p) {
                idle.push_back(used[k]);
                used.erase(used.begin() + k);
                return true;
            }
        return false;
    }
    void trim()
    {
        for (Block &b : idle) (void)hipFree(b.p);
        idle.clear();
    }
};

// the running set-up call of this thread
thread_local Pool *t_pool = nullptr;

void *dev_alloc(size_t bytes)
{
    if (t_pool) return t_pool->take(bytes);
    void *p = nullptr;
    DCHK(device_malloc(&p, bytes));
    return p;
}
void dev_free(void *p)
{
    if (p && !(t_pool && t_pool->give(p))) (void)hipFree(p);
}

template <typename T> struct DBuf {
    T *p = nullptr;
    size_t n = 0;
    DBuf() = default;
    explicit DBuf(size_t k) { alloc(k); }
    void alloc(size_t k)
    {
        release();
        n = k;
        if (k) p = (T *)dev_alloc(k * sizeof(T));
    }
    void release()
    {
        dev_free(p);
        p = nullptr;
        n = 0;
    }
    void own(T *q, size_t k)
    {
        release();
        p = q;
        n = k;
    }
    ~DBuf() { release(); }
    DBuf(const DBuf &) = delete;
    DBuf &operator=(const DBuf &) = delete;
    DBuf(DBuf &&o) noexcept : p(o.p), n(o.n) { o.p = nullptr; o.n = 0; }
    DBuf &operator=(DBuf &&o) noexcept
    {
        release();
        p = o.p; n = o.n; o.p = nullptr; o.n = 0;
        return *this;
    }
};

inline unsigned grid(int64_t n) { return (unsigned)((n + 255) / 256); }

// ---- kernels --------------------------------------------------------------

__device__ inline int64_t find_col(const int64_t *rp, const int32_t *ci, int64_t row, int32_t col)
{
    int64_t lo = rp[row], hi = rp[row + 1] - 1;
    while (lo <= hi) {
        int64_t mid = (lo + hi) >> 1;
        int32_t c = ci[mid];
        if (c == col) return mid;
        if (c < col) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

// The kernels that pass over the entries give a row L neighbouring lanes, so
// that a wavefront reads consecutive entries: bound by memory on the first
// levels, by the launches on the later ones.  A thread per row, which
// strides the wavefront's reads by a row, took for the 10.5M entries of the
// 3D p=3 h=1/32 set-up 9.8 ms in the matching rounds, 7.4 ms in the edge
// weights, 4.0 ms in the keys of the products; 64 lanes take 0.74, 0.63 and
// 0.28 ms.  16 lanes below 100 entries a row: matching rounds of 2D p=2
// (25 a row) 11.8 ms against 26.8 with 64, 2D p=3 (49) 8.5 against 14.5, 3D p=2
// (114) 1.9 against 2.3 but keys 0.44 against 0.35.
#define FOR_ROW(L)                                                                      \
    const int lane = threadIdx.x % L;                                                   \
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / L; i < n; i += (int64_t)gridDim.x * 256 / L)
#define LAUNCH_ROWS(kernel, n, nnz, s, ...)                                                                      \
    do {                                                                                                         \
        if ((nnz) >= 100 * (n))                                                                                  \
            hipLaunchKernelGGL((kernel<64>), dim3(lanes_grid(n, 64)), dim3(256), 0, s, n, __VA_ARGS__);          \
        else hipLaunchKernelGGL((kernel<16>), dim3(lanes_grid(n, 16)), dim3(256), 0, s, n, __VA_ARGS__);         \
        DCHK(hipGetLastError());                                                                                 \
    } while (0)

__global__ void k_diag(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                       const double *__restrict__ v, double *__restrict__ diag)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t k = find_col(rp, ci, i, (int32_t)i);
    diag[i] = k >= 0 ? v[k] : 0.0;
}

// 1 / (k_ii + sum_{j != i} |k_ij|), the sum in ascending j after k_ii
__global__ void k_l1_invdiag(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                             const double *__restrict__ v, double *__restrict__ invd)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double d = 0.0;
    for (int64_t k = rp[i]; k < rp[i + 1]; k++)
        if (ci[k] == i) d = v[k];
    for (int64_t k = rp[i]; k < rp[i + 1]; k++)
        if (ci[k] != i) d = d + fabs(v[k]);
    invd[i] = 1.0 / d;
}

// one relaxation sweep on K w = 0: wout_i = w_i - invd_i sum_j k_ij w_j
__global__ void k_boot_sweep(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                             const double *__restrict__ v, const double *__restrict__ invd,
                             const double *__restrict__ w, double *__restrict__ wout)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double t = 0.0;
    for (int64_t k = rp[i]; k < rp[i + 1]; k++) t = t + v[k] * w[ci[k]];
    wout[i] = w[i] - invd[i] * t;
}

__device__ inline double cij_dev(double kij, double kii, double kjj, double wi, double wj)
{
    double num = ((2.0 * kij) * wi) * wj;
    double den = (kii * wi) * wi + (kjj * wj) * wj;
    return 1.0 - num / den;
}

// c of every stored entry (value of row min(i, j)); NaN marks an ineligible
// entry.  cnt[0] counts entries below the diagonal without a stored transpose.
template <int L>
__global__ void k_edge_c(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                         const double *__restrict__ v, const double *__restrict__ diag, const double *__restrict__ w,
                         int positive_only, double *__restrict__ cw, unsigned long long *cnt)
{
    unsigned long long missing = 0;
    FOR_ROW(L)
        for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += L) {
            const int64_t j = ci[k];
            double val = __builtin_nan("");
            if (j != i) {
                double kv;
                if (i < j) {
                    kv = v[k];
                    if (find_col(rp, ci, j, (int32_t)i) < 0) missing++;
                } else {
                    const int64_t t = find_col(rp, ci, j, (int32_t)i);
                    if (t < 0) missing++;
                    kv = t >= 0 ? v[t] : 0.0;
                }
                if (kv != 0.0) {
                    const int64_t a = i < j ? i : j, b = i < j ? j : i;
                    const double c = cij_dev(kv, diag[a], diag[b], w[a], w[b]);
                    const bool ok = isfinite(c) && (!positive_only || c > 1.0);
                    if (ok) val = c;
                }
            }
            cw[k] = val;
        }
    if (missing) atomicAdd(cnt, missing);
}

// edge (u, v) of weight c before edge (u, v2) of weight c2
__device__ inline bool edge_precedes(int64_t u, double c, int v, double c2, int v2)
{
    if (c != c2) return c > c2;
    const int64_t a = u < v ? u : v, b = u < v ? v : u, a2 = u < v2 ? u : v2, b2 = u < v2 ? v2 : u;
    if (a != a2) return a < a2;
    return b < b2;
}

// every free vertex points to its best eligible free neighbour (or -1): each
// lane the best of its entries, then the best of the lanes (the order is
// strict, so the best does not depend on who meets it first)
template <int L>
__global__ void k_ld_point(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                           const double *__restrict__ cw, const int32_t *__restrict__ mate,
                           int32_t *__restrict__ ptr)
{
    FOR_ROW(L) {
        if (mate[i] >= 0) {
            if (lane == 0) ptr[i] = -1;
            continue;
        }
        int best = -1;
        double bc = 0.0;
        for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += L) {
            const double c = cw[k];
            if (c != c) continue;
            const int v = ci[k];
            if (mate[v] >= 0) continue;
            if (best >= 0 && !edge_precedes(i, c, v, bc, best)) continue;
            best = v; bc = c;
        }
#pragma unroll
        for (int m = L / 2; m > 0; m /= 2) {
            const int v = __shfl_xor(best, m, L);
            const double c = __shfl_xor(bc, m, L);
            if (v >= 0 && (best < 0 || edge_precedes(i, c, v, bc, best))) { best = v; bc = c; }
        }
        if (lane == 0) ptr[i] = best;
    }
}

// any: set where a vertex had a candidate, by one store a block (stores of every
// row to the one word cost 1.2 ms of a round of 36,000 rows)
__global__ void k_ld_match(int64_t n, const int32_t *__restrict__ ptr, int32_t *__restrict__ mate,
                           unsigned int *__restrict__ any)
{
    int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t v = u < n ? ptr[u] : -1;
    if (v >= 0 && ptr[v] == (int32_t)u) mate[u] = v;
    if (__syncthreads_or(v >= 0) && threadIdx.x == 0)
        __hip_atomic_store(any, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_fill_i32(int64_t n, int32_t val, int32_t *__restrict__ d)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = val;
}

// 1 where row i opens a coarse index (singleton or the smaller of its pair)
__global__ void k_open(int64_t n, const int32_t *__restrict__ mate, int32_t *__restrict__ flag)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t m = mate[i];
    flag[i] = (m < 0 || i < m) ? 1 : 0;
}

// coarse index by the smallest member, pairwise prolongator coefficient and
// the restricted test vector (eq. (prolongation))
__global__ void k_pairwise(int64_t n, const int32_t *__restrict__ mate, const double *__restrict__ w,
                           const int32_t *__restrict__ idx, int32_t *__restrict__ agg, double *__restrict__ pc,
                           double *__restrict__ wc)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t j = mate[i];
    const int32_t I = (j < 0 || i < j) ? idx[i] : idx[j];
    agg[i] = I;
    if (j >= 0) {
        const double s = sqrt(w[i] * w[i] + w[j] * w[j]);
        pc[i] = w[i] / s;
        if (i < j) wc[I] = s;
    } else {
        pc[i] = (w[i] != 0.0) ? w[i] / fabs(w[i]) : 1.0;
        wc[I] = fabs(w[i]);
    }
}

// sort keys (coarse row, coarse column), entry indices and contributions
template <int L>
__global__ void k_gal_keys(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                           const double *__restrict__ v, const int32_t *__restrict__ agg, const double *__restrict__ pc,
                           uint64_t *__restrict__ keys, int32_t *__restrict__ vals, double *__restrict__ t, int cb)
{
    FOR_ROW(L) {
        const uint64_t I = (uint64_t)(uint32_t)agg[i];
        const double pi = pc[i];
        for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += L) {
            const int32_t j = ci[k];
            keys[k] = (I << cb) | (uint64_t)(uint32_t)agg[j];
            vals[k] = (int32_t)k;
            t[k] = (pi * v[k]) * pc[j];
        }
    }
}

__global__ void k_run_heads(int64_t m, const uint64_t *__restrict__ keys, int32_t *__restrict__ head)
{
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= m) return;
    head[s] = (s == 0 || keys[s] != keys[s - 1]) ? 1 : 0;
}

__global__ void k_run_starts(int64_t m, const int32_t *__restrict__ head, const int64_t *__restrict__ runid,
                             int64_t *__restrict__ start)
{
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= m) return;
    if (head[s]) start[runid[s]] = s;
}

// one thread per position: the run's contributions in ascending entry index,
// from +0.0; the column, and the row pointers between the run before and this
__global__ void k_run_sums(int64_t nrun, int64_t rows, int cb, const int64_t *__restrict__ start,
                           const uint64_t *__restrict__ keys, const int32_t *__restrict__ vals,
                           const double *__restrict__ t, int32_t *__restrict__ cci, double *__restrict__ cv,
                           int64_t *__restrict__ crp)
{
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nrun) return;
    const int64_t s0 = start[g], s1 = start[g + 1];
    double acc = 0.0;
    for (int64_t s = s0; s < s1; s++) acc = acc + t[vals[s]];
    cv[g] = acc;
    const uint64_t key = keys[s0];
    cci[g] = (int32_t)(uint32_t)(key & ((uint64_t(1) << cb) - 1));
    const int64_t row = (int64_t)(key >> cb);
    for (int64_t r = g == 0 ? 0 : (int64_t)(keys[s0 - 1] >> cb) + 1; r <= row; r++) crp[r] = g;
    if (g == nrun - 1)
        for (int64_t r = row + 1; r <= rows; r++) crp[r] = nrun;
}

__global__ void k_compose(int64_t n, int32_t *__restrict__ agg, double *__restrict__ pc,
                          const int32_t *__restrict__ ag, const double *__restrict__ pcs)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t a = agg[i];
    pc[i] = pc[i] * pcs[a];
    agg[i] = ag[a];
}

// K P: positions (row, aggregate of the column), entry indices, products
template <int L>
__global__ void k_kp_keys(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                          const double *__restrict__ v, const int32_t *__restrict__ agg, const double *__restrict__ pc,
                          uint64_t *__restrict__ keys, int32_t *__restrict__ vals, double *__restrict__ t, int cb)
{
    FOR_ROW(L)
        for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += L) {
            const int32_t j = ci[k];
            keys[k] = ((uint64_t)i << cb) | (uint64_t)(uint32_t)agg[j];
            vals[k] = (int32_t)k;
            t[k] = v[k] * pc[j];
        }
}

// Raises bad unless the entries are in range, ascending, finite and symmetric
// bit for value, with a positive diagonal (validate_csr's conditions).  10.5M
// entries: 353 us; the host's pass 6 ms on 16 threads.
template <int L>
__global__ void k_check_csr(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                            const double *__restrict__ v, unsigned int *__restrict__ bad)
{
    FOR_ROW(L) {
        bool ok = true, diag = false;
        for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += L) {
            const int32_t j = ci[k];
            const double x = v[k];
            if (j < 0 || j >= n || (k > rp[i] && j <= ci[k - 1]) || !isfinite(x)) ok = false;
            else if (j == i) {
                diag = true;
                ok = ok && x > 0.0;
            } else {
                const int64_t t = find_col(rp, ci, j, (int32_t)i);
                ok = ok && t >= 0 && v[t] == x;
            }
        }
        int d = diag;
#pragma unroll
        for (int m = L / 2; m > 0; m /= 2) d |= __shfl_xor(d, m, L);
        if (!ok || !d) __hip_atomic_store(bad, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// widest column gap within a row; a wavefront's rows are gridDim.x * 256 / L apart
template <int L>
__global__ void k_max_gap(int64_t n, const int64_t *__restrict__ rp, const int32_t *__restrict__ ci,
                          unsigned int *__restrict__ gap)
{
    int m = 0;
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / L; i < n; i += (int64_t)gridDim.x * 256 / L)
        for (int64_t k = rp[i] + 1 + threadIdx.x % L; k < rp[i + 1]; k += L) m = max(m, ci[k] - ci[k - 1]);
#pragma unroll
    for (int d = 32; d > 0; d /= 2) m = max(m, __shfl_xor(m, d));
    if (threadIdx.x % 64 == 0 && m > 0) atomicMax(gap, (unsigned int)m);
}

// One block per slice of a SELL-C image, a thread per row and group of 8
// entries: it reads the group's entries from the row (consecutive addresses)
// and writes them as the image's 16-byte pieces, consecutive across the rows.
// Bound by the loads of a row by few lanes: 10.5M entries (0.23 GB in and out)
// 258 us; the host's fill of the same image and its upload took about 25 ms.
// Slices s0 on; ci and v hold the entries from e0 on.
__global__ __launch_bounds__(256) void k_fill_sell(int64_t n, int64_t row0, int64_t e0, const int64_t *__restrict__ rp,
                                                   const int32_t *__restrict__ ci, const double *__restrict__ v, int C,
                                                   int64_t s0, SellFill F)
{
    const int64_t s = s0 + blockIdx.x;
    const int r = threadIdx.x % C;
    const int64_t q = s * C + r, base = F.soff[s], ib = F.ibase[s];
    const int64_t row = F.perm ? (int64_t)F.perm[q] : (q < n ? q : -1);
    const int ng = (int)((F.soff[s + 1] - base) / (8 * C));
    const int64_t r0 = row >= 0 ? rp[row - row0] - e0 : 0;
    const int len = row >= 0 ? (int)(rp[row - row0 + 1] - e0 - r0) : 0;
    const int32_t *so = ib < 0 ? F.shoff + ((-1 - ib) >> 1) : nullptr;
    const int nu = ib < 0 ? F.ulen[s] : 0;
    if (threadIdx.x < C && F.col0) F.col0[q] = ib >= 0 && len > 0 ? ci[r0] : 0;
    for (int g = threadIdx.x / C; g < ng; g += 256 / C) {
        double o[8];
        if (so) {
            // entry of each shared offset, 0 where the row has none
#pragma unroll
            for (int t = 0; t < 8; t++) {
                const int k = 8 * g + t;
                o[t] = 0.0;
                if (k >= nu || len == 0) continue;
                if (len == nu) {   // the row has them all
                    o[t] = v[r0 + k];
                    continue;
                }
                const int32_t col = (int32_t)(row + so[k]);
                int lo = 0, hi = len - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (ci[r0 + mid] < col) lo = mid + 1;
                    else hi = mid;
                }
                if (ci[r0 + lo] == col) o[t] = v[r0 + lo];
            }
        } else {
#pragma unroll
            for (int t = 0; t < 8; t++) o[t] = 8 * g + t < len ? v[r0 + 8 * g + t] : 0.0;
        }
        if (F.v64) {
            double2 *d = reinterpret_cast<double2 *>(F.v64 + base) + (int64_t)(4 * g) * C + r;
#pragma unroll
            for (int t = 0; t < 4; t++) d[t * C] = make_double2(o[2 * t], o[2 * t + 1]);
        }
        if (F.v32) {
            float4 *d = reinterpret_cast<float4 *>(F.v32 + base) + (int64_t)(2 * g) * C + r;
#pragma unroll
            for (int t = 0; t < 2; t++)
                d[t * C] = make_float4((float)o[4 * t], (float)o[4 * t + 1], (float)o[4 * t + 2], (float)o[4 * t + 3]);
        }
        if (ib < 0) continue;
        // columns of the group and the one before it; past the row its last one
        int c[9];
#pragma unroll
        for (int t = 0; t < 9; t++) {
            const int k = min(8 * g + t - 1, len - 1);
            c[t] = len > 0 ? ci[r0 + max(k, 0)] : 0;
        }
        if (F.d16) {
            uint32_t w[4];
#pragma unroll
            for (int t = 0; t < 4; t++)
                w[t] = (uint32_t)(c[2 * t + 1] - c[2 * t]) | (uint32_t)(c[2 * t + 2] - c[2 * t + 1]) << 16;
            reinterpret_cast<uint4 *>(F.d16 + ib)[(int64_t)g * C + r] = make_uint4(w[0], w[1], w[2], w[3]);
            if (F.gcol) F.gcol[ib / 8 + (int64_t)g * C + r] = c[0];
        }
        if (F.c32) {
            int4 *d = reinterpret_cast<int4 *>(F.c32 + ib) + (int64_t)(2 * g) * C + r;
            d[0] = make_int4(c[1], c[2], c[3], c[4]);
            d[C] = make_int4(c[5], c[6], c[7], c[8]);
        }
    }
}

// ---- host driver ----------------------------------------------------------

struct BufCsr {
    int64_t n = 0, nnz = 0;
    DBuf<int64_t> rp;
    DBuf<int32_t> ci;
    DBuf<double> v;
    void take(DevCsr &d)
    {
        n = d.n; nnz = d.nnz;
        rp.own(d.rp, n + 1); ci.own(d.ci, nnz); v.own(d.v, nnz);
        d.rp = nullptr; d.ci = nullptr; d.v = nullptr;
    }
    DevCsr give()
    {
        DevCsr d;
        d.n = n; d.nnz = nnz;
        d.rp = rp.p; d.ci = ci.p; d.v = v.p;
        rp.p = nullptr; ci.p = nullptr; v.p = nullptr;
        return d;
    }
};

template <typename T> void up(DBuf<T> &d, const T *h, size_t k, hipStream_t s)
{
    d.alloc(k);
    if (k) DCHK(hipMemcpyAsync(d.p, h, k * sizeof(T), hipMemcpyHostToDevice, s));
}
template <typename T> void down(std::vector<T> &h, const DBuf<T> &d, size_t k, hipStream_t s)
{
    h.resize(k);
    if (k) DCHK(hipMemcpyAsync(h.data(), d.p, k * sizeof(T), hipMemcpyDeviceToHost, s));
}

template <typename TI, typename TO> void scan(const TI *in, TO *out, int64_t n, hipStream_t s)
{
    size_t b = 0;
    DCHK(hipcub::DeviceScan::ExclusiveSum(nullptr, b, in, out, (int)n, s));
    DBuf<char> tmp(b ? b : 1);
    DCHK(hipcub::DeviceScan::ExclusiveSum(tmp.p, b, in, out, (int)n, s));
}

// CSR (rows x cols) of sums of products: make_keys writes each of the m
// products' position (row << cb | column), its index (ascending order of the
// sum) and its value; equal positions are summed in index order from +0.0.
template <typename Keys>
BufCsr sum_products(int64_t m, int64_t rows, int64_t cols, hipStream_t s_, Keys make_keys)
{
    DBuf<uint64_t> keys(m), keys2(m);
    DBuf<int32_t> vals(m), vals2(m), head(m);
    DBuf<double> t(m);
    int cb = 1, rb = 1;   // bits of a column and of a row: the sort's passes go by their sum
    while ((int64_t(1) << cb) < cols) cb++;
    while ((int64_t(1) << rb) < rows) rb++;
    const int end_bit = cb + rb;
    make_keys(keys.p, vals.p, t.p, cb);
    DCHK(hipGetLastError());
    {
        size_t b = 0;
        DCHK(hipcub::DeviceRadixSort::SortPairs(nullptr, b, keys.p, keys2.p, vals.p, vals2.p, (int)m, 0, end_bit,
                                                s_));
        DBuf<char> tmp(b ? b : 1);
        DCHK(hipcub::DeviceRadixSort::SortPairs(tmp.p, b, keys.p, keys2.p, vals.p, vals2.p, (int)m, 0, end_bit,
                                                s_));
    }
    keys.release();
    vals.release();
    hipLaunchKernelGGL(k_run_heads, dim3(grid(m)), dim3(256), 0, s_, m, keys2.p, head.p);
    DCHK(hipGetLastError());
    DBuf<int64_t> runid(m);
    scan(head.p, runid.p, m, s_);
    int64_t last_run = 0;
    int32_t last_head = 0;
    DCHK(hipMemcpyAsync(&last_run, runid.p + (m - 1), sizeof(int64_t), hipMemcpyDeviceToHost, s_));
    DCHK(hipMemcpyAsync(&last_head, head.p + (m - 1), sizeof(int32_t), hipMemcpyDeviceToHost, s_));
    DCHK(hipStreamSynchronize(s_));
    const int64_t nrun = last_run + last_head;
    DBuf<int64_t> start(nrun + 1);
    hipLaunchKernelGGL(k_run_starts, dim3(grid(m)), dim3(256), 0, s_, m, head.p, runid.p, start.p);
    DCHK(hipMemcpyAsync(start.p + nrun, &m, sizeof(int64_t), hipMemcpyHostToDevice, s_));
    DCHK(hipGetLastError());
    BufCsr C;
    C.n = rows;
    C.nnz = nrun;
    C.ci.alloc(nrun);
    C.v.alloc(nrun);
    C.rp.alloc(rows + 1);
    hipLaunchKernelGGL(k_run_sums, dim3(grid(nrun)), dim3(256), 0, s_, nrun, rows, cb, start.p, keys2.p, vals2.p, t.p,
                       C.ci.p, C.v.p, C.rp.p);
    DCHK(hipGetLastError());
    DCHK(hipStreamSynchronize(s_));
    return C;
}

class DeviceCoarsener : public Coarsener {
  public:
    DeviceCoarsener(hipStream_t s, DevSetupInfo *info) : s_(s), info_(info) {}

    void bootstrap(const CsrView &K0, const double *w0, int sweeps, std::vector<double> &w) override
    {
        BufCsr &K = level0(K0);
        DBuf<double> invd(K.n), a(K.n), b(K.n);
        hipLaunchKernelGGL(k_l1_invdiag, dim3(grid(K.n)), dim3(256), 0, s_, K.n, K.rp.p, K.ci.p, K.v.p, invd.p);
        DCHK(hipMemcpyAsync(a.p, w0, K.n * sizeof(double), hipMemcpyHostToDevice, s_));
        for (int k = 0; k < sweeps; k++) {
            hipLaunchKernelGGL(k_boot_sweep, dim3(grid(K.n)), dim3(256), 0, s_, K.n, K.rp.p, K.ci.p, K.v.p, invd.p,
                               a.p, b.p);
            std::swap(a.p, b.p);
        }
        DCHK(hipGetLastError());
        down(w, a, K.n, s_);
        DCHK(hipStreamSynchronize(s_));
    }

    void coarsen(int level, const CsrView &Kh, const double *w, const SetupParams &prm, CoarsenResult &out) override
    {
        BufCsr &K0 = level == 0 ? level0(Kh) : cur_;
        if (K0.n != Kh.n || K0.nnz != Kh.nnz()) throw HipError("device set-up: level matrix out of step");
        const int64_t nl = K0.n;
        DBuf<int32_t> agg(nl);
        DBuf<double> pc(nl);
        DBuf<double> wv;
        up(wv, w, nl, s_);
        BufCsr C;
        const BufCsr *K = &K0;
        DBuf<double> wcur = std::move(wv);
        int64_t nc = nl;
        for (int sw = 0; sw < prm.sweeps; sw++) {
            DBuf<int32_t> mate(K->n), ag(K->n);
            DBuf<double> pcs(K->n), wc;
            match(*K, wcur.p, prm.positive_only, mate.p);
            nc = pairwise(*K, mate.p, wcur.p, ag, pcs, wc);
            BufCsr Cn = galerkin(*K, nc, ag.p, pcs.p);
            if (sw == 0) {
                DCHK(hipMemcpyAsync(agg.p, ag.p, nl * sizeof(int32_t), hipMemcpyDeviceToDevice, s_));
                DCHK(hipMemcpyAsync(pc.p, pcs.p, nl * sizeof(double), hipMemcpyDeviceToDevice, s_));
            } else {
                hipLaunchKernelGGL(k_compose, dim3(grid(nl)), dim3(256), 0, s_, nl, agg.p, pc.p, ag.p, pcs.p);
                DCHK(hipGetLastError());
            }
            C = std::move(Cn);
            K = &C;
            wcur = std::move(wc);
        }
        out.nc = nc;
        down(out.agg, agg, nl, s_);
        down(out.pc, pc, nl, s_);
        down(out.wc, wcur, nc, s_);
        out.C.n = C.n;
        down(out.C.rp, C.rp, C.n + 1, s_);
        down(out.C.ci, C.ci, C.nnz, s_);
        down(out.C.v, C.v, C.nnz, s_);
        DCHK(hipStreamSynchronize(s_));
        // a level's matrix is done with: the image set-up takes it over
        keep(level, level == 0 ? l0_ : cur_);
        cur_ = std::move(C);
        have_l0_ = have_l0_ && level > 0;
        last_ = level + 1;
    }
    // the coarsest level's
    void finish()
    {
        if (last_ > 0) keep(last_, cur_);
    }

  private:
    static constexpr int ROUNDS = 4;
    hipStream_t s_;
    DevSetupInfo *info_;
    BufCsr l0_, cur_;
    bool have_l0_ = false;
    int last_ = 0;

    void keep(int level, BufCsr &K)
    {
        if (!info_) return;
        if ((int)info_->levels.size() <= level) info_->levels.resize(level + 1);
        info_->levels[level] = K.give();
    }

    BufCsr &level0(const CsrView &K)
    {
        if (!have_l0_ && info_ && !info_->levels.empty() && info_->levels[0].rp) {   // checked there already
            l0_.take(info_->levels[0]);
            have_l0_ = true;
        }
        if (!have_l0_) {
            l0_.n = K.n;
            l0_.nnz = K.nnz();
            up(l0_.rp, K.rp, K.n + 1, s_);
            up(l0_.ci, K.ci, K.nnz(), s_);
            up(l0_.v, K.v, K.nnz(), s_);
            have_l0_ = true;
        }
        return l0_;
    }

    void match(const BufCsr &K, const double *w, int positive_only, int32_t *mate)
    {
        DBuf<double> diag(K.n), cw(K.nnz ? K.nnz : 1);
        DBuf<unsigned long long> cnt(1);
        DBuf<unsigned int> any(ROUNDS);
        DBuf<int32_t> ptr(K.n);
        DCHK(hipMemsetAsync(cnt.p, 0, sizeof(unsigned long long), s_));
        hipLaunchKernelGGL(k_diag, dim3(grid(K.n)), dim3(256), 0, s_, K.n, K.rp.p, K.ci.p, K.v.p, diag.p);
        LAUNCH_ROWS(k_edge_c, K.n, K.nnz, s_, K.rp.p, K.ci.p, K.v.p, diag.p, w, positive_only, cw.p, cnt.p);
        hipLaunchKernelGGL(k_fill_i32, dim3(grid(K.n)), dim3(256), 0, s_, K.n, -1, mate);
        DCHK(hipGetLastError());
        unsigned long long missing = 0;
        DCHK(hipMemcpyAsync(&missing, cnt.p, sizeof(missing), hipMemcpyDeviceToHost, s_));
        DCHK(hipStreamSynchronize(s_));
        if (missing) throw InputError("device set-up needs a structurally symmetric matrix");
        // at most n/2 + 1 rounds: each round with a candidate matches a pair.
        // ROUNDS at a time, one wait for them; those past the first round
        // without a candidate change nothing and are not counted.
        int rounds = 0;
        for (int64_t r = 0; r <= K.n / 2 + 1; r += ROUNDS) {
            unsigned int h_any[ROUNDS];
            DCHK(hipMemsetAsync(any.p, 0, sizeof(h_any), s_));
            for (int k = 0; k < ROUNDS; k++) {
                LAUNCH_ROWS(k_ld_point, K.n, K.nnz, s_, K.rp.p, K.ci.p, cw.p, mate, ptr.p);
                hipLaunchKernelGGL(k_ld_match, dim3(grid(K.n)), dim3(256), 0, s_, K.n, ptr.p, mate, any.p + k);
            }
            DCHK(hipGetLastError());
            DCHK(hipMemcpyAsync(h_any, any.p, sizeof(h_any), hipMemcpyDeviceToHost, s_));
            DCHK(hipStreamSynchronize(s_));
            int k = 0;
            while (k < ROUNDS && h_any[k]) k++;
            rounds += k < ROUNDS ? k + 1 : ROUNDS;
            if (k < ROUNDS) break;
        }
        if (info_) {
            info_->rounds_total += rounds;
            if (rounds > info_->rounds_max) info_->rounds_max = rounds;
            info_->sweeps++;
        }
    }

    int64_t pairwise(const BufCsr &K, const int32_t *mate, const double *w, DBuf<int32_t> &ag, DBuf<double> &pcs,
                     DBuf<double> &wc)
    {
        const int64_t n = K.n;
        DBuf<int32_t> flag(n), idx(n);
        hipLaunchKernelGGL(k_open, dim3(grid(n)), dim3(256), 0, s_, n, mate, flag.p);
        DCHK(hipGetLastError());
        scan(flag.p, idx.p, n, s_);
        int32_t last_idx = 0, last_flag = 0;
        DCHK(hipMemcpyAsync(&last_idx, idx.p + (n - 1), sizeof(int32_t), hipMemcpyDeviceToHost, s_));
        DCHK(hipMemcpyAsync(&last_flag, flag.p + (n - 1), sizeof(int32_t), hipMemcpyDeviceToHost, s_));
        DCHK(hipStreamSynchronize(s_));
        const int64_t nc = (int64_t)last_idx + last_flag;
        wc.alloc(nc);
        hipLaunchKernelGGL(k_pairwise, dim3(grid(n)), dim3(256), 0, s_, n, mate, w, idx.p, ag.p, pcs.p, wc.p);
        DCHK(hipGetLastError());
        return nc;
    }

    BufCsr galerkin(const BufCsr &K, int64_t nc, const int32_t *agg, const double *pc)
    {
        return sum_products(K.nnz, nc, nc, s_, [&](uint64_t *keys, int32_t *vals, double *t, int cb) {
            LAUNCH_ROWS(k_gal_keys, K.n, K.nnz, s_, K.rp.p, K.ci.p, K.v.p, agg, pc, keys, vals, t, cb);
        });
    }
};

}  // namespace

static constexpr int64_t FILL_PIECE = int64_t(1) << 22;   // entries uploaded at a time (50 MB)

template <typename F> static int guarded(std::string &err, F f)
{
    try {
        f();
        return 0;
    } catch (OutOfMemory &e) {
        err = e.what();
        return -4;
    } catch (HipError &e) {
        err = e.what();
        return -3;
    } catch (std::bad_alloc &) {
        err = "host allocation failed";
        return -4;
    }
}

DevCsr::~DevCsr()
{
    for (void *p : {(void *)rp, (void *)ci, (void *)v}) dev_free(p);
}

SetupMemory::SetupMemory()
{
    if (!t_pool) pool_ = t_pool = new (std::nothrow) Pool();
}
void SetupMemory::trim()
{
    if (t_pool) t_pool->trim();
}
SetupMemory::~SetupMemory()
{
    if (!pool_) return;
    t_pool->trim();
    // what is still out (nothing, unless a call failed) is freed by its owner
    t_pool = nullptr;
    delete (Pool *)pool_;
}

int csr_to_device(const CsrView &K, void *stream, DevCsr &D, std::string &err)
{
    return guarded(err, [&] {
        hipStream_t s = (hipStream_t)stream;
        BufCsr B;
        B.n = K.n;
        B.nnz = K.nnz();
        up(B.rp, K.rp, K.n + 1, s);
        up(B.ci, K.ci, K.nnz(), s);
        up(B.v, K.v, K.nnz(), s);
        DCHK(hipStreamSynchronize(s));
        D = B.give();
    });
}

int check_csr(const DevCsr &K, void *stream, bool &valid, std::string &err)
{
    return guarded(err, [&] {
        hipStream_t s = (hipStream_t)stream;
        DBuf<unsigned int> bad(1);
        unsigned int h_bad = 0;
        DCHK(hipMemsetAsync(bad.p, 0, sizeof(h_bad), s));
        LAUNCH_ROWS(k_check_csr, K.n, K.nnz, s, K.rp, K.ci, K.v, bad.p);
        DCHK(hipMemcpyAsync(&h_bad, bad.p, sizeof(h_bad), hipMemcpyDeviceToHost, s));
        DCHK(hipStreamSynchronize(s));
        valid = h_bad == 0;
    });
}

int kp_on_device(const DevCsr &K, int64_t nc, const int32_t *agg, const double *pc, void *stream, DevCsr &KP,
                 std::vector<int64_t> &rp, int64_t &max_gap, std::string &err)
{
    return guarded(err, [&] {
        hipStream_t s = (hipStream_t)stream;
        BufCsr P = sum_products(K.nnz, K.n, nc, s, [&](uint64_t *keys, int32_t *vals, double *t, int cb) {
            LAUNCH_ROWS(k_kp_keys, K.n, K.nnz, s, K.rp, K.ci, K.v, agg, pc, keys, vals, t, cb);
        });
        DBuf<unsigned int> gap(1);
        unsigned int h_gap = 0;
        DCHK(hipMemsetAsync(gap.p, 0, sizeof(unsigned int), s));
        hipLaunchKernelGGL((k_max_gap<16>), dim3(std::min(grid(P.n * 16), 512u)), dim3(256), 0, s, P.n, P.rp.p, P.ci.p,
                           gap.p);
        DCHK(hipGetLastError());
        down(rp, P.rp, P.n + 1, s);
        DCHK(hipMemcpyAsync(&h_gap, gap.p, sizeof(h_gap), hipMemcpyDeviceToHost, s));
        DCHK(hipStreamSynchronize(s));
        max_gap = h_gap;
        KP = P.give();
    });
}

int fill_sell(const DevCsr &K, int C, int64_t nslices, const SellFill &F, void *stream, std::string &err)
{
    return guarded(err, [&] {
        for (int64_t s0 = 0; s0 < nslices; s0 += MAX_BLOCKS) {
            const unsigned g = (unsigned)std::min<int64_t>(nslices - s0, MAX_BLOCKS);
            hipLaunchKernelGGL(k_fill_sell, dim3(g), dim3(256), 0, (hipStream_t)stream, K.n, (int64_t)0, (int64_t)0,
                               K.rp, K.ci, K.v, C, s0, F);
            DCHK(hipGetLastError());
        }
    });
}

static void fill_pieces(const CsrView &K, int C, const SellFill &F, hipStream_t s, int64_t piece)
{
    const int64_t win = 4 * C;   // rows of a sorted window: the pieces end between windows
    for (int64_t a = 0, b; a < K.n; a = b) {
        b = std::min(K.n, a + win);
        while (b < K.n && K.rp[std::min(K.n, b + win)] - K.rp[a] <= piece) b = std::min(K.n, b + win);
        const int64_t e0 = K.rp[a], m = K.rp[b] - e0;
        DBuf<int64_t> rp;
        DBuf<int32_t> ci;
        DBuf<double> v;
        up(rp, K.rp + a, b - a + 1, s);
        up(ci, K.ci + e0, m, s);
        up(v, K.v + e0, m, s);
        hipLaunchKernelGGL(k_fill_sell, dim3((unsigned)((b - a + C - 1) / C)), dim3(256), 0, s, K.n, a, e0, rp.p, ci.p,
                           v.p, C, a / C, F);
        DCHK(hipGetLastError());
        DCHK(hipStreamSynchronize(s));
    }
}

int fill_sell(const CsrView &K, int C, const SellFill &F, void *stream, std::string &err)
{
    return guarded(err, [&] {
        for (int64_t piece = FILL_PIECE;; piece /= 64) {   // smaller pieces where memory is short
            try {
                return fill_pieces(K, C, F, (hipStream_t)stream, piece);
            } catch (OutOfMemory &) {
                if (piece < 64) throw;
                SetupMemory::trim();
            }
        }
    });
}

int build_hierarchy_on_device(const CsrView &K0, const double *w, const SetupParams &prm, HostHierarchy &H,
                              std::string &err, void *stream, DevSetupInfo *info)
{
    if (K0.nnz() >= (int64_t(1) << 31) || K0.n >= (int64_t(1) << 31)) {
        err = "device set-up takes fewer than 2^31 stored entries";
        return -1;
    }
    if (prm.smooth) {
        err = "device set-up builds the tentative prolongator only (smooth_prolong 0)";
        return -1;
    }
    try {
        DeviceCoarsener dc((hipStream_t)stream, info);
        const int rc = build_hierarchy(K0, w, prm, H, err, &dc);
        if (rc == 0) dc.finish();
        return rc;
    } catch (InputError &e) {
        err = e.what();
        return -1;
    } catch (HipError &e) {
        err = e.what();
        return -3;
    } catch (std::bad_alloc &) {
        err = "host allocation failed";
        return -4;
    }
}

}  // namespace amgiga
