// Outer solve of the massive overlap equation (Sec. 4, Sec. 7):
//   (D_ov + mt) x = bt,   mt = m / (1 - m/(2 rho)),
//   bt = [1 + (m/(2 rho)) (1 - D_ov/(2 rho))] b / (1 - m/(2 rho))     complete form, eq. (upshot_complete)
//   bt = b / (1 - m/(2 rho))                                           traditional, eq. (upshot_traditional)
// (lattice spacing 1) by BiCGstab, each operator application being one ov_apply (the
// multi-shift evaluation of the rational) plus mt x.
//
// Cascaded preconditioning (Sec. 8, eqs. (cascaded_one), (cascaded_two)): with D^(0) = D_bri(-rho)
// and D^(k) = X r_{n_k}(X^dag X) the overlap approximants of growing Kenney-Laub order, every
// level works with A_k = rho [D^(k) + 1 + mt/rho] = D_ov^(n_k) + mt (and, at the Brillouin level,
// rho D_bri(-rho) + rho + mt).  A level's operator is inverted by BiCGstab preconditioned from the
// right by the next level's approximate inverse, itself an inner BiCGstab to a loose tolerance.
// Because the preconditioner changes from call to call, x is updated with the preconditioned
// vectors themselves (phat = K p, shat = K s, v = A phat, t = A shat), so the recursive residual
// stays the residual of x.
//
// Several right-hand sides run side by side, each with its own BiCGstab scalars; every operator
// application treats all of them in one batched call.  A column that has converged keeps its x
// and r until every column is done.  The host drives the recurrences; every vector operation and
// reduction runs on the device, reductions in FP64 with fixed block partial sums added in order on
// the host (deterministic).
//
// A half step of the kernel level is a stencil of 45 to 70 us (12^3 x 24, two columns, FP32) and vector
// work that a launch each would make as long, so what belongs together is one launch: a combination
// with the copy the stencil reads, or with the stencil's result and the dot products of the outcome
// (outer_step_kernel), and both updates of an iteration's end with theirs (outer_xr_kernel): five vector
// launches an iteration instead of sixteen.  The blocks write their partial sums straight into pinned
// host memory, so a dot product costs no copy, only the wait.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <complex>
#include <cstring>
#include <map>
#include <vector>

#include "common.hpp"

namespace bri {

int geom_check(const bri_geom *geom, Geom *g);

using cplx = std::complex<double>;

constexpr int MAXC = BRI_MAX_SOLVE_RHS;
constexpr int STEP_BLOCKS = 512;  // per column, at most
constexpr int STEP_THREADS = 256;
constexpr int MAXD = 2;  // dot products per launch

// per-column coefficients of a three-term combination
struct Coef3 {
    double2 c[MAXC][3];
};

// Column maps of the kernel level: only the columns still iterating go through its stencil.
struct ColMap {
    int idx[MAXC];
};

template <typename T> __device__ __forceinline__ T conv(double2 v);
template <> __device__ __forceinline__ double2 conv<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 conv<float2>(double2 v) { return make_float2((float)v.x, (float)v.y); }

// The block's sums of ND complex numbers per thread, to partial[d][col][block]
template <int ND>
__device__ __forceinline__ void step_sums(const double (&acc)[ND > 0 ? ND : 1][2], double2 *partial) {
    if constexpr (ND > 0) {
        __shared__ double2 sh[ND][STEP_THREADS / 64];
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            double sx = acc[d][0], sy = acc[d][1];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                sx += __shfl_down(sx, off, 64);
                sy += __shfl_down(sy, off, 64);
            }
            if (threadIdx.x % 64 == 0) sh[d][threadIdx.x / 64] = make_double2(sx, sy);
        }
        __syncthreads();
        if (threadIdx.x < ND) {
            double2 t = sh[threadIdx.x][0];
            for (int w = 1; w < STEP_THREADS / 64; ++w) {
                t.x += sh[threadIdx.x][w].x;
                t.y += sh[threadIdx.x][w].y;
            }
            partial[((size_t)threadIdx.x * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = t;
        }
    }
}

// <u, v> += conj(u) v
__device__ __forceinline__ void dot_add(double (&acc)[2], double2 u, double2 v) {
    acc[0] += u.x * v.x + u.y * v.y;
    acc[1] += u.x * v.y - u.y * v.x;
}

// One launch of vector work (column = blockIdx.y, vectors [ncol][n]; a null vector is a zero term, out
// may be one of the inputs, elementwise):
//   out = c0 x0 + c1 x1 + c2 x2 + kscale K,  K column kmap[col] of the compacted stencil result k
//         (type T; nothing where kmap < 0),
//   zero = 0,
//   column lmap[col] of lo = out converted to T (nothing where lmap < 0),
//   partial sums of <da, db> for ND pairs, a null vector standing for out.
struct Step {
    size_t n;
    double2 *out, *zero;
    Coef3 cf;
    const double2 *x[3];
    const void *k;
    double kscale;
    ColMap kmap;
    void *lo;
    ColMap lmap;
    const double2 *da[MAXD], *db[MAXD];
    double2 *partial;
};

template <typename T, int ND>
__global__ __launch_bounds__(STEP_THREADS) void outer_step_kernel(Step a) {
    const int col = blockIdx.y;
    const size_t off = (size_t)col * a.n;
    const int kc = a.k ? a.kmap.idx[col] : -1, lc = a.lo ? a.lmap.idx[col] : -1;
    const T *k = (const T *)a.k + (kc < 0 ? 0 : kc) * a.n;
    T *lo = (T *)a.lo + (lc < 0 ? 0 : lc) * a.n;
    double acc[ND > 0 ? ND : 1][2] = {};
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < a.n; i += (size_t)gridDim.x * blockDim.x) {
        double2 u[3], ud[ND > 0 ? ND : 1][2];
        T uk{};
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (a.x[j]) u[j] = a.x[j][off + i];
        if (kc >= 0) uk = k[i];
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            if (a.da[d]) ud[d][0] = a.da[d][off + i];
            if (a.db[d]) ud[d][1] = a.db[d][off + i];
        }
        double2 v = make_double2(0.0, 0.0);
        if (kc >= 0) v = make_double2(a.kscale * (double)uk.x, a.kscale * (double)uk.y);
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (a.x[j]) {
                const double2 c = a.cf.c[col][j];
                v.x += c.x * u[j].x - c.y * u[j].y;
                v.y += c.x * u[j].y + c.y * u[j].x;
            }
        a.out[off + i] = v;
        if (a.zero) a.zero[off + i] = make_double2(0.0, 0.0);
        if (lc >= 0) lo[i] = conv<T>(v);
#pragma unroll
        for (int d = 0; d < ND; ++d) dot_add(acc[d], a.da[d] ? ud[d][0] : v, a.db[d] ? ud[d][1] : v);
    }
    step_sums<ND>(acc, a.partial);
}

// the end of an iteration, for the columns with c[col][2].x != 0 (the others keep x and r):
//   x += c0 ph + c1 sh,  r = s - c1 t,  partial sums of <r, r> and <r0, r>
__global__ __launch_bounds__(STEP_THREADS) void outer_xr_kernel(size_t n, Coef3 cf, double2 *x, double2 *r,
                                                                const double2 *ph, const double2 *sh,
                                                                const double2 *s, const double2 *t,
                                                                const double2 *r0, double2 *partial) {
    const int col = blockIdx.y;
    if (cf.c[col][2].x == 0.0) return;
    const size_t off = (size_t)col * n;
    const double2 c0 = cf.c[col][0], c1 = cf.c[col][1];
    double acc[2][2] = {};
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        double2 xv = x[off + i];
        const double2 p = ph[off + i], q = sh[off + i], sv = s[off + i], tv = t[off + i], z = r0[off + i];
        xv.x += c0.x * p.x - c0.y * p.y;
        xv.y += c0.x * p.y + c0.y * p.x;
        xv.x += c1.x * q.x - c1.y * q.y;
        xv.y += c1.x * q.y + c1.y * q.x;
        x[off + i] = xv;
        double2 rv = sv;
        rv.x -= c1.x * tv.x - c1.y * tv.y;
        rv.y -= c1.x * tv.y + c1.y * tv.x;
        r[off + i] = rv;
        dot_add(acc[0], rv, rv);
        dot_add(acc[1], z, rv);
    }
    step_sums<2>(acc, partial);
}

static inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

using Cols = std::vector<cplx>;  // one coefficient per column

// one level of the cascade: its operator and the BiCGstab vectors of its solves
struct Level {
    int kl_n;       // 0: kernel operator, else overlap approximant of this order
    ov_params prm;  // overlap apply parameters (kl_n > 0)
    double tol;
    int max_iter;
    int kprec;  // kernel level: precision of its stencil (BRI_F64, or BRI_F32 / BRI_F32_BF16W on Wlo)
    double2 *r, *p, *v, *s, *t, *ph, *sh;  // [ncol][12 V] each
    int iters = 0, calls = 0, applies = 0;
};
constexpr int NVEC = 7;

// The pinned host memory that the partial sums of a solve go to: one buffer (256 KiB) per host thread and device,
// allocated on the thread's first solve there and freed when the thread ends, so that no solve pins or frees
// memory on its path (50 us a solve, and freeing waits for the whole device).  A thread runs one solve at a time.
constexpr size_t SUMS_COUNT = (size_t)MAXD * STEP_BLOCKS * MAXC;
struct ThreadSums {
    std::map<int, double2 *> bufs;
    ~ThreadSums() {
        for (auto &b : bufs) (void)hipHostFree(b.second);
    }
    double2 *get(int dev) {
        auto it = bufs.find(dev);
        if (it != bufs.end()) return it->second;
        void *p = nullptr;
        if (hipHostMalloc(&p, SUMS_COUNT * sizeof(double2), hipHostMallocDefault) != hipSuccess) return nullptr;
        return bufs[dev] = (double2 *)p;
    }
};
static thread_local ThreadSums t_sums;

struct HostSums {
    double2 *p = nullptr;
    hipStream_t s = nullptr;
    int dev = 0;
    bool get(hipStream_t stream) {
        s = stream;
        if (hipGetDevice(&dev) == hipSuccess) p = t_sums.get(dev);
        return p != nullptr;
    }
    ~HostSums() {
        // a launch of a solve that failed may still write; if that cannot be waited for, the buffer is given up
        if (p && hipStreamSynchronize(s) != hipSuccess) t_sums.bufs.erase(dev);
    }
};

struct Cascade {
    const bri_geom *geom;
    Geom g;
    const void *W64, *Wlo;
    double rho, mt;
    size_t n;  // complex entries per column
    int ncol;
    hipStream_t s;
    void *ov;
    size_t ov_bytes;
    float2 *lo_in = nullptr, *lo_out = nullptr;  // low-precision kernel level: [ncol][12 V] each
    double2 *k_in = nullptr, *k_out = nullptr;   // FP64 kernel level, compacted columns
    HostSums sums;
    std::vector<Level> lev;
    int inner_iters = 0;
    ov_stats ist;

    Cols all(cplx v) const { return Cols(ncol, v); }

    int blocks() const { return (int)std::min<size_t>(STEP_BLOCKS, (n + STEP_THREADS - 1) / STEP_THREADS); }

    // out = c0 x0 + c1 x1 + c2 x2
    Step comb(double2 *out, const Cols &c0, const double2 *x0, const Cols &c1 = Cols(), const double2 *x1 = nullptr,
              const Cols &c2 = Cols(), const double2 *x2 = nullptr) const {
        Step a{};
        a.n = n;
        a.out = out;
        for (int c = 0; c < ncol; ++c) {
            const cplx k[3] = {c0.empty() ? 0.0 : c0[c], c1.empty() ? 0.0 : c1[c], c2.empty() ? 0.0 : c2[c]};
            for (int j = 0; j < 3; ++j) a.cf.c[c][j] = make_double2(k[j].real(), k[j].imag());
        }
        a.x[0] = x0;
        a.x[1] = x1;
        a.x[2] = x2;
        a.partial = sums.p;
        return a;
    }

    // the launch of a, with the compacted vectors k and lo complex float (narrow) or double
    int run(const Step &a, int nd = 0, bool narrow = false) {
        const dim3 grid(blocks(), ncol), block(STEP_THREADS);
        if (nd == 0 && narrow)
            hipLaunchKernelGGL((outer_step_kernel<float2, 0>), grid, block, 0, s, a);
        else if (nd == 0)
            hipLaunchKernelGGL((outer_step_kernel<double2, 0>), grid, block, 0, s, a);
        else if (nd == 1 && narrow)
            hipLaunchKernelGGL((outer_step_kernel<float2, 1>), grid, block, 0, s, a);
        else if (nd == 1)
            hipLaunchKernelGGL((outer_step_kernel<double2, 1>), grid, block, 0, s, a);
        else if (nd == 2 && narrow)
            hipLaunchKernelGGL((outer_step_kernel<float2, 2>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((outer_step_kernel<double2, 2>), grid, block, 0, s, a);
        return hipGetLastError() == hipSuccess ? BRI_OK : BRI_EHIP;
    }

    // the nd dot products per column of the launch before, their partial sums added in order;
    // res[d][col]; synchronises the stream.  Columns outside `act` hold nothing of use.
    int take_dots(int nd, std::vector<Cols> &res) {
        if (hipStreamSynchronize(s) != hipSuccess) return BRI_EHIP;
        const int nb = blocks();
        res.assign(nd, Cols(ncol));
        for (int d = 0; d < nd; ++d)
            for (int c = 0; c < ncol; ++c) {
                double re = 0.0, im = 0.0;
                const double2 *q = sums.p + ((size_t)d * ncol + c) * nb;
                for (int i = 0; i < nb; ++i) {
                    re += q[i].x;
                    im += q[i].y;
                }
                res[d][c] = cplx(re, im);
            }
        return BRI_OK;
    }
    int run_dots(const Step &a, int nd, std::vector<Cols> &res, bool narrow = false) {
        const int rc = run(a, nd, narrow);
        return rc != BRI_OK ? rc : take_dots(nd, res);
    }

    // whether the kernel level's stencil works on a compacted copy of its input: in low precision, or
    // of the active columns where some are not
    bool compacted(const Level &L, const std::vector<char> &act) const {
        return L.kl_n == 0 && (L.kprec != BRI_F64 || std::count(act.begin(), act.end(), 0) > 0);
    }
    ColMap compact_map(const std::vector<char> &act, int *k) const {
        ColMap m{};
        *k = 0;
        for (int c = 0; c < ncol; ++c) m.idx[c] = act[c] ? (*k)++ : -1;
        return m;
    }
    // a leaves the copy the stencil of level L reads as well
    bool feed(Step &a, const Level &L, const std::vector<char> &act) const {
        if (!compacted(L, act)) return false;
        int k;
        a.lmap = compact_map(act, &k);
        a.lo = L.kprec != BRI_F64 ? (void *)lo_in : (void *)k_in;
        return L.kprec != BRI_F64;
    }

    // out = A_k v (a.out, with a's dot products; a holds nothing else yet), out != v.  Columns outside
    // `act` are zero in v and come out zero: the multi-shift drops zero columns at its start, and the
    // kernel level applies its stencil to the active columns only, from the copy that the launch which
    // made v left (feed), in the level's precision.
    int apply_a(Level &L, const double2 *v, Step a, const std::vector<char> &act, int nd, std::vector<Cols> &res) {
        double2 *dst = a.out;
        const Step dotted = a;
        if (L.kl_n == 0 && compacted(L, act)) {
            ++L.applies;
            const bool lo = L.kprec != BRI_F64;
            int k;
            a = comb(dst, all(rho + mt), v);
            a.kmap = compact_map(act, &k);
            a.k = lo ? (const void *)lo_out : (const void *)k_out;
            a.kscale = rho;
            const int r = kernel_apply(L, lo ? Wlo : W64, lo ? (const void *)lo_in : (const void *)k_in,
                                       lo ? (void *)lo_out : (void *)k_out, k);
            if (r != BRI_OK) return r;
        } else {
            const int r = apply_d(L, v, dst);
            if (r != BRI_OK) return r;
            a = L.kl_n == 0 ? comb(dst, all(rho), dst, all(rho + mt), v) : comb(dst, all(1.0), dst, all(mt), v);
        }
        for (int d = 0; d < MAXD; ++d) {
            a.da[d] = dotted.da[d];
            a.db[d] = dotted.db[d];
        }
        return run_dots(a, nd, res, L.kl_n == 0 && L.kprec != BRI_F64);
    }

    // D_kernel(-rho) of k columns in the level's precision
    int kernel_apply(const Level &L, const void *W, const void *in, void *out, int k) {
        return L.prm.kernel == BRI_KERNEL_WILSON ? ::wil_apply(geom, W, L.kprec, -rho, in, out, k, s)
                                                 : ::bri_apply(geom, W, L.kprec, -rho, in, out, k, s);
    }

    // dst = D_ov^(n_k) v (kl_n > 0) or D_kernel(-rho) v (kl_n = 0) of every column; dst != v
    int apply_d(Level &L, const double2 *v, double2 *dst) {
        ++L.applies;
        if (L.kl_n == 0) return kernel_apply(L, W64, v, dst, ncol);
        size_t ob = ov_bytes;
        const int r = ::ov_apply(geom, W64, Wlo, &L.prm, v, dst, ncol, ov, &ob, &ist, s);
        inner_iters += ist.iters;
        // a loose preconditioner may stop its multi-shift at the cap
        return (r == BRI_ENOCONV && &L != &lev[0]) ? BRI_OK : r;
    }

    // *res = approximate A_{k+1}^{-1} v, in dst, or v itself below the last level
    int precondition(int k, const double2 *v, double2 *dst, const double2 **res) {
        *res = v;
        if (k + 1 >= (int)lev.size()) return BRI_OK;
        *res = dst;
        int it;
        const int r = solve(k + 1, v, dst, it, nullptr);
        // an inner level that stops at its cap (or breaks down after progress) still preconditions
        return (r == BRI_ENOCONV) ? BRI_OK : r;
    }

    // BiCGstab on A_k x = b from x = 0 (shadow residual r0 = b) for every column, right-
    // preconditioned by level k+1.  A column stops at its own tolerance; at the outer level a
    // breakdown is an error, inside the cascade the column keeps what it has.
    int solve(int k, const double2 *b, double2 *x, int &it, std::vector<double> *rel_out) {
        Level &L = lev[k];
        ++L.calls;
        std::vector<Cols> d;
        int rc;
        {
            Step a = comb(L.r, all(1.0), b);  // r = b, x = 0, <b, b>
            a.zero = x;
            if ((rc = run_dots(a, 1, d)) != BRI_OK) return rc;
        }
        std::vector<double> bn(ncol), rel(ncol, 0.0);
        std::vector<char> active(ncol, 0);
        Cols rho_new(ncol), rho_old(ncol, 1.0), alpha(ncol, 1.0), omega(ncol, 1.0);
        int nact = 0;
        for (int c = 0; c < ncol; ++c) {
            bn[c] = std::sqrt(d[0][c].real());
            if (!std::isfinite(bn[c])) return BRI_ENAN;
            active[c] = bn[c] > 0.0;
            nact += active[c];
            rel[c] = active[c] ? 1.0 : 0.0;
            rho_new[c] = d[0][c];
        }
        const bool outer = k == 0;
        auto finish = [&](int status) {
            if (rel_out) *rel_out = rel;
            return status;
        };
        it = 0;
        while (nact > 0 && it < L.max_iter) {
            ++it;
            ++L.iters;
            Cols beta(ncol, 0.0), mbw(ncol, 0.0);
            for (int c = 0; c < ncol; ++c)
                if (active[c]) {
                    beta[c] = (rho_new[c] / rho_old[c]) * (alpha[c] / omega[c]);
                    mbw[c] = -beta[c] * omega[c];
                }
            // p = r + beta (p - omega v); a finished column gets p = 0, so the inner solves and the
            // multi-shift skip it
            Cols one_act(ncol, 0.0);
            for (int c = 0; c < ncol; ++c) one_act[c] = active[c] ? 1.0 : 0.0;
            Step a = it == 1 ? comb(L.p, one_act, L.r) : comb(L.p, one_act, L.r, beta, L.p, mbw, L.v);
            bool lo = feed(a, L, active);
            if ((rc = run(a, 0, lo)) != BRI_OK) return rc;
            const double2 *ph, *sh;
            if ((rc = precondition(k, L.p, L.ph, &ph)) != BRI_OK) return rc;
            a = Step{};
            a.out = L.v;
            a.da[0] = b;
            if ((rc = apply_a(L, ph, a, active, 1, d)) != BRI_OK) return rc;  // v = A K p, <r0, v>
            Cols ma(ncol, 0.0), half(ncol, 0.0);
            for (int c = 0; c < ncol; ++c) {
                if (!active[c]) continue;
                if (std::abs(d[0][c]) == 0.0 || !std::isfinite(d[0][c].real())) {
                    if (outer) return finish(BRI_ENAN);
                    active[c] = 0;
                    --nact;
                    continue;
                }
                alpha[c] = rho_new[c] / d[0][c];
                ma[c] = -alpha[c];
            }
            for (int c = 0; c < ncol; ++c) one_act[c] = active[c] ? 1.0 : 0.0;
            a = comb(L.s, one_act, L.r, ma, L.v);  // s = r - alpha v, <s, s>
            lo = feed(a, L, active);
            if ((rc = run_dots(a, 1, d, lo)) != BRI_OK) return rc;
            bool any_half = false;
            for (int c = 0; c < ncol; ++c) {
                if (!active[c]) continue;
                const double srel = std::sqrt(d[0][c].real()) / bn[c];
                if (!std::isfinite(srel)) return finish(BRI_ENAN);
                if (srel <= L.tol) {  // converged half way: x += alpha K p
                    half[c] = alpha[c];
                    rel[c] = srel;
                    active[c] = 0;
                    --nact;
                    any_half = true;
                }
            }
            if (any_half && (rc = run(comb(x, all(1.0), x, half, ph))) != BRI_OK) return rc;
            if (nact == 0) break;
            if (any_half) {  // the columns that just finished leave s as well
                for (int c = 0; c < ncol; ++c) one_act[c] = active[c] ? 1.0 : 0.0;
                a = comb(L.s, one_act, L.s);
                lo = feed(a, L, active);
                if ((rc = run(a, 0, lo)) != BRI_OK) return rc;
            }
            if ((rc = precondition(k, L.s, L.sh, &sh)) != BRI_OK) return rc;
            a = Step{};
            a.out = L.t;
            a.db[0] = L.s;
            if ((rc = apply_a(L, sh, a, active, 2, d)) != BRI_OK) return rc;  // t = A K s, <t, s>, <t, t>
            Coef3 cf{};
            for (int c = 0; c < ncol; ++c) {
                if (!active[c]) continue;
                if (d[1][c].real() == 0.0 || !std::isfinite(d[1][c].real())) {
                    if (outer) return finish(BRI_ENAN);
                    active[c] = 0;
                    --nact;
                    continue;
                }
                omega[c] = d[0][c] / d[1][c].real();
                cf.c[c][0] = make_double2(alpha[c].real(), alpha[c].imag());
                cf.c[c][1] = make_double2(omega[c].real(), omega[c].imag());
                cf.c[c][2].x = 1.0;
            }
            // x += alpha Kp + omega Ks, r = s - omega t, <r, r>, <r0, r>
            hipLaunchKernelGGL(outer_xr_kernel, dim3(blocks(), ncol), dim3(STEP_THREADS), 0, s, n, cf, x, L.r, ph, sh,
                               L.s, L.t, b, sums.p);
            if (hipGetLastError() != hipSuccess) return BRI_EHIP;
            rho_old = rho_new;
            if ((rc = take_dots(2, d)) != BRI_OK) return rc;
            for (int c = 0; c < ncol; ++c) {
                if (!active[c]) continue;
                rel[c] = std::sqrt(d[0][c].real()) / bn[c];
                rho_new[c] = d[1][c];
                if (!std::isfinite(rel[c])) return finish(BRI_ENAN);
                if (rel[c] <= L.tol) {
                    active[c] = 0;
                    --nact;
                } else if (std::abs(omega[c]) == 0.0 || std::abs(rho_new[c]) == 0.0) {
                    if (outer) return finish(BRI_ENAN);
                    active[c] = 0;
                    --nact;
                }
            }
        }
        return finish(nact > 0 ? BRI_ENOCONV : BRI_OK);
    }
};

static int check_levels(const ov_params *prm, const ov_mass_params *mp, int nprec, const ov_level *prec) {
    const double rho = prm->rho, m = mp->mass;
    if (!(m >= 0.0 && m < 2.0 * rho) || !(mp->tol > 0.0) || mp->max_iter < 1 ||
        (mp->complete != 0 && mp->complete != 1))
        return BRI_EINVAL;
    if (nprec < 0 || nprec > BRI_MAX_LEVELS || (nprec > 0 && !prec)) return BRI_EINVAL;
    for (int k = 0; k < nprec; ++k) {
        const ov_level &l = prec[k];
        if (l.kl_n < 0 || l.kl_n > BRI_MAX_SHIFTS || !(l.tol > 0.0) || l.max_iter < 1) return BRI_EINVAL;
        if (l.kl_n > 0 && !(l.ms_tol > 0.0)) return BRI_EINVAL;
        if (l.inner != BRI_F64 && l.inner != BRI_F32 && l.inner != BRI_F32_BF16W) return BRI_EINVAL;
        if (l.kl_n == 0 && k != nprec - 1) return BRI_EINVAL;  // the kernel level ends the chain
    }
    return BRI_OK;
}

static ov_params level_params(const ov_params *top, const ov_level &l) {
    ov_params p = *top;
    p.kl_n = l.kl_n;
    p.tol = l.ms_tol;
    p.inner = l.inner;
    p.kind = BRI_KL_DIAG;  // the cascade nests f_{1,1}: diagonal approximants only
    p.relax = 0;
    if (p.inner != BRI_F64 && p.max_refine == 0) p.max_refine = 10;
    return p;
}

}  // namespace bri

extern "C" {

int ov_solve(const bri_geom *geom, const void *W64, const void *Wlo, const ov_params *params,
             const ov_mass_params *mp, int nprec, const ov_level *prec, const void *in, void *out, int nrhs,
             void *work, size_t *work_bytes, ov_solve_stats *stats, void *stream) {
    using namespace bri;
    const auto t0 = std::chrono::steady_clock::now();
    Geom g;
    int rc = geom_check(geom, &g);
    if (rc != BRI_OK) return rc;
    if (!params || !mp || !work_bytes || nrhs < 1 || nrhs > MAXC) return BRI_EINVAL;
    if ((rc = check_levels(params, mp, nprec, prec)) != BRI_OK) return rc;
    // every low-precision piece reads the one array Wlo, so they must agree on its precision
    int lo_prec = params->inner != BRI_F64 ? params->inner : -1;
    bool lo_kernel = false;
    for (int k = 0; k < nprec; ++k) {
        if (prec[k].inner == BRI_F64) continue;
        if (lo_prec >= 0 && prec[k].inner != lo_prec) return BRI_EINVAL;
        lo_prec = prec[k].inner;
        lo_kernel = lo_kernel || prec[k].kl_n == 0;
    }
    // workspace: the largest ov_apply workspace of all levels, the vectors of every level, bt
    size_t ovb = 0;
    bool low = false;
    for (int k = -1; k < nprec; ++k) {
        if (k >= 0 && prec[k].kl_n == 0) continue;
        const ov_params p = k < 0 ? *params : level_params(params, prec[k]);
        low = low || p.inner != BRI_F64;
        size_t b = 0;
        rc = ov_apply(geom, nullptr, nullptr, &p, nullptr, nullptr, nrhs, nullptr, &b, nullptr, nullptr);
        if (rc != BRI_OK) return rc;
        ovb = b > ovb ? b : ovb;
    }
    const size_t vb = al256((size_t)12 * g.V * sizeof(double2) * nrhs);
    // (a level uses seven vectors; the reported size stays that of eight, the shadow residual's included)
    const size_t nvec = (size_t)(NVEC + 1) * (nprec + 1) + 1;
    bool f64_kernel = false;
    for (int k = 0; k < nprec; ++k) f64_kernel = f64_kernel || (prec[k].kl_n == 0 && prec[k].inner == BRI_F64);
    const size_t lb = lo_kernel ? al256((size_t)12 * g.V * sizeof(float2) * nrhs) : 0;
    const size_t kb = f64_kernel ? vb : 0;
    const size_t need = nvec * vb + al256(ovb) + 2 * lb + 2 * kb;
    if (!work) {
        *work_bytes = need;
        return BRI_OK;
    }
    if (*work_bytes < need || !W64 || !in || !out || ((low || lo_kernel) && !Wlo)) return BRI_EINVAL;
    {
        const size_t vbytes = (size_t)12 * g.V * nrhs * sizeof(double2);
        if (ranges_overlap(in, vbytes, out, vbytes) || ranges_overlap(in, vbytes, work, need) ||
            ranges_overlap(out, vbytes, work, need))
            return BRI_EINVAL;
    }

    Cascade c;
    c.geom = geom;
    c.g = g;
    c.W64 = W64;
    c.Wlo = Wlo;
    c.rho = params->rho;
    const double m = mp->mass, rho = params->rho;
    const double den = 1.0 - m / (2.0 * rho);
    c.mt = m / den;
    c.n = (size_t)12 * g.V;
    c.ncol = nrhs;
    c.s = (hipStream_t)stream;
    if (!c.sums.get(c.s)) return BRI_EHIP;
    char *base = (char *)work;
    auto take = [&](size_t b) {
        char *p = base;
        base += b;
        return p;
    };
    double2 *bt = (double2 *)take(vb);
    c.lev.resize(nprec + 1);
    for (int k = 0; k <= nprec; ++k) {
        Level &L = c.lev[k];
        if (k == 0) {
            L.kl_n = params->kl_n;
            L.prm = *params;
            L.tol = mp->tol;
            L.max_iter = mp->max_iter;
            L.kprec = BRI_F64;
        } else {
            L.kl_n = prec[k - 1].kl_n;
            L.prm = level_params(params, prec[k - 1]);
            L.tol = prec[k - 1].tol;
            L.max_iter = prec[k - 1].max_iter;
            L.kprec = prec[k - 1].kl_n == 0 ? prec[k - 1].inner : BRI_F64;
        }
        double2 **vs[NVEC] = {&L.r, &L.p, &L.v, &L.s, &L.t, &L.ph, &L.sh};
        for (auto vp : vs) *vp = (double2 *)take(vb);
    }
    c.ov = take(al256(ovb));
    c.ov_bytes = ovb;
    if (lo_kernel) {
        c.lo_in = (float2 *)take(lb);
        c.lo_out = (float2 *)take(lb);
    }
    if (f64_kernel) {
        c.k_in = (double2 *)take(kb);
        c.k_out = (double2 *)take(kb);
    }

    // bt
    const double2 *b = (const double2 *)in;
    double2 *x = (double2 *)out;
    Level &top = c.lev[0];
    const std::vector<char> every(nrhs, 1);
    if (mp->complete) {
        if ((rc = c.apply_d(top, b, top.t)) != BRI_OK) return rc;
        rc = c.run(c.comb(bt, c.all((1.0 + m / (2.0 * rho)) / den), b, c.all(-m / (4.0 * rho * rho) / den), top.t));
    } else {
        rc = c.run(c.comb(bt, c.all(1.0 / den), b));
    }
    if (rc != BRI_OK) return rc;
    int it = 0;
    const int result = c.solve(0, bt, x, it, nullptr);
    if (result != BRI_OK && result != BRI_ENOCONV) return result;
    // true residual |bt - A x| / |bt|, worst column
    double true_rel = 0.0;
    {
        std::vector<Cols> d, e;
        Step a{};
        a.out = top.t;
        a.da[0] = a.db[0] = bt;
        if ((rc = c.apply_a(top, x, a, every, 1, d)) != BRI_OK) return rc;
        if ((rc = c.run_dots(c.comb(top.t, c.all(1.0), bt, c.all(-1.0), top.t), 1, e)) != BRI_OK) return rc;
        for (int k = 0; k < nrhs; ++k) {
            const double bn = std::sqrt(d[0][k].real());
            if (bn > 0.0) true_rel = std::max(true_rel, std::sqrt(e[0][k].real()) / bn);
        }
    }
    if (stats) {
        std::memset(stats, 0, sizeof(*stats));
        stats->iters = it;
        stats->inner_iters = c.inner_iters;
        stats->applies = top.applies;
        stats->rel_resid = true_rel;
        for (int k = 1; k <= nprec; ++k) {
            stats->level_iters[k - 1] = c.lev[k].iters;
            stats->level_calls[k - 1] = c.lev[k].calls;
            stats->level_applies[k - 1] = c.lev[k].applies;
        }
        stats->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    return result;
}

}  // extern "C"
