// Plain conjugate residual on the Hermitian indefinite H = Gamma5 D_dwf (Sec. 3), FP64.
//
//   r = b - H x;  p = r;  Ar = H r;  Ap = Ar
//   repeat:  alpha = Re<r,Ar>/|Ap|^2;  x += alpha p;  r -= alpha Ap
//            Ar = H r;  beta = Re<r',Ar'>/Re<r,Ar>;  p = r + beta p;  Ap = Ar + beta Ap
//
// A step is three launches: Ar = H r, the inner products with Ar, and one update
// of p, Ap, x and r.  The scalars live in device memory: every workgroup of the
// update reduces the partial sums of the two kernels before it, in the same
// fixed order, and so takes the same decisions; convergence and breakdown set a
// flag that ends the later launches of a batch and is not read in its own.  The
// host enqueues a batch of steps and reads the flag and the residual norms back
// once per batch.  On convergence of the updated residual the true residual b - H x
// is recomputed; if it does not meet the tolerance the iteration restarts from it.
//
// The steps' vectors are streamed, so their bytes bound a step: |Ap|^2 comes from
//   |Ar + beta Ap|^2 = |Ar|^2 + 2 beta Re<Ap,Ar> + beta^2 |Ap|^2,
// so that one pass updates all four vectors, and x takes the steps two at a
// time, from the old and the new p of the second: the update moves 8 vectors a
// step on average (two passes with a reduction between them moved 12).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "solver.h"

namespace hdcr {

namespace {

// device scalars of the iteration
enum { S_RR0 = 0,    // |r|^2 of the residual the iteration starts from
       S_BB = 1,     // |b|^2
       S_RAR = 2,    // Re<r,Ar> of the even (2) and odd (3) steps
       S_ALPHA = 4,  // alpha of the even (4) and odd (5) steps
       S_HIST = 6 }; // |r|^2 after each step of the batch
constexpr int CR_BLOCKS = 512;  // most workgroups of the update: each of them adds up the others' partials
constexpr int CR_BATCH = 32;  // most steps between two read-backs
constexpr int CR_COMPRESS = 32;  // workgroups that sum the apply's own partials
constexpr int S_COUNT = S_HIST + CR_BATCH;
// flags: stop reason and completed steps since the start
enum { CR_RUN = 0, CR_CONVERGED = 1, CR_BREAKDOWN = 2, CR_NAN = 3 };
struct CrState {
    double S[S_COUNT];
    // of the even / odd steps: step k reads the reason of step k - 1 and writes its own.
    // If a launch read the one that it writes, a late workgroup could end some of its
    // wavefronts and not the others, whose sums would then take in what LDS held before
    int reason[2];
    int steps;
};

// sums of NQ doubles over the workgroup (REDUCE_THREADS work-items, fixed order:
// lanes by halves, then the wavefronts in order); every work-item gets them
template <int NQ> __device__ __forceinline__ void wg_sums(double (&v)[NQ]) {
    constexpr int WAVES = REDUCE_THREADS / 64;
    __shared__ double sh[NQ][WAVES];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) v[q] += __shfl_xor(v[q], m);
    __syncthreads();  // an earlier call may still be reading sh
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) sh[q][threadIdx.x >> 6] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        v[q] = sh[q][0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v[q] += sh[q][w];
    }
}

// Columns i, i + REDUCE_THREADS, ... of ROWS rows of np partials, four at a time,
// zeros past the end: every load is issued before the first is used (the sums
// with error terms keep the compiler from unrolling the loop over them).
template <int ROWS>
__device__ __forceinline__ void load_partials(const double* __restrict__ part, int np, int i, double (&o)[ROWS][4]) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = i + u * REDUCE_THREADS;
            const double v = part[(size_t)r * np + (k < np ? k : 0)];
            o[r][u] = k < np ? v : 0.0;
        }
}
// v[q] = sums of NQ rows of partials
template <int NQ> __device__ __forceinline__ void add_partials(const double* __restrict__ part, int np, double (&v)[NQ]) {
    for (int i = threadIdx.x; i < np; i += 4 * REDUCE_THREADS) {
        double o[NQ][4];
        load_partials<NQ>(part, np, i, o);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[q] += o[q][u];
    }
}

// the same for a sum with its error terms; NS of them from NS row pairs (hi, lo)
template <int NS> __device__ __forceinline__ void wg_sums2(Sum2 (&v)[NS]) {
    constexpr int WAVES = REDUCE_THREADS / 64;
    __shared__ Sum2 sh[NS][WAVES];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) v[q] = v[q] + shfl_xor2(v[q], m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < NS; ++q) sh[q][threadIdx.x >> 6] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        v[q] = sh[q][0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) v[q] = v[q] + sh[q][w];
    }
}
// v += row 0, q[k] += rows 1 + 2 k (hi) and 2 + 2 k (lo) of the partials; o: the first
// chunk, loaded before
template <int NS>
__device__ __forceinline__ void add_rows(const double* __restrict__ part, int np, double (&o)[1 + 2 * NS][4], double& v,
                                         Sum2* q) {
    for (int i = threadIdx.x;;) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v += o[0][u];
#pragma unroll
            for (int k = 0; k < NS; ++k) q[k] = q[k] + Sum2{o[1 + 2 * k][u], o[2 + 2 * k][u]};
        }
        if ((i += 4 * REDUCE_THREADS) >= np) break;
        load_partials<1 + 2 * NS>(part, np, i, o);
    }
}

// stop test of |r_k|^2, k >= 1
__device__ __forceinline__ int cr_stop(double rr, double tol2) {
    return !isfinite(rr) ? CR_NAN : (rr <= tol2 ? CR_CONVERGED : CR_RUN);
}

// Step `step` (1, 2, ... since the start), after Ar = H r and its inner products
// (dpart: DOT_ROWS rows of ndot partials):
//   p = r + beta p, Ap = Ar + beta Ap, r -= alpha Ap  (step 1: p = r, Ap = Ar),
// every second step x += alpha_old p_old + alpha p.  uin / uout: partials of |r|^2
// and |Ap|^2 (hi, lo) of the previous and of this step.  slot: place of the previous
// step's |r|^2 in the batch's history, or -1.
// Bound by the 7 or 9 vectors it streams (24^4 x 16: 1.46 and 1.77 ms, 4.9 and 5.2 TB/s),
// and on small lattices by the start: with the apply a step takes 37.4 us at 8^4 x 16,
// 39.6 with the first elements loaded after the scalars (then 1024 workgroups with two
// elements in flight 43.2, 256 with four 39.1, against these 512 with three).
template <bool FIRST, bool XUP>
__global__ void __launch_bounds__(REDUCE_THREADS) cr_step_kernel(int64_t n, double2* __restrict__ x,
                                                                 double2* __restrict__ r, double2* __restrict__ p,
                                                                 const double2* __restrict__ Ar,
                                                                 double2* __restrict__ Ap, const double* dpart, int ndot,
                                                                 const double* uin, double* uout, CrState* st, int step,
                                                                 int slot, double tol) {
    // the partials and the first elements are on their way before the scalars are known;
    // indices past the end repeat the last element, which is then not stored
    constexpr int U = 3;
    struct Batch {
        double2 r[U], ar[U], p[U], ap[U], x[U];
    };
    const int64_t stride = (int64_t)gridDim.x * REDUCE_THREADS;
    auto load = [&](int64_t i, Batch& b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = min(i + u * stride, n - 1);
            b.r[u] = r[k];
            b.ar[u] = Ar[k];
            b.p[u] = FIRST ? make_double2(0, 0) : p[k];
            b.ap[u] = FIRST ? make_double2(0, 0) : Ap[k];
            b.x[u] = XUP ? x[k] : make_double2(0, 0);
        }
    };
    double od[DOT_ROWS][4], ou[3][4];
    load_partials<DOT_ROWS>(dpart, ndot, (int)threadIdx.x, od);
    if constexpr (!FIRST) load_partials<3>(uin, (int)gridDim.x, (int)threadIdx.x, ou);
    int64_t i = (int64_t)blockIdx.x * REDUCE_THREADS + threadIdx.x;
    Batch cur;
    load(i, cur);
    __builtin_amdgcn_sched_barrier(0);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    const int before = st->reason[(step - 1) & 1];
    int* const reason = &st->reason[step & 1];
    if (before != CR_RUN) {
        if (lead) *reason = before;
        return;
    }
    double t[2] = {0.0, 0.0};                     // <r,Ar>, |r|^2
    Sum2 q[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};  // |Ar|^2, Re<Ap,Ar>, |Ap|^2 of the old Ap
    add_rows<2>(dpart, ndot, od, t[0], q);
    if constexpr (!FIRST) add_rows<1>(uin, (int)gridDim.x, ou, t[1], q + 2);
    wg_sums<2>(t);
    wg_sums2<3>(q);
    const double rr = FIRST ? st->S[S_RR0] : t[1], arar = q[0].hi + q[0].lo;
    if constexpr (!FIRST) {
        const int stop = cr_stop(rr, tol * tol * st->S[S_BB]);
        if (lead && slot >= 0) st->S[S_HIST + slot] = rr;
        if (stop != CR_RUN) {
            if (lead) *reason = stop;
            return;
        }
    }
    const double rar = t[0];
    // (near-)breakdown: <r,Ar> at rounding level of |r||Ar|
    if (!(fabs(rar) >= 1e-13 * sqrt(rr) * sqrt(arar))) {
        if (lead) *reason = isfinite(rar) ? CR_BREAKDOWN : CR_NAN;
        return;
    }
    const double beta = FIRST ? 0.0 : rar / st->S[S_RAR + ((step - 1) & 1)];
    const Sum2 e = add_scaled(add_scaled(q[0], 2.0 * beta, q[1]), beta, add_scaled(Sum2{0.0, 0.0}, beta, q[2]));
    const double apap = FIRST ? arar : e.hi + e.lo;
    // no step to take along p; r, p, Ap and x stay those of the step before
    if (!(apap > 0.0 && isfinite(apap))) {
        if (lead) *reason = isfinite(apap) ? CR_BREAKDOWN : CR_NAN;
        return;
    }
    const double alpha = rar / apap, aold = XUP ? st->S[S_ALPHA + ((step - 1) & 1)] : 0.0;
    double v[1] = {0.0};
    Sum2 an[1] = {{0.0, 0.0}};
    auto element = [&](int64_t i, double2 ri, double2 ari, double2 po, double2 apo, double2 xi) {
        double2 pi = ri, api = ari;
        if constexpr (!FIRST) {
            pi.x = fma(beta, po.x, ri.x);
            pi.y = fma(beta, po.y, ri.y);
            api.x = fma(beta, apo.x, ari.x);
            api.y = fma(beta, apo.y, ari.y);
        }
        if constexpr (XUP) {
            xi.x = fma(alpha, pi.x, fma(aold, po.x, xi.x));
            xi.y = fma(alpha, pi.y, fma(aold, po.y, xi.y));
            x[i] = xi;
        }
        ri.x = fma(-alpha, api.x, ri.x);
        ri.y = fma(-alpha, api.y, ri.y);
        p[i] = pi;
        Ap[i] = api;
        r[i] = ri;
        v[0] += ri.x * ri.x + ri.y * ri.y;
        add_product(an[0], api.x, api.x);
        add_product(an[0], api.y, api.y);
    };
    while (i < n) {
        Batch next;
        load(i + U * stride, next);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + u * stride < n) element(i + u * stride, cur.r[u], cur.ar[u], cur.p[u], cur.ap[u], cur.x[u]);
        cur = next;
        i += U * stride;
    }
    wg_sums<1>(v);
    wg_sums2<1>(an);
    if (threadIdx.x == 0) {
        uout[blockIdx.x] = v[0];
        uout[gridDim.x + blockIdx.x] = an[0].hi;
        uout[2 * gridDim.x + blockIdx.x] = an[0].lo;
    }
    if (lead) {
        st->S[S_RAR + (step & 1)] = rar;
        st->S[S_ALPHA + (step & 1)] = alpha;
        st->steps = step;
    }
}

// |r|^2 after the last step of a batch, and its stop test
__global__ void __launch_bounds__(REDUCE_THREADS) cr_check_kernel(const double* uin, int nu, CrState* st, int step,
                                                                  int slot, double tol) {
    if (st->reason[step & 1] != CR_RUN) return;
    double t[1] = {0.0};
    add_partials<1>(uin, nu, t);
    wg_sums<1>(t);
    if (threadIdx.x == 0) {
        st->S[S_HIST + slot] = t[0];
        st->reason[step & 1] = cr_stop(t[0], tol * tol * st->S[S_BB]);  // one workgroup: all have read it
    }
}

// x += alpha p of an odd last step, which x has not taken yet
__global__ void __launch_bounds__(REDUCE_THREADS) cr_flush_kernel(int64_t n, double2* __restrict__ x,
                                                                  const double2* __restrict__ p, const CrState* st) {
    const double alpha = st->S[S_ALPHA + 1];
    const int64_t stride = (int64_t)gridDim.x * REDUCE_THREADS;
    for (int64_t i = (int64_t)blockIdx.x * REDUCE_THREADS + threadIdx.x; i < n; i += stride) {
        double2 xi = x[i];
        const double2 pi = p[i];
        xi.x = fma(alpha, pi.x, xi.x);
        xi.y = fma(alpha, pi.y, xi.y);
        x[i] = xi;
    }
}

// the workgroup's sums to its column of DOT_ROWS rows
__device__ __forceinline__ void store_dots(double* __restrict__ part, double (&v)[1], Sum2 (&q)[2]) {
    wg_sums<1>(v);
    wg_sums2<2>(q);
    if (threadIdx.x == 0) {
        const double o[DOT_ROWS] = {v[0], q[0].hi, q[0].lo, q[1].hi, q[1].lo};
#pragma unroll
        for (int r = 0; r < DOT_ROWS; ++r) part[(size_t)r * gridDim.x + blockIdx.x] = o[r];
    }
}

// The apply's own partials (nin columns) summed into gridDim.x columns: a large
// lattice has more of them than every workgroup of the update can add up.
__global__ void __launch_bounds__(REDUCE_THREADS) cr_compress_kernel(const double* __restrict__ in, int nin,
                                                                     const CrState* __restrict__ st, int step,
                                                                     double* __restrict__ out) {
    if (st->reason[(step - 1) & 1] != CR_RUN) return;
    double v[1] = {0.0};
    Sum2 q[2] = {{0.0, 0.0}, {0.0, 0.0}};
    for (int i = blockIdx.x * REDUCE_THREADS + threadIdx.x; i < nin; i += gridDim.x * REDUCE_THREADS) {
        v[0] += in[i];
#pragma unroll
        for (int r = 0; r < 2; ++r)
            q[r] = q[r] + Sum2{in[(size_t)(1 + 2 * r) * nin + i], in[(size_t)(2 + 2 * r) * nin + i]};
    }
    store_dots(out, v, q);
}

// the inner products in a pass of their own, for the applies that do not take them
template <bool FIRST>
__global__ void __launch_bounds__(REDUCE_THREADS) cr_dots_kernel(int64_t n, const double2* __restrict__ r,
                                                                 const double2* __restrict__ Ar,
                                                                 const double2* __restrict__ Ap,
                                                                 const CrState* __restrict__ st, int step,
                                                                 double* __restrict__ dpart) {
    if (st->reason[(step - 1) & 1] != CR_RUN) return;
    double v[1] = {0.0};
    Sum2 q[2] = {{0.0, 0.0}, {0.0, 0.0}};
    const int64_t stride = (int64_t)gridDim.x * REDUCE_THREADS;
    auto element = [&](double2 a, double2 b, double2 c) {
        v[0] += a.x * b.x + a.y * b.y;
        add_product(q[0], b.x, b.x);
        add_product(q[0], b.y, b.y);
        if constexpr (!FIRST) {
            add_product(q[1], c.x, b.x);
            add_product(q[1], c.y, b.y);
        }
    };
    const double2 zero = make_double2(0, 0);
    int64_t i = (int64_t)blockIdx.x * REDUCE_THREADS + threadIdx.x;
    for (; i + stride < n; i += 2 * stride) {
        const double2 a0 = r[i], b0 = Ar[i], c0 = FIRST ? zero : Ap[i];
        const double2 a1 = r[i + stride], b1 = Ar[i + stride], c1 = FIRST ? zero : Ap[i + stride];
        element(a0, b0, c0);
        element(a1, b1, c1);
    }
    if (i < n) element(r[i], Ar[i], FIRST ? zero : Ap[i]);
    store_dots(dpart, v, q);
}

// r = b - Hx; partial |r|^2 (row 0) and |b|^2 (row 1)
__global__ void __launch_bounds__(REDUCE_THREADS) residual_kernel(int64_t n, const double2* __restrict__ b,
                                                                  const double2* __restrict__ Hx,
                                                                  double2* __restrict__ r,
                                                                  double* __restrict__ part) {
    double v[2] = {0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * REDUCE_THREADS;
#pragma unroll 2
    for (int64_t i = (int64_t)blockIdx.x * REDUCE_THREADS + threadIdx.x; i < n; i += stride) {
        const double2 bi = b[i], hi = Hx[i];
        const double2 ri = make_double2(bi.x - hi.x, bi.y - hi.y);
        r[i] = ri;
        v[0] += ri.x * ri.x + ri.y * ri.y;
        v[1] += bi.x * bi.x + bi.y * bi.y;
    }
    wg_sums<2>(v);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = v[0];
        part[gridDim.x + blockIdx.x] = v[1];
    }
}

// start of the iteration: |r|^2 and |b|^2 from residual_kernel, flags cleared
__global__ void __launch_bounds__(REDUCE_THREADS) cr_start_kernel(const double* part, int np, CrState* st) {
    double t[2] = {0.0, 0.0};
    add_partials<2>(part, np, t);
    wg_sums<2>(t);
    if (threadIdx.x == 0) {
        st->S[S_RR0] = t[0];
        st->S[S_BB] = t[1];
        st->reason[0] = st->reason[1] = CR_RUN;
        st->steps = 0;
    }
}

struct CrBuffers {
    double2 *r, *p, *Ar, *Ap;
    double* dpart;     // DOT_ROWS rows
    double* apart;     // the same of the apply's own partials, where there are more than REDUCE_BLOCKS
    double* upart[2];  // 3 rows each
    CrState* st;
};
CrBuffers cr_carve(Carver& c, const FineGeom& g) {
    const size_t n = (size_t)12 * g.N5;
    CrBuffers w;
    w.r = c.take<double2>(n);
    w.p = c.take<double2>(n);
    w.Ar = c.take<double2>(n);
    w.Ap = c.take<double2>(n);
    w.dpart = c.take<double>(DOT_ROWS * REDUCE_BLOCKS);
    const int nd = dslash_dots_blocks(g);
    w.apart = c.take<double>(nd > REDUCE_BLOCKS ? (size_t)DOT_ROWS * nd : 0);
    for (int i = 0; i < 2; ++i) w.upart[i] = c.take<double>(3 * CR_BLOCKS);
    w.st = c.take<CrState>(1);
    return w;
}

}  // namespace

size_t cr_workspace_bytes(const FineGeom& g) {
    Carver c(nullptr, 0);
    cr_carve(c, g);
    return c.used();
}

int cr_solve(const FineGeom& g, const hdcr_solve_params* prm, const double2* U, const double2* b, double2* x,
             hdcr_solve_stats* st, double* history, int hcap, void* work, size_t work_bytes, hipStream_t s) {
    const auto t0 = std::chrono::steady_clock::now();
    const int64_t n = 12LL * g.N5;
    Carver c(work, work_bytes);
    const CrBuffers w = cr_carve(c, g);
    if (!c.ok()) return fail(HDCR_ENOMEM, "hdcr_solve: workspace too small for CR");

    // three or more elements per work-item, at most CR_BLOCKS workgroups
    const int64_t want = (n + 3 * REDUCE_THREADS - 1) / (3 * REDUCE_THREADS);
    const int nwg = (int)std::min<int64_t>(want < 1 ? 1 : want, CR_BLOCKS);
    const dim3 rg(nwg), rt(REDUCE_THREADS);
    const int ndots = dslash_dots_blocks(g);  // partials of the apply that takes the inner products with it
    CrState h;
    auto read = [&]() -> hipError_t {
        hipError_t e = hipMemcpyAsync(&h, w.st, sizeof(h), hipMemcpyDeviceToHost, s);
        if (e != hipSuccess) return e;
        return hipStreamSynchronize(s);
    };
    int64_t napply = 0;
    // r = b - H x, |r|^2, |b|^2
    auto true_residual = [&]() -> hipError_t {
        launch_dslash<double>(g, U, x, w.Ar, s);
        ++napply;
        hipLaunchKernelGGL(residual_kernel, rg, rt, 0, s, n, b, w.Ar, w.r, w.dpart);
        hipLaunchKernelGGL(cr_start_kernel, dim3(1), rt, 0, s, (const double*)w.dpart, nwg, w.st);
        return read();
    };

    HDCR_HIP_CHECK(true_residual());
    const double bb = h.S[S_BB];
    const double tol2 = prm->tol * prm->tol * bb;
    int status = HDCR_ENOTCONV;
    int it = 0;
    int hl = 0;
    double rr = h.S[S_RR0];
    if (bb == 0.0) {
        HDCR_HIP_CHECK(hipMemsetAsync(x, 0, n * sizeof(double2), s));
        HDCR_HIP_CHECK(hipStreamSynchronize(s));
        status = HDCR_OK;
        rr = 0.0;
    } else if (!std::isfinite(rr) || !std::isfinite(bb)) {
        status = HDCR_ENAN;
    } else if (rr <= tol2) {
        status = HDCR_OK;
    }
    // Steps behind the stop cost an application of H each, and a read-back some 25 us with
    // the GPU idle.  Where a step is longer than ten of those, a batch is two steps at first,
    // a quarter of the steps so far later, and ends by the rate of all of them, which a few
    // steps do not give (24^4 x 16, to 0.9 |b|, two steps: 7.6 ms, eight in the first batch 12.9;
    // to 0.01 |b|: 114.4 ms, by the last batch's rate 120.7).
    const bool long_steps = g.N5 >= 1 << 19;
    bool fresh = true;  // r is the true residual of x
    while (status == HDCR_ENOTCONV && it < prm->maxiter) {
        // steps from the residual in r, in batches
        int step = 0, reason = CR_RUN, batch = long_steps ? 2 : 8;
        const int nd = ndots > REDUCE_BLOCKS ? CR_COMPRESS : (ndots > 0 ? ndots : nwg);  // rows of dpart past step 1
        const double rr0 = rr;
        while (reason == CR_RUN && it < prm->maxiter) {
            const int done = step;
            const int nb = std::min(batch, prm->maxiter - it);
            for (int k = 0; k < nb; ++k) {
                ++step;
                ++napply;  // those past the stop run too
                const double* uin = w.upart[(step - 1) & 1];
                double* uout = w.upart[step & 1];
                const int slot = k > 0 ? k - 1 : -1;
#define HDCR_CR_STEP(F, XU)                                                                                        \
    hipLaunchKernelGGL((cr_step_kernel<F, XU>), rg, rt, 0, s, n, x, w.r, w.p, (const double2*)w.Ar, w.Ap,          \
                   (const double*)w.dpart, step == 1 ? nwg : nd, uin, uout, w.st, step, slot, prm->tol)
                if (step == 1) {
                    launch_dslash<double>(g, U, w.r, w.Ar, s);
                    hipLaunchKernelGGL(cr_dots_kernel<true>, rg, rt, 0, s, n, w.r, w.Ar, w.Ap, w.st, step, w.dpart);
                    HDCR_CR_STEP(true, false);
                    continue;
                }
                if (ndots > REDUCE_BLOCKS) {
                    launch_dslash_dots(g, U, w.r, w.Ar, w.Ap, w.apart, s);
                    hipLaunchKernelGGL(cr_compress_kernel, dim3(CR_COMPRESS), rt, 0, s, (const double*)w.apart, ndots,
                                       w.st, step, w.dpart);
                } else if (ndots > 0) {
                    launch_dslash_dots(g, U, w.r, w.Ar, w.Ap, w.dpart, s);
                } else {
                    launch_dslash<double>(g, U, w.r, w.Ar, s);
                    hipLaunchKernelGGL(cr_dots_kernel<false>, rg, rt, 0, s, n, w.r, w.Ar, w.Ap, w.st, step,
                                       w.dpart);
                }
                if (step % 2 == 0)
                    HDCR_CR_STEP(false, true);
                else
                    HDCR_CR_STEP(false, false);
#undef HDCR_CR_STEP
            }
            hipLaunchKernelGGL(cr_check_kernel, dim3(1), rt, 0, s, (const double*)w.upart[step & 1], nwg, w.st, step,
                               nb - 1, prm->tol);
            HDCR_HIP_CHECK(read());
            reason = h.reason[step & 1];
            step = h.steps;
            const int did = step - done;
            for (int k = 0; k < did; ++k)
                if (history && hl < hcap) history[hl++] = std::sqrt(h.S[S_HIST + k] / bb);
            const double before = rr;
            if (did > 0) rr = h.S[S_HIST + did - 1];
            it += did;
            // the next batch: half the steps that the rate predicts
            batch = CR_BATCH;
            const double from = long_steps ? rr0 : before;
            if (did > 0 && rr < from) {
                const double left = std::log(rr / tol2) / std::log(from / rr) * (long_steps ? step : did);
                if (left < 2.0 * CR_BATCH) batch = std::max(long_steps ? 1 : 4, (int)(0.5 * left));
            }
            if (long_steps) batch = std::min(batch, std::max(2, step / 4));
        }
        if (step % 2 == 1) hipLaunchKernelGGL(cr_flush_kernel, rg, rt, 0, s, n, x, (const double2*)w.p, w.st);
        fresh = false;
        if (reason == CR_BREAKDOWN) status = HDCR_EBREAKDOWN;
        if (reason == CR_NAN) status = HDCR_ENAN;
        if (reason != CR_CONVERGED) break;
        HDCR_HIP_CHECK(true_residual());
        rr = h.S[S_RR0];
        fresh = true;
        if (rr <= tol2) status = HDCR_OK;
    }
    // final true residual (also when not converged)
    if (!fresh || bb == 0.0) HDCR_HIP_CHECK(true_residual());
    HDCR_HIP_CHECK(hipGetLastError());
    const double t = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (st) {
        st->status = status;
        st->outer_iters = it;
        st->coarse_iters = 0;
        st->fine_applies_f64 = napply;
        st->fine_applies_inner = 0;
        st->coarse_applies = 0;
        st->true_rel_residual = bb > 0 ? std::sqrt(h.S[S_RR0] / bb) : 0.0;
        st->seconds_total = t;
        st->seconds_fine = 0;
        st->seconds_coarse = 0;
        st->seconds_outer = t;
        st->history_len = hl;
    }
    return status;
}

}  // namespace hdcr
