// Newton driver (Sec. 2.4.2, 2.5, App. A, App. B) as a per-instance state
// machine, and the scheduler that advances any number of instances together:
// every instance runs until it needs a linear solve, then one batched GMRES
// (gmres_batched.hip) serves all of them.  A single solve is a batch of one.
//
// Newton: Phi = Phi_L + Phi_NL, c = b - A Phi, d = c - N(u); solve
// (A + J) Delta = d; Phi_NL += omega Delta; stop when omega ||Delta||_2 <
// Tol_NL.  The first step uses the cubic Taylor scheme (T3), later steps
// sinh (HS), unless a schedule of Taylor orders is given (T3-T5-HS and the
// like of Sec. 3.3.1).  omega is the root of f_d (eq. fd=0) found by Newton's method
// with the derivative of App. A (second derivative r'' = -H[Delta], the
// minus sign the printed formula drops), started at 2 in the T3 step and 1
// afterwards, each iterate clamped to [omega_min, omega_max]; it is frozen
// once e_k < L_e, and the GMRES tolerance is tightened tenfold per step once
// e_k < 1250 tol (App. B).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <thread>

#include "pbfb_internal.hpp"

namespace pbfb {

static inline unsigned nbk(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

// sums over the 256 threads of a workgroup, valid in thread 0
template <int K> __device__ inline void block_sums(double (&v)[K])
{
    __shared__ double red[4][K];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o);
        if (lane == 0) red[wv][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = (red[0][k] + red[1][k]) + (red[2][k] + red[3][k]);
}

// Inverse diagonal of the Newton matrix (diag(A + J) on the FEM rows, the
// diagonals of the signed single layers on the surface rows), and the
// Gershgorin bound of diag(F)^-1 F for the FEM block F = A + J_N (the upper
// end of the Chebyshev interval) as one maximum per slice, which the batched
// solve reduces.  Workgroups of the slices, then 256 surface rows each.
__global__ void __launch_bounds__(256)
    k_diag_bound(int64_t nn, int64_t nm, int64_t n, int64_t nsl, const int32_t *__restrict__ sptr, SellLong lng,
                 const int32_t *__restrict__ col, const double *__restrict__ val, const int32_t *__restrict__ diag,
                 const double *__restrict__ vdm, const double *__restrict__ vds, double *__restrict__ dinv,
                 double *__restrict__ part)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t q = blockIdx.x;
    if (q >= nsl) {
        const int64_t i = nn + (q - nsl) * 256 + threadIdx.x;
        if (i < n) dinv[i] = 1.0 / (i < nn + nm ? vdm[i - nn] : vds[i - nn - nm]);
        return;
    }
    const int64_t i = q * SLICE + lane;
    const int32_t b0 = sptr[q], w = (sptr[q + 1] - b0) / SLICE;
    double sum = 0.0; // slice padding adds zeros
    for (int32_t k = wv; k < w; k += SELL_W) {
        const int64_t e = b0 + int64_t(SLICE) * k + lane;
        if (col[e] < nn) sum += fabs(val[e]);
    }
    sum = sell_reduce(sum, lane, wv);
    if (lng.ptr) {
        __shared__ double red[SELL_W];
        for (int32_t l = lng.ptr[q]; l < lng.ptr[q + 1]; ++l) {
            double t = 0.0;
            for (int32_t e = lng.off[l] + int32_t(threadIdx.x); e < lng.off[l + 1]; e += 256)
                if (col[e] < nn) t += fabs(val[e]);
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
            if (lane == 0) red[wv] = t;
            __syncthreads();
            if (wv == 0 && i == lng.row[l]) sum = (red[0] + red[1]) + (red[2] + red[3]);
            __syncthreads();
        }
    }
    if (wv != 0) return;
    double v = 0.0;
    if (i < nn) {
        const double dg = val[diag[i]];
        dinv[i] = 1.0 / dg;
        v = sum / dg;
    }
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    if (lane == 0) part[q] = v;
}

enum RunPhase { PH_START = 0, PH_LINEAR = 1, PH_NEWTON = 2, PH_DONE = 3, PH_POST = 4 };
// PH_POST: back from a Newton linear solve, omega of the step set up (searched with the batch's)

// the linear-solve request of the current Newton matrix (its FEM values,
// diagonal and Chebyshev bound are computed here)
static GmresJob make_job(NewtonRun &r, const double *b, double *x, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n(), nsl = nbk(p.nn, SLICE);
    hipLaunchKernelGGL(k_diag_bound, dim3(unsigned(nsl) + nbk(n - p.nn, 256)), dim3(256), 0, s, p.nn, p.surf[0].nv, n,
                       nsl, p.d_sptr, p.fr.sell(), p.d_col, p.d_val, p.d_diag, p.surf[0].vdiag, p.surf[1].vdiag, r.dinv,
                       r.lmax);
    PB_HIP(hipGetLastError());
    GmresJob J{&p, b, x, r.dinv, r.tol, r.o.gmres_restart, r.o.max_gmres, 0, 0, r.o.krylov_fp32};
    J.pc = r.o.precond;
    J.cheb_k = r.o.cheb_degree;
    J.cheb_ratio = r.o.cheb_ratio;
    J.lmax = r.lmax;
    J.applies = 0;
    J.graph = r.o.hip_graph;
    return J;
}

NewtonRun::NewtonRun(Problem *p_, const pbfb_solve_opts &o_, pbfb_result *res_, double *out)
    : p(p_), o(o_), res(res_), phi_out_dev(out)
{
    *res = pbfb_result{};
    t0 = std::chrono::steady_clock::now(); // batch start / admission time
}

static void finish(NewtonRun &r, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n();
    double en[4] = {0, 0, 0, 0};
    if (r.phil) {
        energy(p, r.phil, r.phinl, en, s);
        if (r.phi_out_dev) {
            PB_HIP(hipMemcpyAsync(r.phi_out_dev, r.phil, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
            PB_HIP(hipMemcpyAsync(r.phi_out_dev + n, r.phinl, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
        }
    }
    PB_HIP(hipStreamSynchronize(s));
    auto t2 = std::chrono::steady_clock::now();
    r.res->total = en[0];
    r.res->lc = en[1];
    r.res->nc = en[2];
    r.res->dg_omega_i = en[3];
    r.res->newton_iters = r.k;
    r.res->status = pbfb_status(r.status);
    r.res->t_setup_s = std::chrono::duration<double>(r.t1 - r.t0).count();
    r.res->t_solve_s = std::chrono::duration<double>(t2 - r.t1).count();
    r.phase = PH_DONE;
}

// Newton pre-step: residual, Jacobian values, preconditioner, linear solve request
static void newton_pre(NewtonRun &r, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n();
    if (r.o.n_schedule > 0) r.sch = r.k <= r.o.n_schedule ? r.o.schedule[r.k - 1] : PBFB_HS;
    else r.sch = (r.k == 1 && r.o.scheme_first == PBFB_T3) ? PBFB_T3 : PBFB_HS;
    if (!r.c_ready) { // else c was carried over from the last step's omega search
        coupled_apply_linear(p, r.phi, r.c, s);
        vec_axpby(n, 1.0, p.d_b, -1.0, r.c, s);
        r.res->applies += 1; // c = b - A Phi
    }
    r.c_ready = false;
    // d = c - N; a residual that is not finite ends the linear solve with ENAN
    fem_nonlinear(p, r.sch, r.phi, r.c, -1.0, nullptr, r.d, s);
    // Newton: (A + J_N) Delta = d; Picard: A Delta = d
    if (r.o.nonlinear_method == PBFB_PICARD) fem_assemble_linear(p, s);
    else fem_assemble_jacobian(p, r.sch, r.phi, s);
    r.job = make_job(r, r.d, r.D, s);
}

// ---------------------------------------------------------------------------
// root of f_d (Sec. 2.5; the appendix on one-dimensional root finding and
// the first-iteration start of the appendix on other optimisations), on the
// device.  Every method stops at |f_d| < tol_omega or after max_omega_it
// evaluations; iterates are clamped to [omega_min, omega_max]; an undefined
// f_d (beta = 0) or a vanishing derivative / secant slope gives omega = 1.
//
// The search of one instance is a small state machine in device memory
// (OmegaSearch).  One evaluation round is four launches: the f_d terms at S.w
// per tet (the element kernel reads omega from S.w) and per node, the partial
// sums of their six dot products (which form the residual on the way), then
// k_omega_step, which adds them, forms f_d and f_d' and moves the state to the
// next point to evaluate or to its result, leaving what the host asks for in
// pinned memory.  Once S.done is set the round's kernels return at once.  The
// host enqueues rounds for every searching instance of the batch and looks
// only every few rounds, one synchronisation for all of them.
// ---------------------------------------------------------------------------
enum OmPhase {
    OM_NEWTON = 0, // evaluating w of the Newton iteration
    OM_SEC_A,      // secant: the first point w0
    OM_SEC_B,      // secant: the second point / each new point w1
    OM_BIS_LO,     // bisection: the lower end
    OM_BIS_HI,     // bisection: the upper end
    OM_BIS_MID,    // bisection: a midpoint
    OM_BS_START,   // first-iteration start: the three midpoints of [2, 3]
    OM_BS_SEC,     // first-iteration start: its secant steps
    OM_DF          // direct secant through (0, 1): the point 1/8
};

struct OmegaSearch {
    // setup
    int method, k, max_it;
    double tol, wmin, wmax, omega0;
    double pp; // p.p of this step
    // state
    int phase, ev, done, si;
    double w; // the point of the next evaluation (the element kernel reads it)
    double lo, hi, flo, wstart;
    double w0, f0, w1, f1;
    double blo, bhi, bw[3], bf[3];
    double result;
};

__device__ inline double om_clamp(const OmegaSearch &S, double w) { return fmin(S.wmax, fmax(S.wmin, w)); }
__device__ inline void om_finish(OmegaSearch &S, double w)
{
    S.result = w;
    S.done = 1;
}
// Newton from w (the while condition of the iteration is checked first)
__device__ inline void om_newton_start(OmegaSearch &S, double w)
{
    if (S.ev >= S.max_it) return om_finish(S, w);
    S.phase = OM_NEWTON;
    S.w = w;
}
__device__ inline void om_bisect_start(OmegaSearch &S, double lo, double hi, double wstart)
{
    S.lo = lo;
    S.hi = hi;
    S.wstart = wstart;
    S.phase = OM_BIS_LO;
    S.w = lo;
}
__device__ inline void om_secant_start(OmegaSearch &S, double w0, double w1)
{
    S.w0 = w0;
    S.w1 = w1;
    S.phase = OM_SEC_A;
    S.w = w0;
}
// the secant loop of the first-iteration start, from (w0, f0), (w1, f1)
__device__ inline void om_bs_loop(OmegaSearch &S)
{
    if (S.ev >= S.max_it) return om_newton_start(S, S.w1);
    const double slope = S.f0 - S.f1;
    if (slope == 0.0 || !isfinite(slope)) return om_newton_start(S, S.w1);
    const double w2 = om_clamp(S, S.w0 - (S.w0 - S.w1) * S.f0 / slope);
    if (fabs(w2 - S.w1) < 0.05) return om_newton_start(S, w2);
    S.w0 = S.w1;
    S.f0 = S.f1;
    S.w1 = w2;
    S.phase = OM_BS_SEC;
    S.w = w2;
}

// p = -A Delta from A Delta, and the partial sums of p.p
__global__ void __launch_bounds__(256) k_search_begin(int64_t n, double *__restrict__ pv, double *__restrict__ part)
{
    double t[1] = {0.0};
    for (int64_t i = blockIdx.x * int64_t(256) + threadIdx.x; i < n; i += int64_t(DOT_BLOCKS) * 256) {
        const double v = -pv[i];
        pv[i] = v;
        t[0] = fma(v, v, t[0]);
    }
    block_sums(t);
    if (threadIdx.x == 0) part[blockIdx.x] = t[0];
}

static_assert(DOT_BLOCKS == 256, "one partial per thread of the summing workgroup");
__global__ void __launch_bounds__(256) k_omega_init(OmegaSearch *__restrict__ S_, int method, int k, int max_it,
                                                    double tol, double wmin, double wmax, double omega0,
                                                    const double *__restrict__ part)
{
    double pp[1] = {part[threadIdx.x]};
    block_sums(pp);
    if (threadIdx.x != 0) return;
    OmegaSearch S{};
    S.pp = pp[0];
    S.method = method;
    S.k = k;
    S.max_it = max_it;
    S.tol = tol;
    S.wmin = wmin;
    S.wmax = wmax;
    S.omega0 = omega0;
    switch (method) {
    case PBFB_OMEGA_BISECT: om_bisect_start(S, wmin, wmax, omega0); break;
    case PBFB_OMEGA_SECANT: om_secant_start(S, omega0, omega0 + 0.125); break;
    case PBFB_OMEGA_BSEC:
        if (k == 1) om_bisect_start(S, wmin, wmax, omega0);
        else om_secant_start(S, omega0, omega0 + 0.125);
        break;
    case PBFB_OMEGA_NEWTON_BS:
        if (k == 1) {
            S.blo = 2.0;
            S.bhi = 3.0;
            S.si = 0;
            S.phase = OM_BS_START;
            S.w = 2.5;
        } else {
            om_newton_start(S, omega0);
        }
        break;
    case PBFB_OMEGA_BSEC_DF:
        if (k == 1) {
            om_bisect_start(S, wmin, wmax, omega0);
        } else {
            S.phase = OM_DF;
            S.w = 0.125;
        }
        break;
    default: om_newton_start(S, omega0); break;
    }
    *S_ = S;
}

// f_d and f_d' at S.w from the dot products (eq. fd=0 and its derivative,
// r' = -[rJ; 0; 0], r'' = -[rH; 0; 0]), then the next state
//
// six partial sums per block: p.r over all unknowns, then rJ.r, rJ.p, rJ.rJ,
// r.rH, p.rH over the FEM rows, with r = c - N
__global__ void __launch_bounds__(256)
    k_omega_dots(int64_t n, int64_t nn, const double *__restrict__ c, const double *__restrict__ pv,
                 const double *__restrict__ rN, const double *__restrict__ rJ, const double *__restrict__ rH,
                 double *__restrict__ part, const int *__restrict__ skip)
{
    if (*skip) return;
    double t[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t i = blockIdx.x * int64_t(256) + threadIdx.x; i < n; i += int64_t(DOT_BLOCKS) * 256) {
        const double p = pv[i];
        if (i >= nn) {
            t[0] = fma(p, c[i], t[0]);
            continue;
        }
        const double r = c[i] - rN[i], J = rJ[i], H = rH[i];
        t[0] = fma(p, r, t[0]);
        t[1] = fma(J, r, t[1]);
        t[2] = fma(J, p, t[2]);
        t[3] = fma(J, J, t[3]);
        t[4] = fma(r, H, t[4]);
        t[5] = fma(p, H, t[5]);
    }
    block_sums(t);
    if (threadIdx.x == 0)
        for (int k = 0; k < 6; ++k) part[6 * blockIdx.x + k] = t[k];
}

// host: done, omega, evaluations (pinned)
__device__ inline void om_next(OmegaSearch &S, const double (&v)[6]);
__global__ void __launch_bounds__(256) k_omega_step(OmegaSearch *__restrict__ S_, const double *__restrict__ part,
                                                    double *__restrict__ host)
{
    if (S_->done) return;
    double v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = part[6 * threadIdx.x + k];
    block_sums(v);
    if (threadIdx.x != 0) return;
    OmegaSearch S = *S_;
    om_next(S, v);
    *S_ = S;
    host[0] = S.done;
    host[1] = S.result;
    host[2] = S.ev;
}

__device__ inline void om_next(OmegaSearch &S, const double (&v)[6])
{
    const double w = S.w;
    const double a = v[0] - v[1];     // (p + r').r
    const double beta = S.pp - v[2];  // (p + r').p
    const bool ok = beta != 0.0;
    double fd = 0.0, dfd = 0.0;
    if (ok) {
        fd = -a / beta - w;
        dfd = -(-v[2] + v[3] - v[4]) / beta + a * (-v[5]) / (beta * beta) - 1.0;
    }
    ++S.ev;
    if (!ok) return om_finish(S, 1.0);
    switch (S.phase) {
    case OM_NEWTON:
        if (fabs(fd) < S.tol) om_finish(S, w);
        else if (dfd == 0.0 || !isfinite(dfd)) om_finish(S, 1.0);
        else {
            const double wn = om_clamp(S, w - fd / dfd);
            if (S.ev >= S.max_it) om_finish(S, wn);
            else S.w = wn;
        }
        break;
    case OM_SEC_A:
        if (fabs(fd) < S.tol) {
            om_finish(S, w);
        } else {
            S.f0 = fd;
            S.phase = OM_SEC_B;
            S.w = S.w1;
        }
        break;
    case OM_SEC_B:
        S.f1 = fd;
        if (fabs(S.f1) >= S.tol && S.ev < S.max_it) {
            const double slope = S.f0 - S.f1;
            if (slope == 0.0 || !isfinite(slope)) {
                om_finish(S, 1.0);
            } else {
                const double w2 = om_clamp(S, S.w0 - (S.w0 - S.w1) * S.f0 / slope);
                S.w0 = S.w1;
                S.f0 = S.f1;
                S.w1 = w2;
                S.w = w2;
            }
        } else {
            om_finish(S, S.w1);
        }
        break;
    case OM_BIS_LO:
        if (fabs(fd) < S.tol) {
            om_finish(S, S.lo);
        } else {
            S.flo = fd;
            S.phase = OM_BIS_HI;
            S.w = S.hi;
        }
        break;
    case OM_BIS_HI:
        if (fabs(fd) < S.tol) om_finish(S, S.hi);
        else if ((S.flo > 0.0) == (fd > 0.0)) om_newton_start(S, S.wstart); // no sign change over the interval
        else if (S.ev >= S.max_it) om_finish(S, 0.5 * (S.lo + S.hi));
        else {
            S.phase = OM_BIS_MID;
            S.w = 0.5 * (S.lo + S.hi);
        }
        break;
    case OM_BIS_MID:
        if (fabs(fd) < S.tol) {
            om_finish(S, w);
        } else {
            if ((fd > 0.0) == (S.flo > 0.0)) {
                S.lo = w;
                S.flo = fd;
            } else {
                S.hi = w;
            }
            if (S.ev < S.max_it) S.w = 0.5 * (S.lo + S.hi);
            else om_finish(S, w);
        }
        break;
    case OM_BS_START:
        S.bw[S.si] = w;
        S.bf[S.si] = fd;
        if (fd > 0.0) S.blo = w;
        else S.bhi = w;
        ++S.si;
        if (S.si < 3) {
            S.w = 0.5 * (S.blo + S.bhi);
        } else {
            S.w0 = S.bw[1];
            S.f0 = S.bf[1];
            S.w1 = S.bw[2];
            S.f1 = S.bf[2];
            om_bs_loop(S);
        }
        break;
    case OM_BS_SEC:
        S.f1 = fd;
        om_bs_loop(S);
        break;
    case OM_DF:
        if (fd == 1.0 || !isfinite(fd)) om_finish(S, 1.0);
        else om_finish(S, om_clamp(S, 0.125 / (1.0 - fd)));
        break;
    default: om_finish(S, 1.0); break;
    }
}

static OmegaSearch *om_state(NewtonRun &r) { return static_cast<OmegaSearch *>(r.om_dev); }

// one evaluation round of a search; host: its three pinned words
static void omega_round(NewtonRun &r, double *host, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n(), nn = p.nn;
    OmegaSearch *S = om_state(r);
    const int *skip = &S->done;
    double *part = dot_partials(p);
    fem_omega_terms_dev(p, r.sch, r.phi, r.D, &S->w, skip, r.rN, r.rJ, r.rH, s);
    hipLaunchKernelGGL(k_omega_dots, dim3(DOT_BLOCKS), dim3(256), 0, s, n, nn, r.c, r.pv, r.rN, r.rJ, r.rH, part, skip);
    hipLaunchKernelGGL(k_omega_step, dim3(1), dim3(256), 0, s, S, part, host);
    PB_HIP(hipGetLastError());
}

// the searches of all runs in `srch` together: rounds for every run whose
// search is not known to be done, looked at every few rounds
static void omega_search_all(std::vector<NewtonRun *> &srch, hipStream_t s)
{
    constexpr int ROUNDS = 2; // evaluation rounds between two host checks
    std::vector<NewtonRun *> act = srch;
    while (!act.empty()) {
        double *host = pinned_doubles(3 * act.size());
        for (size_t i = 0; i < act.size(); ++i) host[3 * i] = 0.0;
        for (int q = 0; q < ROUNDS; ++q)
            for (size_t i = 0; i < act.size(); ++i) omega_round(*act[i], host + 3 * i, s);
        PB_HIP(hipStreamSynchronize(s));
        std::vector<NewtonRun *> next;
        for (size_t i = 0; i < act.size(); ++i) {
            NewtonRun *r = act[i];
            if (host[3 * i] != 0.0) {
                r->omega = host[3 * i + 1];
                r->evals = int(host[3 * i + 2]);
                r->searching = false;
            } else {
                next.push_back(r);
            }
        }
        act.swap(next);
    }
}

// omega of this step: fixed, frozen, reused (Picard) or searched.  A search
// is set up here (p = -A Delta, p.p into the device state) and run later
// together with the other instances' (omega_search_all).
static void newton_post_begin(NewtonRun &r, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n();
    const pbfb_solve_opts &o = r.o;
    r.searching = r.searched = false;
    if (!o.omega_auto) {
        r.omega = o.omega_fixed;
    } else if (r.frozen) {
        r.omega = r.omega_last;
    } else if (o.nonlinear_method == PBFB_PICARD && o.r_e > 0 && r.k >= 3 && r.e_km2 >= o.r_e * r.e_km1) {
        r.omega = r.omega_last; // e_{k-2} / e_{k-1} >= R_e: converging fast enough, reuse
    } else {
        const double omega0 = r.sch == PBFB_T3 ? o.omega0_first : o.omega0_next;
        // p = -A Delta
        coupled_apply_linear(p, r.D, r.pv, s);
        r.res->applies += 1;
        r.searched = r.searching = true;
        r.om_dev = scratch<double>(p, SCR_OMEGA, sizeof(OmegaSearch) / 8 + 8);
        double *part = dot_partials(p);
        hipLaunchKernelGGL(k_search_begin, dim3(DOT_BLOCKS), dim3(256), 0, s, n, r.pv, part);
        hipLaunchKernelGGL(k_omega_init, dim3(1), dim3(256), 0, s, om_state(r), o.omega_method, r.k, o.max_omega_it,
                           o.tol_omega, o.omega_min, o.omega_max, omega0, part);
        PB_HIP(hipGetLastError());
    }
}

// Phi_NL += omega Delta, Phi = Phi_L + Phi_NL, after a search also the next
// c = b - A Phi without an apply (A (Phi + omega Delta) = A Phi - omega p),
// and the partial sums of Delta.Delta
__global__ void __launch_bounds__(256)
    k_newton_update(int64_t n, double omega, const double *__restrict__ D, const double *__restrict__ pv,
                    const double *__restrict__ phil, double *__restrict__ phinl, double *__restrict__ phi,
                    double *__restrict__ c, double *__restrict__ part)
{
    double t[1] = {0.0};
    for (int64_t i = blockIdx.x * int64_t(256) + threadIdx.x; i < n; i += int64_t(DOT_BLOCKS) * 256) {
        const double dv = D[i], u = fma(omega, dv, phinl[i]);
        phinl[i] = u;
        phi[i] = phil[i] + u;
        if (pv) c[i] = fma(omega, pv[i], c[i]);
        t[0] = fma(dv, dv, t[0]);
    }
    block_sums(t);
    if (threadIdx.x == 0) part[blockIdx.x] = t[0];
}
__global__ void __launch_bounds__(256) k_partials_sum(const double *__restrict__ part, double *__restrict__ out)
{
    double t[1] = {part[threadIdx.x]};
    block_sums(t);
    if (threadIdx.x == 0) *out = t[0];
}

// the update of a step whose omega is known; Delta.Delta goes to the pinned word
static void newton_post_update(NewtonRun &r, double *host, hipStream_t s)
{
    Problem &p = *r.p;
    double *part = dot_partials(p);
    hipLaunchKernelGGL(k_newton_update, dim3(DOT_BLOCKS), dim3(256), 0, s, p.n(), r.omega, r.D,
                       r.searched ? r.pv : (const double *)nullptr, r.phil, r.phinl, r.phi, r.c, part);
    hipLaunchKernelGGL(k_partials_sum, dim3(1), dim3(256), 0, s, part, host);
    PB_HIP(hipGetLastError());
}

// stop test after the update; true when converged
static bool newton_post_end(NewtonRun &r)
{
    const pbfb_solve_opts &o = r.o;
    const int idx = std::min(r.k - 1, 63);
    const double omega = r.omega;
    int oit = 0;
    if (r.searched) {
        oit = r.evals > 0 ? r.evals - 1 : 0;
        r.omega_last = omega;
        r.c_ready = true;
    }
    const double ek = omega * std::sqrt(r.dd);
    r.res->omega[idx] = omega;
    r.res->e_k[idx] = ek;
    r.res->omega_iters[idx] = oit;
    r.e_km2 = r.e_km1;
    r.e_km1 = ek;
    if (!std::isfinite(ek)) {
        r.status = PBFB_ENAN;
        return true;
    }
    if (o.l_e > 0 && ek < o.l_e) r.frozen = true;
    if (o.tol_gr0 > o.tol_gr && ek < 1250.0 * r.tol) r.tol = std::max(o.tol_gr, 0.1 * r.tol);
    // only a sinh step ends the iteration: a Taylor step solves another equation
    if (ek < o.tol_nl && r.sch == PBFB_HS) return true;
    if (r.k >= o.max_newton) {
        r.status = PBFB_ENOTCONV;
        return true;
    }
    return false;
}

// Advance one instance until it needs a linear solve (returns true) or is done.
static bool advance_impl(NewtonRun &r, hipStream_t s)
{
    Problem &p = *r.p;
    const int64_t n = p.n(), nn = p.nn;
    if (r.phase == PH_START) {
        ensure_all(p, s);
        PB_HIP(hipStreamSynchronize(s));
        r.t1 = std::chrono::steady_clock::now();
        r.phil = scratch<double>(p, SCR_G3, n);
        r.phinl = scratch<double>(p, SCR_G4, n);
        r.phi = scratch<double>(p, SCR_G5, n);
        r.c = scratch<double>(p, SCR_G6, n);
        r.d = scratch<double>(p, SCR_G7, n);
        r.D = scratch<double>(p, SCR_G8, n);
        r.pv = scratch<double>(p, SCR_G9, n);
        double *t3 = scratch<double>(p, SCR_G11, 3 * nn);
        r.rN = t3;
        r.rJ = t3 + nn;
        r.rH = t3 + 2 * nn;
        r.dinv = scratch<double>(p, SCR_G2, n);
        r.tol = r.o.tol_gr0;
        PB_HIP(hipMemsetAsync(r.phinl, 0, sizeof(double) * n, s));
        // linear component: (A + eps_s kappa^2 M) Phi_L = b
        r.lmax = scratch<double>(p, SCR_LMAX, nbk(nn, SLICE));
        fem_assemble_jacobian(p, PBFB_LIN, r.phinl, s);
        r.job = make_job(r, p.d_b, r.phil, s);
        r.phase = PH_LINEAR;
        return true;
    }
    if (r.phase == PH_LINEAR) {
        r.res->gmres_lin = r.job.iters;
        r.res->gmres_iters_total = r.job.iters;
        r.res->applies += r.job.applies;
        if (r.job.status) {
            r.status = r.job.status;
            finish(r, s);
            return false;
        }
        r.k = 1;
        // Phi = Phi_L (Phi_NL = 0); newton_post_update keeps it from here on
        PB_HIP(hipMemcpyAsync(r.phi, r.phil, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
        r.phase = PH_NEWTON;
        newton_pre(r, s);
        return true;
    }
    if (r.phase == PH_NEWTON) {
        const int idx = std::min(r.k - 1, 63);
        r.res->gmres_iters[idx] = r.job.iters;
        r.res->gmres_iters_total += r.job.iters;
        r.res->applies += r.job.applies;
        if (r.job.status) {
            r.status = r.job.status;
            finish(r, s);
            return false;
        }
        newton_post_begin(r, s);
        r.phase = PH_POST; // the search (if any) runs with the other instances'
        return false;
    }
    if (r.phase == PH_POST) {
        if (newton_post_end(r)) {
            finish(r, s);
            return false;
        }
        ++r.k;
        r.phase = PH_NEWTON;
        newton_pre(r, s);
        return true;
    }
    return false;
}

bool advance(NewtonRun &r, hipStream_t s)
{
    try {
        return advance_impl(r, s);
    } catch (const Error &e) {
        r.status = e.code;
        r.message = e.msg;
        r.res->status = e.code;
        r.phase = PH_DONE;
        return false;
    }
}

// Device setup (geometry, load, operators) of the runs that have not
// started, on up to N_ASM_WS host threads with a stream of the context each:
// the assembly kernels of a small instance leave most of the GPU idle, and
// several instances at once fill it.  Each run's state machine then finds its
// operators ready.  An error ends that run with its code.
static void parallel_setup(std::vector<NewtonRun *> &fresh, hipStream_t s)
{
    Ctx *C = fresh[0]->p->ctx;
    for (NewtonRun *r : fresh)
        if (r->p->ctx != C) return; // the streams and workspaces are the context's
    const int nt = int(std::min<size_t>(N_ASM_WS, fresh.size()));
    PB_HIP(hipStreamSynchronize(s)); // work the caller enqueued before the solve is complete
    {
        std::lock_guard<std::mutex> lk(C->setup_mu);
        for (int t = 0; t < nt; ++t)
            if (!C->setup_stream[t]) PB_HIP(hipStreamCreateWithFlags(&C->setup_stream[t], hipStreamNonBlocking));
    }
    std::atomic<size_t> next{0};
    std::vector<std::thread> th;
    for (int t = 0; t < nt; ++t)
        th.emplace_back([&, t] {
            const bool dev_ok = hipSetDevice(C->device) == hipSuccess;
            for (size_t i; (i = next++) < fresh.size();) {
                NewtonRun &r = *fresh[i];
                try {
                    PB_CHECK(dev_ok, PBFB_EDEVICE, "hipSetDevice failed in the setup thread");
                    ensure_all(*r.p, C->setup_stream[t]);
                    PB_HIP(hipStreamSynchronize(C->setup_stream[t]));
                } catch (const Error &e) {
                    r.status = e.code;
                    r.message = e.msg;
                    r.res->status = e.code;
                    r.phase = PH_DONE;
                }
            }
        });
    for (std::thread &x : th) x.join();
}

void advance_all(std::vector<NewtonRun *> &runs, std::vector<GmresJob *> &jobs, std::vector<NewtonRun *> *finished,
                 hipStream_t s)
{
    std::vector<NewtonRun *> fresh;
    for (NewtonRun *r : runs)
        if (r->phase == PH_START) fresh.push_back(r);
    if (fresh.size() > 1) parallel_setup(fresh, s);
    for (NewtonRun *r : fresh)
        if (r->phase == PH_DONE && finished) finished->push_back(r);
    auto step = [&](NewtonRun *r) {
        if (advance(*r, s)) jobs.push_back(&r->job);
        else if (r->phase == PH_DONE && finished) finished->push_back(r);
    };
    for (NewtonRun *r : runs)
        if (r->phase != PH_DONE && r->phase != PH_POST) step(r);
    // relaxation searches of every instance between two linear solves, together
    std::vector<NewtonRun *> srch;
    for (NewtonRun *r : runs)
        if (r->phase == PH_POST && r->searching) srch.push_back(r);
    if (!srch.empty()) {
        try {
            omega_search_all(srch, s);
        } catch (const Error &e) {
            for (NewtonRun *r : srch) {
                r->status = e.code;
                r->message = e.msg;
                r->res->status = e.code;
                r->phase = PH_DONE;
                if (finished) finished->push_back(r);
            }
        }
    }
    // the updates of every instance, then one look at their norms
    std::vector<NewtonRun *> post;
    for (NewtonRun *r : runs)
        if (r->phase == PH_POST) post.push_back(r);
    if (!post.empty()) {
        try {
            double *host = pinned_doubles(post.size());
            for (size_t i = 0; i < post.size(); ++i) newton_post_update(*post[i], host + i, s);
            PB_HIP(hipStreamSynchronize(s));
            for (size_t i = 0; i < post.size(); ++i) post[i]->dd = host[i];
        } catch (const Error &e) {
            for (NewtonRun *r : post) {
                r->status = e.code;
                r->message = e.msg;
                r->res->status = e.code;
                r->phase = PH_DONE;
                if (finished) finished->push_back(r);
            }
            post.clear();
        }
    }
    for (NewtonRun *r : post) step(r);
}

void run_newton(std::vector<NewtonRun *> &runs, hipStream_t s)
{
    std::vector<GmresJob *> jobs;
    for (;;) {
        jobs.clear();
        advance_all(runs, jobs, nullptr, s);
        if (jobs.empty()) break;
        try {
            batched_gmres(jobs, s);
        } catch (const Error &e) {
            // a device error ends every instance of the batch with its code
            for (NewtonRun *r : runs)
                if (r->phase != PH_DONE) {
                    r->job.status = e.code;
                    r->message = e.msg;
                }
        }
    }
}

pbfb_status solve(Problem &p, const pbfb_solve_opts &o, pbfb_result &res, double *phi_out_dev, hipStream_t s)
{
    NewtonRun r(&p, o, &res, phi_out_dev);
    std::vector<NewtonRun *> runs{&r};
    run_newton(runs, s);
    if (!r.message.empty()) set_error(r.message);
    return res.status;
}

} // namespace pbfb
