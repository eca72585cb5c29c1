// Batched restarted GMRES with device-resident control.
//
// Every instance of a batch solves its own system J x = b (right
// preconditioned by the block diagonal, x0 = 0, classical Gram-Schmidt
// applied twice, Givens rotations), and all of them advance together: each
// kernel below takes a packed work list that covers every instance, so one
// launch per step serves the whole batch whatever the mesh sizes.  The Krylov
// scalars (Hessenberg column, rotations, residual estimate, restart and
// convergence decisions, triangular solve) live on the device in one wavefront
// per instance, so the host only enqueues steps, two ahead of a progress word
// in pinned memory; nothing waits on the host between steps.
//
// Per-instance state machine (P^-1 the right preconditioner):
//   INIT  -> w = b, V_0 = b/|b|, target = tol |b|              -> ARN (or DONE if b = 0)
//   ARN   -> z = P^-1 V_j, w = J z, CGS2, V_{j+1}, Givens       -> ARN; at convergence, restart
//            or limit y = H^{-1} g, t = V y                     -> RES (FIN: see GSt)
//   RES   -> x += P^-1 t, w = b - J x, beta = |w|: beta <= target -> DONE, else V_0 = w/beta -> ARN
//   FIN   -> x += P^-1 t                                        -> DONE
// which is the restarted GMRES of the oracle (true residual at every restart).
// P^-1 is either the inverse diagonal of J or the block preconditioner:
// Jacobi-scaled Chebyshev terms on the FEM block (one SpMV launch per term
// after the first two) and a sparse approximate inverse on each single-layer
// block.
//
// One Krylov step of the batch is k_bfirst (approximate inverse, the first
// two Chebyshev terms), k_bcheb per further term, k_bgemv, k_btail (second
// stage of the dense product and the FEM SpMV), k_bmdot, k_bmid, k_bend (the
// two Gram-Schmidt passes), k_bcontrol and k_bnext: 8 + (terms - 2) launches.
// A launch of a few hundred workgroups takes 2-4 us however little it does,
// so below about 20k triangles a step's time is its launch count; every
// kernel here therefore takes the neighbouring small passes in (the packing
// of the dense input into the last Chebyshev term, the coefficient sums into
// the pass that uses them, the norm into control, the scaling and t = V y
// into one).
//
// Mixed precision may store the basis in FP32 (products, projections, norms,
// Hessenberg, rotations, w and x stay FP64).  A restart cycle is then an
// FP32-basis inner solve for the correction of the current iterate, and the
// FP64 true residual b - J x that starts the next cycle is the outer
// iterative refinement: the tolerance is always decided on that residual.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <thread>
#include <utility>

#include "gemv_rows.hpp"
#include "pbfb_internal.hpp"
#include "sell_slice.hpp"

namespace pbfb {


struct GDesc {
    const void *Bm, *Bs;
    int64_t ldm, lds, nm, ns;
    int f32;  // operator values in FP32
    int vf32; // Krylov basis stored in FP32
    int two_field; // lambda_m is not an unknown (two-field form): identity row, no Gamma_m GEMV
    // symmetric use of the stored single layer, per surface: column partials, Delta rows
    int symm[2];
    void *symP[2]; // FP64 column partials
    const int32_t *dl_ptr[2], *dl_col[2];
    const double *dl_val[2];
    // operator index -> surface vertex (Morton vertex order of the stored
    // operators; matrix-free: ascending, null)
    const int32_t *mvm, *mvs;
    // FEM node -> surface vertex and surface vertex -> operator index (null: the same), per surface
    const int32_t *nvert[2], *minv[2];
    const int32_t *sptr, *col; // FEM rows, sliced ELL
    SellLong lng;              // its long rows
    const void *val;
    int64_t nn, n;
    const double *dinv;
    void *V; // (m + 1) x n basis, FP64 or FP32 (vf32)
    double *w, *xm, *xs, *x;
    const double *b;
    double *H, *cs, *sn, *g, *y, *h1, *h2, *part, *part2, *npart, *nrm;
    int64_t chb, nchb; // rows per Gram-Schmidt chunk, chunks
    double tol;
    int m, maxit;
    // preconditioner
    int pc, cheb_k;
    double cheb_ratio;
    const double *lmax;
    const int32_t *sp_ptr[2], *sp_col[2];
    const double *sp_val[2];
    double *z, *zb, *dk, *t; // P^-1 input (full), Chebyshev ping-pong buffer and direction, V y
    double *coef;            // Chebyshev coefficients: [0] = theta, [2s], [2s+1] = rho_s rho_{s-1}, 2 rho_s/delta
};

struct GState {
    int st, j, total, code, napply;
    double beta, target;
};

struct WItem {
    int inst, a;
    int64_t b; // no padding: lists are compared byte by byte
    // FEM slices: first stored entry and width.  A small launch is a chain of
    // dependent loads, about 0.2 us each: item -> state and descriptor -> values
    // and columns -> inputs, with nothing to wait for in between (offsets read
    // from sptr: 15.5 -> 15.1 ms per 1 280-triangle solve)
    int32_t e0 = 0, w = 0;
};

constexpr int CH = 256;      // rows per chunk: one per thread of a workgroup
constexpr int GROWS = GSYM; // GEMV rows per workgroup


__device__ inline bool applies(int st) { return st == G_ARN || st == G_RES; }

// basis entry V_i[k], widened to FP64
__device__ inline double vget(const GDesc &d, int64_t i, int64_t k)
{
    return d.vf32 ? double(static_cast<const float *>(d.V)[i * d.n + k]) : static_cast<const double *>(d.V)[i * d.n + k];
}
template <typename VT> __device__ inline const VT *vcol(const GDesc &d, int64_t i)
{
    return static_cast<const VT *>(d.V) + i * d.n;
}

// product of the FEM rows of a slice item with the input x(column), valid in wavefront 0
template <bool FEM_ONLY, typename XF>
__device__ inline double fem_rows(const GDesc &d, XF &&x, const WItem &it, int lane, int wv)
{
    const int64_t q = it.b / SLICE;
    return d.f32 ? sell_rows<float, FEM_ONLY>(it.e0, it.w, d.lng, d.col, static_cast<const float *>(d.val), x, q, lane,
                                              wv, d.nn)
                 : sell_rows<double, FEM_ONLY>(it.e0, it.w, d.lng, d.col, static_cast<const double *>(d.val), x, q,
                                               lane, wv, d.nn);
}

// ---------------------------------------------------------------------------
// start of a batched solve: x = 0, the padding of the packed inputs, the
// Chebyshev coefficients from the bound's maxima (grid: blocks x instances)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_binit(const GDesc *__restrict__ D)
{
    const GDesc &d = D[blockIdx.y];
    const int64_t i0 = blockIdx.x * int64_t(256) + threadIdx.x, step = gridDim.x * int64_t(256);
    for (int64_t k = i0; k < d.n; k += step) d.x[k] = 0.0;
    for (int64_t k = 2 * d.nm + i0; k < d.ldm; k += step) d.xm[k] = 0.0;
    for (int64_t k = 2 * d.ns + i0; k < d.lds; k += step) d.xs[k] = 0.0;
    if (blockIdx.x != 0 || d.pc != PBFB_PC_CHEB_SPAI) return;
    __shared__ double red[4];
    double hi = 0.0; // the bound: the largest of the slices' maxima
    for (int64_t q = threadIdx.x; q < (d.nn + SLICE - 1) / SLICE; q += 256) hi = fmax(hi, d.lmax[q]);
    for (int o = 32; o > 0; o >>= 1) hi = fmax(hi, __shfl_xor(hi, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = hi;
    __syncthreads();
    if (threadIdx.x != 0) return;
    hi = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    const double lo = hi / d.cheb_ratio;
    const double theta = 0.5 * (hi + lo), delta = 0.5 * (hi - lo), sigma = theta / delta;
    double rho = 1.0 / sigma;
    d.coef[0] = theta;
    d.coef[1] = 0.0;
    for (int s = 1; s < d.cheb_k; ++s) {
        const double rho1 = 1.0 / (2.0 * sigma - rho);
        d.coef[2 * s] = rho1 * rho;
        d.coef[2 * s + 1] = 2.0 * rho1 / delta;
        rho = rho1;
    }
}

// ---------------------------------------------------------------------------
// preconditioner stage: z = P^-1 src with src = V_j (ARN) or t = V y (RES and
// FIN, which also add the result to x).  Chebyshev term s (0-based) of the
// FEM block is written to z when k - 1 - s is even and to zb otherwise, so
// the last term always lands in z.
// ---------------------------------------------------------------------------
__device__ inline bool prec_active(int st) { return st == G_ARN || st == G_RES || st == G_FIN; }
__device__ inline double pc_src(const GDesc &d, const GState &s, int64_t r)
{
    return s.st == G_ARN ? vget(d, s.j, r) : d.t[r];
}

// the final value z_k of P^-1 src: x += z at the end of a cycle, and the
// entry of the apply's input (ARN: z, RES: x) into the packed surface
// vectors x_w = [u on the surface | lambda] (operator order)
__device__ inline void prec_final(const GDesc &d, const GState &s, int64_t k, double zv)
{
    d.z[k] = zv;
    double in = zv;
    if (s.st != G_ARN) d.x[k] = in = d.x[k] + zv;
    if (s.st == G_FIN) return;
    if (k < d.nn) {
        const int32_t v0 = d.nvert[0][k], v1 = d.nvert[1][k];
        if (v0 >= 0) d.xm[d.minv[0] ? d.minv[0][v0] : v0] = in;
        if (v1 >= 0) d.xs[d.minv[1] ? d.minv[1][v1] : v1] = in;
    } else if (k < d.nn + d.nm) {
        const int64_t i = k - d.nn;
        if (d.two_field) d.w[k] = in; // identity row of lambda_m
        else d.xm[d.nm + (d.minv[0] ? d.minv[0][i] : i)] = in;
    } else {
        const int64_t i = k - d.nn - d.nm;
        d.xs[d.ns + (d.minv[1] ? d.minv[1][i] : i)] = in;
    }
}

// surface row k of the preconditioner stage
__device__ inline void prec_surface(const GDesc &d, const GState &s, int64_t k)
{
    double zv = 0.0;
    if (d.pc == PBFB_PC_CHEB_SPAI) {
        const int w = k < d.nn + d.nm ? 0 : 1;
        const int64_t off = d.nn + (w == 0 ? 0 : d.nm), i = k - off;
        for (int32_t e = d.sp_ptr[w][i]; e < d.sp_ptr[w][i + 1]; ++e)
            zv = fma(d.sp_val[w][e], pc_src(d, s, off + d.sp_col[w][e]), zv);
    } else {
        zv = d.dinv[k] * pc_src(d, s, k);
    }
    prec_final(d, s, k, zv);
}

// One Chebyshev term of a row: its direction (written out so that the slices
// and the single workgroup below round alike)
__device__ inline double cheb_dir(double c0, double dk, double c1, double di, double src, double acc)
{
    return fma(c0, dk, (c1 * di) * (src - acc));
}

// Work items: a = 0: the 64 FEM rows from b, a = 1: the 256 surface rows from
// nn + b.  Surface rows: the approximate inverse.  FEM rows: the first two
// Chebyshev terms in one pass -- the first, z_0 = D^-1 src / theta, is
// pointwise, so the second's SpMV forms it at the gathered columns.  Without
// the block preconditioner every row is the inverse diagonal.
__global__ void __launch_bounds__(256) k_bfirst(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                                const GState *__restrict__ S)
{
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (!prec_active(s.st)) return;
    const GDesc &d = D[it.inst];
    const bool cheb = d.pc == PBFB_PC_CHEB_SPAI;
    if (it.a) {
        const int64_t k = d.nn + it.b + threadIdx.x;
        if (k < d.n) prec_surface(d, s, k);
        return;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t row = it.b + lane;
    if (!cheb || d.cheb_k == 1) {
        if (wv == 0 && row < d.nn)
            prec_final(d, s, row, d.dinv[row] * pc_src(d, s, row) / (cheb ? d.coef[0] : 1.0));
        return;
    }
    const double theta = d.coef[0];
    auto z0 = [&](int64_t c) { return d.dinv[c] * pc_src(d, s, c) / theta; };
    const double acc = fem_rows<true>(d, z0, it, lane, wv);
    if (wv != 0 || row >= d.nn) return;
    const double zp = z0(row);
    const double dv = cheb_dir(d.coef[2], zp, d.coef[3], d.dinv[row], pc_src(d, s, row), acc);
    d.dk[row] = dv;
    if (d.cheb_k == 2) prec_final(d, s, row, zp + dv);
    else ((d.cheb_k - 2) % 2 == 0 ? d.z : d.zb)[row] = zp + dv;
}

// Chebyshev term `step` >= 2 of the FEM block: one workgroup per 64-row
// slice (work item: inst, b = first row of the slice)
__global__ void __launch_bounds__(256) k_bcheb(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                               const GState *__restrict__ S, int step)
{
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (!prec_active(s.st)) return;
    const GDesc &d = D[it.inst];
    if (d.pc != PBFB_PC_CHEB_SPAI || step >= d.cheb_k) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t row = it.b + lane;
    const double *zp = ((d.cheb_k - step) % 2 == 0) ? d.z : d.zb; // term step - 1
    double *zn = ((d.cheb_k - 1 - step) % 2 == 0) ? d.z : d.zb;
    // the row's own entries, read ahead of the slice product (1 280-triangle
    // solve 16.3 -> 15.5 ms, 5 120 triangles 21.9 -> 21.4)
    double dk = 0.0, di = 0.0, src = 0.0, z0 = 0.0;
    const double c0 = d.coef[2 * step], c1 = d.coef[2 * step + 1];
    if (wv == 0 && row < d.nn) {
        dk = d.dk[row];
        di = d.dinv[row];
        src = pc_src(d, s, row);
        z0 = zp[row];
    }
    const double acc = fem_rows<true>(d, [zp](int64_t c) { return zp[c]; }, it, lane, wv);
    if (wv != 0 || row >= d.nn) return;
    const double dv = cheb_dir(c0, dk, c1, di, src, acc);
    d.dk[row] = dv;
    const double zv = z0 + dv;
    if (step == d.cheb_k - 1) prec_final(d, s, row, zv);
    else zn[row] = zv;
}

// The whole preconditioner stage of a small FEM block (prec_tiny) in one
// workgroup: the terms follow each other in LDS, with a barrier where k_bcheb
// needs a launch.  The matrix is read once, into registers (two rows of up
// to TINY_W FEM entries per thread), and a term is then LDS gathers on one CU:
// 23 terms of 1 134 rows take 44 us, as launches about 100 (sphere of 320
// triangles: 8.8 -> 6.8 ms per solve).  With the values streamed from L2 at
// every term one workgroup was slower than the launches (11.0 ms).  The
// arithmetic is that of the slices, so a batch may take either path: it takes
// this one only when every instance can, since beside larger instances the
// slices ride in launches that run anyway.
constexpr int TINY_T = 1024, TINY_H = 2, TINY_ROWS = TINY_T * TINY_H, TINY_W = 16;
static bool prec_tiny(const Problem &p, int pc, int cheb_k)
{
    return pc == PBFB_PC_CHEB_SPAI && cheb_k >= 2 && p.nn <= TINY_ROWS && p.max_fem <= TINY_W;
}
template <typename VT>
__device__ inline void tiny_terms(const GDesc &d, const GState &s, double (&zs)[2][TINY_ROWS])
{
    const int tid = threadIdx.x, nn = int(d.nn);
    const VT *val = static_cast<const VT *>(d.val);
    VT v[TINY_H][TINY_W];
    uint32_t c2[TINY_H][TINY_W / 2]; // two 16-bit columns each
    double src[TINY_H], di[TINY_H], dk[TINY_H];
#pragma unroll
    for (int h = 0; h < TINY_H; ++h) {
        const int r = tid + h * TINY_T;
        const bool in = r < nn;
        src[h] = in ? pc_src(d, s, r) : 0.0;
        di[h] = in ? d.dinv[r] : 0.0;
        dk[h] = di[h] * src[h] / d.coef[0];
        zs[0][r] = dk[h];
        const int b = in ? d.sptr[r / SLICE] : 0, w = in ? (d.sptr[r / SLICE + 1] - b) / SLICE : 0;
#pragma unroll
        for (int k = 0; k < TINY_W; ++k) {
            // past the row, and coupling columns (after the FEM ones): the row itself with value 0
            const int e = b + SLICE * (k < w ? k : 0) + r % SLICE;
            const int32_t c = k < w ? d.col[e] : nn;
            v[h][k] = c < nn ? val[e] : VT(0);
            const uint32_t cc = uint32_t(c < nn ? c : r);
            if (k % 2 == 0) c2[h][k / 2] = cc;
            else c2[h][k / 2] |= cc << 16;
        }
    }
    __syncthreads();
    for (int step = 1; step < d.cheb_k; ++step) {
        const double *zp = zs[(step - 1) & 1];
        double *zn = zs[step & 1];
        const double c0 = d.coef[2 * step], c1 = d.coef[2 * step + 1];
#pragma unroll
        for (int h = 0; h < TINY_H; ++h) {
            const int r = tid + h * TINY_T;
            if (h * TINY_T >= nn) break; // uniform
            double a4[SELL_W] = {}; // the order of sell_part_of and sell_reduce
#pragma unroll
            for (int k = 0; k < TINY_W; ++k)
                a4[k % SELL_W] = fma(double(v[h][k]), zp[k % 2 == 0 ? c2[h][k / 2] & 0xffff : c2[h][k / 2] >> 16],
                                     a4[k % SELL_W]);
            const double acc = ((a4[0] + a4[1]) + a4[2]) + a4[3];
            dk[h] = cheb_dir(c0, dk[h], c1, di[h], src[h], acc);
            const double zv = zp[r] + dk[h];
            zn[r] = zv;
            if (step == d.cheb_k - 1 && r < nn) prec_final(d, s, r, zv);
        }
        __syncthreads();
    }
}
__global__ void __launch_bounds__(TINY_T) k_btiny(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                                  const GState *__restrict__ S)
{
    __shared__ double zs[2][TINY_ROWS];
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (!prec_active(s.st)) return;
    const GDesc &d = D[it.inst];
    for (int64_t k = d.nn + threadIdx.x; k < d.n; k += TINY_T) prec_surface(d, s, k);
    if (d.f32) tiny_terms<float>(d, s, zs);
    else tiny_terms<double>(d, s, zs);
}

// work item: inst, a = interface (0/1), b = first row of the workgroup.  One
// instantiation per storage type, each skipping the instances of the other:
// a kernel holding both row routines would be register-allocated for their
// union and run at half the occupancy of either.
template <typename MT>
__global__ void __launch_bounds__(GEMV_THREADS, gemv_occupancy<MT>()) k_bgemv(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                               const GState *__restrict__ S)
{
    const WItem it = wl[blockIdx.x];
    if (!applies(S[it.inst].st)) return;
    const GDesc &d = D[it.inst];
    if (d.f32 != (sizeof(MT) == 4)) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int a = it.a & 1; // surface; it.a & 2: K item of the symmetric use
    const int64_t n = a == 0 ? d.nm : d.ns;
    const int64_t ld = a == 0 ? d.ldm : d.lds;
    const double *x = a == 0 ? d.xm : d.xs;
    double *y = d.w + d.nn + (a == 0 ? 0 : d.nm);
    const MT *B = static_cast<const MT *>(a == 0 ? d.Bm : d.Bs);
    if (!d.symm[a]) {
        const int64_t r0 = it.b + wv * GEMV_RW;
        if (r0 < n) gemv_rows<MT>(B, x, y, a == 0 ? d.mvm : d.mvs, n, ld, r0, lane);
    } else if (it.a & 2) {
        gemv_rows_symK<MT>(B, x, y, a == 0 ? d.mvm : d.mvs, n, ld, it.b, threadIdx.x);
    } else {
        gemv_rows_symV<MT>(B, x, static_cast<sym_part_t<MT> *>(d.symP[a]), n, ld, it.b, threadIdx.x);
    }
}

// The rest of the apply after k_bgemv, item first + blockIdx: the first nfin
// items are the second stage of the symmetric use (inst, a = surface, b =
// first of GFIN_ROWS rows) and the dense rows of small surfaces (a = surface
// | 2, b = first of GSMALL_ROWS rows), the others FEM SpMV slices (b = first
// row); only the second stages depend on k_bgemv.
__global__ void __launch_bounds__(256) k_btail(const WItem *__restrict__ wl, unsigned first, unsigned nfin,
                                               const GDesc *__restrict__ D, const GState *__restrict__ S)
{
    const unsigned bi = first + blockIdx.x;
    const WItem it = wl[bi];
    const int st = S[it.inst].st;
    if (!applies(st)) return;
    const GDesc &d = D[it.inst];
    if (bi < nfin) {
        const int a = it.a & 1;
        const int64_t n = a == 0 ? d.nm : d.ns, ld = a == 0 ? d.ldm : d.lds;
        const double *x = a == 0 ? d.xm : d.xs;
        double *y = d.w + d.nn + (a == 0 ? 0 : d.nm);
        const int32_t *oidx = a == 0 ? d.mvm : d.mvs;
        const void *B = a == 0 ? d.Bm : d.Bs;
        if (!(it.a & 2))
            gemv_sym_finish(n, static_cast<const double *>(d.symP[a]), d.dl_ptr[a], d.dl_col[a], d.dl_val[a], x, y,
                            oidx, it.b, threadIdx.x);
        else if (d.f32)
            gemv_rows_small<float>(static_cast<const float *>(B), x, y, oidx, n, ld, it.b, threadIdx.x);
        else
            gemv_rows_small<double>(static_cast<const double *>(B), x, y, oidx, n, ld, it.b, threadIdx.x);
        return;
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t row = it.b + lane;
    const double *in = st == G_ARN ? d.z : d.x;
    const double acc = fem_rows<false>(d, [in](int64_t c) { return in[c]; }, it, lane, wv);
    if (wv == 0 && row < d.nn) d.w[row] = acc;
}

// ---------------------------------------------------------------------------
// classical Gram-Schmidt, two passes over row chunks (work item: inst, a =
// chunk, b = first row): k_bmdot leaves the chunk's partial dot products
// V_i . w; k_bmid adds every chunk's (each workgroup for itself, in chunk
// order), subtracts and leaves the partials of the second pass from the rows
// it still holds; k_bend adds those, subtracts and leaves the chunk's |w|^2.
// Kernel boundaries order the passes, every sum has a fixed order.
// ---------------------------------------------------------------------------
// Rows per chunk: about 96 chunks (the sum over chunks that every workgroup
// of the next pass repeats stays a few loads per thread) of at most 2048 rows
// (so that large instances still fill the chip)
constexpr int CHB_MAX = 8; // x 256 rows
static int64_t chunk_rows(int64_t n)
{
    return 256 * std::min<int64_t>(CHB_MAX, std::max<int64_t>(1, (n + 256 * 96 - 1) / (256 * 96)));
}

// sums over the workgroup of 256 threads of eight values; valid in threads 0..7 (value = thread id)
__device__ inline double block_sum8(const double (&acc)[8], double (&red)[4][8])
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        double v = acc[q];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) red[wv][q] = v;
    }
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x < 8) r = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
    __syncthreads();
    return r;
}

// hs[i] = sum over chunks of part[c][i], i < jj: 8 x 32 threads, each 32
// coefficients at a time over every eighth chunk
__device__ inline void chunk_sums(const GDesc &d, const double *__restrict__ part, int jj, double *hs,
                                  double (&red)[8][33])
{
    const int g = threadIdx.x >> 5, l = threadIdx.x & 31;
    for (int i0 = 0; i0 < jj; i0 += 32) {
        const int i = i0 + l;
        double t = 0.0;
        if (i < jj) {
#pragma unroll 4
            for (int64_t c = g; c < d.nchb; c += 8) t += part[c * (d.m + 1) + i];
        }
        red[g][l] = t;
        __syncthreads();
        if (g == 0 && i < jj) {
            double v = red[0][l];
#pragma unroll
            for (int k = 1; k < 8; ++k) v += red[k][l];
            hs[i] = v;
        }
        __syncthreads();
    }
}

constexpr int DOT_GROUPS = 4; // groups of eight coefficients in flight per chunk
__global__ void __launch_bounds__(256) k_bmdot(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                               const GState *__restrict__ S)
{
    __shared__ double red[4][8];
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (s.st != G_ARN) return;
    const GDesc &d = D[it.inst];
    for (int i0 = blockIdx.y * 8; i0 <= s.j; i0 += 8 * DOT_GROUPS) {
        const int kk = min(8, s.j + 1 - i0);
        double acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.0;
        auto body = [&](auto *V0) {
            for (int64_t k = it.b + threadIdx.x; k < it.b + d.chb && k < d.n; k += 256) {
                const double wk = d.w[k];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (q < kk) acc[q] = fma(double(V0[int64_t(q) * d.n + k]), wk, acc[q]);
            }
        };
        if (d.vf32) body(vcol<float>(d, i0));
        else body(vcol<double>(d, i0));
        const double r = block_sum8(acc, red);
        if (threadIdx.x < kk) d.part[int64_t(it.a) * (d.m + 1) + i0 + threadIdx.x] = r;
    }
}

// w -= sum_i h1_i V_i; partial dot products of the second pass
__global__ void __launch_bounds__(256) k_bmid(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                              const GState *__restrict__ S)
{
    __shared__ double hs[1024];
    __shared__ double red[4][8], redc[8][33];
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (s.st != G_ARN) return;
    const GDesc &d = D[it.inst];
    const int jj = s.j + 1;
    chunk_sums(d, d.part, jj, hs, redc);
    if (it.a == 0)
        for (int i = threadIdx.x; i < jj; i += 256) d.h1[i] = hs[i];
    const int64_t kend = std::min(it.b + d.chb, d.n);
    double v[CHB_MAX]; // this thread's rows
    auto body = [&](auto *V0) {
#pragma unroll
        for (int r = 0; r < CHB_MAX; ++r) {
            const int64_t k = it.b + 256 * r + threadIdx.x;
            v[r] = 0.0;
            if (k >= kend) continue;
            double t = d.w[k];
#pragma unroll 8
            for (int i = 0; i < jj; ++i) t = fma(-hs[i], double(V0[int64_t(i) * d.n + k]), t);
            d.w[k] = v[r] = t;
        }
        for (int i0 = 0; i0 < jj; i0 += 8) {
            double acc[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] = 0.0;
#pragma unroll
            for (int r = 0; r < CHB_MAX; ++r) {
                const int64_t k = it.b + 256 * r + threadIdx.x;
                if (k >= kend) continue;
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (i0 + q < jj) acc[q] = fma(double(V0[int64_t(i0 + q) * d.n + k]), v[r], acc[q]);
            }
            const double r = block_sum8(acc, red);
            if (threadIdx.x < 8 && i0 + int(threadIdx.x) < jj)
                d.part2[int64_t(it.a) * (d.m + 1) + i0 + threadIdx.x] = r;
        }
    };
    if (d.vf32) body(vcol<float>(d, 0));
    else body(vcol<double>(d, 0));
}

// ARN: w -= sum_i h2_i V_i;  RES: w = b - w;  INIT: w = b; the chunk's |w|^2
__global__ void __launch_bounds__(256) k_bend(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                              const GState *__restrict__ S)
{
    __shared__ double hs[1024];
    __shared__ double red[4][8], redc[8][33];
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    const bool arn = s.st == G_ARN;
    if (!arn && s.st != G_RES && s.st != G_INIT) return;
    const GDesc &d = D[it.inst];
    const int jj = arn ? s.j + 1 : 0;
    if (arn) {
        chunk_sums(d, d.part2, jj, hs, redc);
        if (it.a == 0)
            for (int i = threadIdx.x; i < jj; i += 256) d.h2[i] = hs[i];
    }
    const int64_t kend = std::min(it.b + d.chb, d.n);
    double nrm[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    auto body = [&](auto *V0) {
        for (int64_t k = it.b + threadIdx.x; k < kend; k += 256) {
            double v;
            if (s.st == G_INIT) v = d.b[k];
            else if (s.st == G_RES) v = d.b[k] - d.w[k];
            else {
                v = d.w[k];
#pragma unroll 8
                for (int i = 0; i < jj; ++i) v = fma(-hs[i], double(V0[int64_t(i) * d.n + k]), v);
            }
            d.w[k] = v;
            nrm[0] = fma(v, v, nrm[0]);
        }
    };
    if (d.vf32) body(vcol<float>(d, 0));
    else body(vcol<double>(d, 0));
    const double t = block_sum8(nrm, red);
    if (threadIdx.x == 0) d.npart[it.a] = t;
}

// ---------------------------------------------------------------------------
// control: one wavefront per instance.  |w| from the chunk partials.  ARN:
// Hessenberg column, Givens chain (in LDS, one lane), residual estimate, cycle
// end; at the end of a cycle the triangular solve H y = g (column sweep across
// the lanes).  INIT/RES: true residual test and cycle start.
//
// What the host needs to know goes to pinned host memory at the end of every
// step of the batch (the last instance writes it): the step, the instances
// that need no step after the next one (DONE, FAIL or FIN) and those that
// need none at all (DONE or FAIL).
// ---------------------------------------------------------------------------
struct GCount {
    int tick, ending, ended;
};
// the host word: step << 40 | ending << 20 | ended (20 bits hold a batch's instances)
constexpr int GCOUNT_BITS = 20;
constexpr int64_t GCOUNT_MAX = (int64_t(1) << GCOUNT_BITS) - 1;

__global__ void __launch_bounds__(64) k_bcontrol(const GDesc *__restrict__ D, GState *__restrict__ S,
                                                 GCount *__restrict__ C, unsigned long long *__restrict__ host,
                                                 GState *__restrict__ hstate)
{
    __shared__ double hc[1024], cs[1024], sn[1024], gl[1024];
    __shared__ GState ss;
    const int q = blockIdx.x, lane = threadIdx.x;
    const GDesc &d = D[q];
    if (lane == 0) ss = S[q];
    __syncthreads();
    const int st0 = ss.st;
    const int m = d.m;
    double nr = 0.0;
    if (st0 == G_ARN || st0 == G_RES || st0 == G_INIT) {
        for (int64_t c = lane; c < d.nchb; c += 64) nr += d.npart[c];
        for (int off = 32; off > 0; off >>= 1) nr += __shfl_xor(nr, off);
        nr = sqrt(nr);
        if (lane == 0) *d.nrm = nr;
    }
    if (st0 == G_ARN) {
        const int j = ss.j;
        for (int i = lane; i <= j; i += 64) {
            hc[i] = d.h1[i] + d.h2[i];
            if (i < j) {
                cs[i] = d.cs[i];
                sn[i] = d.sn[i];
            }
        }
        __syncthreads();
        bool cycle_end = false;
        if (lane == 0) {
            double t = hc[0];
            for (int i = 0; i < j; ++i) {
                const double c2 = hc[i + 1];
                hc[i] = cs[i] * t + sn[i] * c2;
                t = -sn[i] * t + cs[i] * c2;
            }
            const double den = hypot(t, nr);
            const double cj = t / den, sj = nr / den;
            d.cs[j] = cj;
            d.sn[j] = sj;
            hc[j] = den;
            const double gj = d.g[j];
            d.g[j + 1] = -sj * gj;
            d.g[j] = cj * gj;
            ss.j = j + 1;
            ss.total += 1;
            ss.napply += 1;
            const double res = fabs(d.g[j + 1]);
            if (!(res == res)) {
                ss.st = G_FAIL;
                ss.code = PBFB_ENAN;
            } else if (res <= ss.target || nr == 0.0 || ss.j == m || ss.total >= d.maxit) {
                // converged on the estimate: no true-residual check, except with an
                // FP32 basis, whose restarts are refinement steps that need it
                ss.st = (res <= ss.target || nr == 0.0) && !d.vf32 ? G_FIN : G_RES;
            }
        }
        __syncthreads();
        cycle_end = ss.st == G_FIN || ss.st == G_RES;
        double *Hj = d.H + int64_t(j) * (m + 1);
        for (int i = lane; i <= j; i += 64) Hj[i] = hc[i];
        if (lane == 0) Hj[j + 1] = 0.0;
        if (cycle_end) {
            // back substitution by columns: y_i = g_i / H_ii, then g_k -= H_ki y_i for k < i
            const int jc = ss.j;
            __threadfence_block();
            for (int i = lane; i < jc; i += 64) gl[i] = d.g[i];
            __syncthreads();
            for (int i = jc - 1; i >= 0; --i) {
                // column j (this step's) is taken from LDS, older columns from global memory
                const double yi = gl[i] / (i == j ? hc[j] : d.H[int64_t(i) * (m + 1) + i]);
                for (int k = lane; k < i; k += 64) gl[k] -= (i == j ? hc[k] : d.H[int64_t(i) * (m + 1) + k]) * yi;
                if (lane == 0) d.y[i] = yi;
                __syncthreads();
            }
        }
    } else if (lane == 0 && st0 == G_FIN) {
        ss.st = G_DONE;
    } else if (lane == 0 && (st0 == G_RES || st0 == G_INIT)) {
        if (st0 == G_INIT) ss.target = d.tol * nr;
        else ss.napply += 1; // RES: the true residual took one application
        ss.beta = nr;
        if (!(nr <= 1.7976931348623157e308)) { // NaN or infinite
            ss.st = G_FAIL;
            ss.code = PBFB_ENAN;
        } else if (nr <= ss.target) {
            ss.st = G_DONE;
        } else if (ss.total >= d.maxit) {
            ss.st = G_FAIL;
            ss.code = PBFB_ENOTCONV;
        } else {
            for (int i = 0; i <= m; ++i) d.g[i] = 0.0;
            d.g[0] = nr;
            ss.j = 0;
            ss.st = G_ARN;
        }
    }
    __syncthreads();
    if (lane != 0) return;
    S[q] = ss;
    const bool over = ss.st == G_DONE || ss.st == G_FAIL, was = st0 == G_DONE || st0 == G_FAIL;
    if (!was) hstate[q] = ss; // read by the host after its last synchronisation
    if (over && !was) atomicAdd(&C->ended, 1);
    if ((over || ss.st == G_FIN) && !was && st0 != G_FIN) atomicAdd(&C->ending, 1);
    __threadfence(); // the counts before the tick
    const int nb = int(gridDim.x), t = atomicAdd(&C->tick, 1) + 1;
    if (t % nb) return;
    const unsigned long long ending = atomicAdd(&C->ending, 0), ended = atomicAdd(&C->ended, 0);
    __hip_atomic_store(host, (static_cast<unsigned long long>(t / nb) << (2 * GCOUNT_BITS)) | (ending << GCOUNT_BITS) | ended,
                       __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// what the new state asks for: ARN: V_j = w / |w| (j = 0 at a cycle start);
// RES, FIN (a cycle just ended): t = V y
__global__ void __launch_bounds__(256) k_bnext(const WItem *__restrict__ wl, const GDesc *__restrict__ D,
                                               const GState *__restrict__ S)
{
    __shared__ double ys[1024];
    const WItem it = wl[blockIdx.x];
    const GState s = S[it.inst];
    if (!prec_active(s.st)) return;
    const GDesc &d = D[it.inst];
    const int64_t k = it.b + threadIdx.x;
    if (s.st == G_ARN) {
        const double nr = *d.nrm;
        const double inv = nr > 0.0 ? 1.0 / nr : 0.0;
        const int64_t off = int64_t(s.j) * d.n;
        if (k < d.n) {
            if (d.vf32) static_cast<float *>(d.V)[off + k] = float(d.w[k] * inv);
            else static_cast<double *>(d.V)[off + k] = d.w[k] * inv;
        }
        return;
    }
    for (int i = threadIdx.x; i < s.j; i += 256) ys[i] = d.y[i];
    __syncthreads();
    if (k >= d.n) return;
    double v = 0.0;
    auto body = [&](auto *V0) {
#pragma unroll 8
        for (int i = 0; i < s.j; ++i) v = fma(ys[i], double(V0[int64_t(i) * d.n + k]), v);
    };
    if (d.vf32) body(vcol<float>(d, 0));
    else body(vcol<double>(d, 0));
    d.t[k] = v;
}

// ===========================================================================
// host driver
// ===========================================================================
// a captured Krylov step is valid for the same device buffer and launch shapes
struct GraphKey {
    void *dev = nullptr;
    unsigned nvec = 0, ngemv = 0, nspmv = 0, ncheb = 0, nfirst = 0, ntiny = 0, ndot = 0, nb = 0, nfin = 0;
    int kmax = 0, types = 0; // types: bit 0 FP64 operators present, bit 1 FP32
    bool operator==(const GraphKey &o) const
    {
        return dev == o.dev && nvec == o.nvec && ngemv == o.ngemv && nspmv == o.nspmv && ncheb == o.ncheb &&
               nfirst == o.nfirst && ntiny == o.ntiny && ndot == o.ndot && nb == o.nb && nfin == o.nfin && kmax == o.kmax && types == o.types;
    }
};

// per host thread: the device copy of a batch's descriptors and work lists,
// its pinned source, and the word the control kernel reports to
struct BatchBuffers {
    void *dev = nullptr, *stage = nullptr;
    size_t dev_bytes = 0, stage_bytes = 0;
    unsigned long long *word = nullptr;
    GState *state = nullptr; // pinned: every instance's state as control left it
    size_t nstate = 0;
    size_t listed = 0, head = 0; // bytes of the stage that the device copy holds (0: none), of them before the lists
    hipGraphExec_t step = nullptr; // the captured Krylov step (left to process exit)
    GraphKey key;
    ~BatchBuffers()
    {
        if (dev) (void)hipFree(dev);
        if (stage) (void)hipHostFree(stage);
        if (word) (void)hipHostFree(word);
        if (state) (void)hipHostFree(state);
    }
    void reserve(size_t bytes, size_t nb)
    {
        if (nstate < nb) {
            if (step) PB_HIP(hipGraphExecDestroy(step)); // it holds the pointer
            step = nullptr;
            if (state) PB_HIP(hipHostFree(state));
            state = nullptr;
            nstate = 0;
            PB_HIP(hipHostMalloc(reinterpret_cast<void **>(&state), sizeof(GState) * nb, hipHostMallocDefault));
            nstate = nb;
        }
        if (!word) PB_HIP(hipHostMalloc(reinterpret_cast<void **>(&word), 64, hipHostMallocDefault));
        if (stage_bytes < bytes) {
            if (stage) PB_HIP(hipHostFree(stage));
            stage = nullptr;
            stage_bytes = 0;
            listed = 0;
            PB_HIP(hipHostMalloc(&stage, bytes, hipHostMallocDefault));
            stage_bytes = bytes;
        }
        if (dev_bytes < bytes) {
            if (step) PB_HIP(hipGraphExecDestroy(step));
            step = nullptr;
            if (dev) PB_HIP(hipFree(dev));
            dev = nullptr;
            dev_bytes = 0;
            listed = 0;
            PB_HIP(hipMalloc(&dev, bytes));
            dev_bytes = bytes;
        }
    }
};

static BatchBuffers &batch_buffers()
{
    static thread_local BatchBuffers B;
    return B;
}

// Workgroups go to the eight XCDs in turn, each with its own L2: the item list
// whose first item is workgroup `first` of its launch, reordered so that every
// XCD gets a contiguous eighth.  Neighbouring slices gather the same input
// entries, and each slice returns to the same XCD in every launch (5 120
// triangles FP64 24.0 -> 23.4 ms per solve, 20 480: 105.3 -> 104.7).
static void xcd_order(std::vector<WItem> &v, size_t first)
{
    constexpr size_t NX = 8;
    const size_t n = v.size();
    std::vector<WItem> out;
    out.reserve(n);
    size_t next[NX], end[NX];
    for (size_t x = 0; x < NX; ++x) {
        next[x] = n * x / NX;
        end[x] = n * (x + 1) / NX;
    }
    for (size_t i = 0; i < n; ++i) {
        size_t x = (first + i) % NX;
        while (next[x] == end[x]) x = (x + 1) % NX; // the last round
        out.push_back(v[next[x]++]);
    }
    v.swap(out);
}

void batched_gmres(std::vector<GmresJob *> &jobs, hipStream_t s)
{
    const int nb = int(jobs.size());
    if (nb == 0) return;
    std::vector<GDesc> desc(nb);
    std::vector<GState> st(nb);
    std::vector<WItem> wl_vec, wl_gemv, wl_spmv, wl_cheb, wl_surf, wl_tiny, wl_dot, wl_fin;
    // GEMV items in the order of gemv_item, over the batch: the heavy V items
    // of every instance, then the K and full-row items, then the other V items
    std::vector<WItem> wl_gemv_k, wl_gemv_v;
    int maxiter_host = 0, kmax = 1;
    int64_t nmax = 0;
    const bool tiny = std::all_of(jobs.begin(), jobs.end(),
                                  [](const GmresJob *J) { return prec_tiny(*J->p, J->pc, J->cheb_k); });
    for (int q = 0; q < nb; ++q) {
        GmresJob &J = *jobs[q];
        Problem &p = *J.p;
        const int m = J.restart;
        const int64_t n = p.n();
        GDesc &d = desc[q];
        d.Bm = p.surf[0].B;
        d.Bs = p.surf[1].B;
        d.nm = p.surf[0].nv;
        d.ns = p.surf[1].nv;
        d.ldm = bem_ld(d.nm);
        d.lds = bem_ld(d.ns);
        d.f32 = p.precision == PBFB_MIXED;
        d.two_field = p.two_field() ? 1 : 0;
        d.mvm = p.bem_mf ? nullptr : p.surf[0].mvert;
        d.mvs = p.bem_mf ? nullptr : p.surf[1].mvert;
        d.sptr = p.d_sptr;
        d.col = p.d_col;
        d.lng = p.fr.sell();
        d.val = d.f32 ? static_cast<const void *>(p.d_val32) : static_cast<const void *>(p.d_val);
        d.nn = p.nn;
        d.n = n;
        d.dinv = J.dinv;
        d.pc = J.pc;
        d.cheb_k = J.cheb_k;
        d.cheb_ratio = J.cheb_ratio;
        d.lmax = J.lmax;
        for (int w = 0; w < 2; ++w) {
            d.nvert[w] = p.surf[w].nvert;
            d.minv[w] = p.bem_mf ? nullptr : p.surf[w].minv;
            d.sp_ptr[w] = p.surf[w].ring_ptr;
            d.sp_col[w] = p.surf[w].ring;
            d.sp_val[w] = p.surf[w].spai;
            const SurfaceDev &SD = p.surf[w];
            d.symm[w] = (!p.bem_mf && SD.sym) ? 1 : 0;
            d.symP[w] = d.symm[w] ? scratch<double>(p, w == 0 ? SCR_SYMP0 : SCR_SYMP1,
                                                    size_t(sym_partials_doubles(SD.nv)))
                                  : nullptr;
            d.dl_ptr[w] = SD.d_ptr;
            d.dl_col[w] = SD.d_col;
            d.dl_val[w] = SD.d_val;
        }
        d.z = scratch<double>(p, SCR_PZ, n);
        d.t = scratch<double>(p, SCR_PT, n);
        d.zb = scratch<double>(p, SCR_PZB, p.nn);
        d.dk = scratch<double>(p, SCR_PDK, p.nn);
        d.coef = scratch<double>(p, SCR_PCOEF, 2 * 64 + 2);
        d.vf32 = J.basis32 && p.precision == PBFB_MIXED;
        if (d.vf32) d.V = scratch<float>(p, SCR_BASIS32, size_t(m + 1) * n);
        else d.V = scratch<double>(p, SCR_BASIS, size_t(m + 1) * n);
        d.w = scratch<double>(p, SCR_G0, n);
        d.xm = scratch<double>(p, SCR_XM, d.ldm);
        d.xs = scratch<double>(p, SCR_XS, d.lds);
        d.x = J.x;
        d.b = J.b;
        double *kry = scratch<double>(p, SCR_HVEC, size_t(m) * (m + 1) + 3 * m + 3 * (m + 1) + 8);
        d.H = kry;
        d.cs = d.H + size_t(m) * (m + 1);
        d.sn = d.cs + m;
        d.y = d.sn + m;
        d.g = d.y + m;
        d.h1 = d.g + (m + 1);
        d.h2 = d.h1 + (m + 1);
        d.chb = chunk_rows(n);
        d.nchb = (n + d.chb - 1) / d.chb;
        d.part = scratch<double>(p, SCR_HPART, 2 * size_t(d.nchb) * (m + 1));
        d.part2 = d.part + size_t(d.nchb) * (m + 1);
        d.npart = scratch<double>(p, SCR_NRM, d.nchb + 1);
        d.nrm = d.npart + d.nchb;
        d.tol = J.tol;
        d.m = m;
        d.maxit = J.maxit;
        st[q] = GState{G_INIT, 0, 0, 0, 0, 0.0, 0.0};
        nmax = std::max(nmax, n);
        for (int64_t k = 0; k < n; k += CH) wl_vec.push_back(WItem{q, 0, k});
        for (int64_t c = 0; c < d.nchb; ++c) wl_dot.push_back(WItem{q, int(c), c * d.chb});
        static_assert(GROWS == GSYM, "GEMV work items are the symmetric routine's row blocks");
        {
            // per surface: K (or full-row) items in row order, V items last
            // row block first (the last rows read the most); the first
            // gemv_heavy of the V items go before every K item; the two
            // surfaces alternate inside each stretch
            std::vector<WItem> kit[2], vit[2];
            for (int a = d.two_field ? 1 : 0; a < 2; ++a) {
                const int64_t nv = a == 0 ? d.nm : d.ns;
                if (p.bem_mf) continue; // no stored operator
                if (gemv_small(nv, d.f32 != 0)) {
                    for (int64_t r = 0; r < nv; r += GSMALL_ROWS) wl_fin.push_back(WItem{q, a | 2, r});
                    continue;
                }
                for (int64_t r = 0; r < nv; r += GROWS) kit[a].push_back(WItem{q, a | (d.symm[a] ? 2 : 0), r});
                if (d.symm[a]) {
                    for (int64_t r = (nv - 1) / GROWS * GROWS; r >= 0; r -= GROWS) vit[a].push_back(WItem{q, a, r});
                    for (int64_t r = 0; r < nv; r += GFIN_ROWS) wl_fin.push_back(WItem{q, a, r});
                }
            }
            auto alternate = [](const std::vector<WItem> &u, size_t u0, size_t u1, const std::vector<WItem> &v,
                                size_t v0, size_t v1, std::vector<WItem> &out) {
                for (size_t i = u0, j = v0; i < u1 || j < v1;) {
                    if (i < u1) out.push_back(u[i++]);
                    if (j < v1) out.push_back(v[j++]);
                }
            };
            const size_t h0 = size_t(gemv_heavy(d.f32 != 0, int64_t(vit[0].size())));
            const size_t h1 = size_t(gemv_heavy(d.f32 != 0, int64_t(vit[1].size())));
            alternate(vit[0], 0, h0, vit[1], 0, h1, wl_gemv);
            alternate(kit[0], 0, kit[0].size(), kit[1], 0, kit[1].size(), wl_gemv_k);
            alternate(vit[0], h0, vit[0].size(), vit[1], h1, vit[1].size(), wl_gemv_v);
        }
        auto slice = [&](int64_t r) {
            const int32_t e0 = p.sptr[r / SLICE];
            return WItem{q, 0, r, e0, (p.sptr[r / SLICE + 1] - e0) / SLICE};
        };
        for (int64_t r = 0; r < p.nn; r += SLICE) wl_spmv.push_back(slice(r));
        if (tiny) {
            wl_tiny.push_back(WItem{q, 0, 0});
        } else {
            for (int64_t r = 0; r < p.nn; r += SLICE) wl_cheb.push_back(slice(r));
            for (int64_t k = 0; k < n - p.nn; k += CH) wl_surf.push_back(WItem{q, 1, k});
            if (J.pc == PBFB_PC_CHEB_SPAI) kmax = std::max(kmax, J.cheb_k);
        }
        maxiter_host = std::max(maxiter_host, J.maxit + J.maxit / std::max(m, 1) + 4);
    }
    wl_gemv.insert(wl_gemv.end(), wl_gemv_k.begin(), wl_gemv_k.end());
    wl_gemv.insert(wl_gemv.end(), wl_gemv_v.begin(), wl_gemv_v.end());
    xcd_order(wl_cheb, 0);
    xcd_order(wl_spmv, wl_fin.size());
    // k_btail: the dense items, then the SpMV slices; k_bfirst: the FEM slices
    // of the instances that are not tiny (k_bcheb's list), then the surface rows
    const unsigned nvec = unsigned(wl_vec.size()), ngemv = unsigned(wl_gemv.size()),
                   nspmv = unsigned(wl_spmv.size()), ncheb = unsigned(wl_cheb.size()),
                   nfirst = ncheb + unsigned(wl_surf.size()), ntiny = unsigned(wl_tiny.size()),
                   ndot = unsigned(wl_dot.size()), nfin = unsigned(wl_fin.size());
    PB_CHECK(nb <= GCOUNT_MAX, PBFB_EINVAL, "too many instances in one batch");
    // descriptors, states, counters and work lists: one pinned block, one copy
    BatchBuffers &BB = batch_buffers();
    const size_t items = wl_vec.size() + wl_gemv.size() + wl_fin.size() + wl_spmv.size() + nfirst +
                         ntiny + wl_dot.size();
    const size_t bytes = (sizeof(GDesc) + sizeof(GState)) * nb + sizeof(GCount) + sizeof(WItem) * items + 512;
    BB.reserve(bytes, size_t(nb));
    // the block and the reported word belong to this call until its stream has drained
    struct Drain {
        hipStream_t s;
        ~Drain() { (void)hipStreamSynchronize(s); }
    } drain{s};
    size_t cur = 0;
    bool same = true; // the lists are those of the previous call
    // until the copy is enqueued the device copy holds none: an exception on
    // the way leaves new lists in the stage alone
    const size_t listed = std::exchange(BB.listed, 0);
    auto put = [&](const void *src, size_t b, bool list) {
        char *to = static_cast<char *>(BB.stage) + cur;
        if (!list) {
            std::memcpy(to, src, b);
        } else if (!same || cur + b > listed || std::memcmp(to, src, b)) {
            same = false;
            std::memcpy(to, src, b);
        }
        char *d = static_cast<char *>(BB.dev) + cur;
        cur += (b + 15) / 16 * 16;
        return static_cast<void *>(d);
    };
    auto put_items = [&](std::initializer_list<const std::vector<WItem> *> lists) {
        const std::vector<WItem> *const *l = lists.begin();
        std::vector<WItem> v(**l);
        for (++l; l != lists.end(); ++l) v.insert(v.end(), (*l)->begin(), (*l)->end());
        return static_cast<WItem *>(put(v.data(), sizeof(WItem) * v.size(), true));
    };
    GDesc *dD = static_cast<GDesc *>(put(desc.data(), sizeof(GDesc) * nb, false));
    GState *dS = static_cast<GState *>(put(st.data(), sizeof(GState) * nb, false));
    const GCount zero{};
    GCount *dC = static_cast<GCount *>(put(&zero, sizeof(zero), false));
    const size_t head = cur;
    WItem *dvec = put_items({&wl_vec});
    WItem *dgemv = put_items({&wl_gemv});
    WItem *dtail = put_items({&wl_fin, &wl_spmv});
    WItem *dfirst = put_items({&wl_cheb, &wl_surf});
    WItem *dtiny = put_items({&wl_tiny});
    WItem *ddot = put_items({&wl_dot});
    if (listed != cur || BB.head != head) same = false;
    PB_HIP(hipMemcpyAsync(BB.dev, BB.stage, same ? head : cur, hipMemcpyHostToDevice, s));
    BB.listed = cur;
    BB.head = head;
    __atomic_store_n(BB.word, 0ull, __ATOMIC_RELEASE);

    EventTimer *tm = nullptr;
    for (auto *J : jobs)
        if (J->p->timing) {
            tm = &J->p->timer;
            break;
        }
    hipLaunchKernelGGL(k_binit, dim3(unsigned(std::min<int64_t>((nmax + 255) / 256, 512)), unsigned(nb)), dim3(256), 0,
                       s, dD);
    int types = 0;
    bool any_mf = false;
    for (auto *J : jobs) {
        if (J->p->bem_mf) any_mf = true;
        else types |= J->p->precision == PBFB_MIXED ? 2 : 1;
    }
    // the end of a step: |w| and control, the next basis vector or t = V y
    auto enqueue_end = [&]() {
        hipLaunchKernelGGL(k_bend, dim3(ndot), dim3(256), 0, s, ddot, dD, dS);
        hipLaunchKernelGGL(k_bcontrol, dim3(unsigned(nb)), dim3(64), 0, s, dD, dS, dC, BB.word, BB.state);
        hipLaunchKernelGGL(k_bnext, dim3(nvec), dim3(256), 0, s, dvec, dD, dS);
    };
    // one Krylov step of the whole batch
    auto enqueue_step = [&]() {
        if (tm) tm->begin(T_PREC, s);
        if (ntiny) hipLaunchKernelGGL(k_btiny, dim3(ntiny), dim3(TINY_T), 0, s, dtiny, dD, dS);
        if (nfirst) hipLaunchKernelGGL(k_bfirst, dim3(nfirst), dim3(256), 0, s, dfirst, dD, dS);
        for (int step = 2; step < kmax; ++step)
            hipLaunchKernelGGL(k_bcheb, dim3(ncheb), dim3(256), 0, s, dfirst, dD, dS, step);
        if (tm) tm->end(s);
        if (tm) tm->begin(T_APPLY, s);
        if (tm) tm->begin(T_GEMV, s);
        if (ngemv && (types & 1)) hipLaunchKernelGGL(k_bgemv<double>, dim3(ngemv), dim3(GEMV_THREADS), 0, s, dgemv, dD, dS);
        if (ngemv && (types & 2)) hipLaunchKernelGGL(k_bgemv<float>, dim3(ngemv), dim3(GEMV_THREADS), 0, s, dgemv, dD, dS);
        // matrix-free instances: their own launches, gated by their state word
        for (size_t q = 0; q < jobs.size() && any_mf; ++q) {
            Problem &pq = *jobs[q]->p;
            if (!pq.bem_mf) continue;
            const int *stq = reinterpret_cast<const int *>(dS + q);
            mf_apply(pq, 0, desc[q].xm, desc[q].w + pq.nn, stq, s);
            mf_apply(pq, 1, desc[q].xs, desc[q].w + pq.nn + pq.surf[0].nv, stq, s);
        }
        if (!tm) {
            hipLaunchKernelGGL(k_btail, dim3(nfin + nspmv), dim3(256), 0, s, dtail, 0u, nfin, dD, dS);
        } else { // the timed classes apart
            if (nfin) hipLaunchKernelGGL(k_btail, dim3(nfin), dim3(256), 0, s, dtail, 0u, nfin, dD, dS);
            tm->end(s);
            tm->begin(T_SPMV, s);
            hipLaunchKernelGGL(k_btail, dim3(nspmv), dim3(256), 0, s, dtail, nfin, nfin, dD, dS);
            tm->end(s);
            tm->end(s);
        }
        hipLaunchKernelGGL(k_bmdot, dim3(ndot, DOT_GROUPS), dim3(256), 0, s, ddot, dD, dS);
        hipLaunchKernelGGL(k_bmid, dim3(ndot), dim3(256), 0, s, ddot, dD, dS);
        enqueue_end();
    };
    // Without timers the step is captured once as a HIP graph (kernel nodes
    // only) and replayed; the capture is reused while the buffer and launch
    // shapes stay the same (the Newton steps of a solve, repeated solves).
    bool graph = !tm && !any_mf; // matrix-free launches carry per-instance pointers: not captured
    for (auto *J : jobs) graph = graph && J->graph;
    if (graph) {
        const GraphKey key{BB.dev, nvec, ngemv, nspmv, ncheb, nfirst, ntiny, ndot, unsigned(nb), nfin, kmax, types};
        if (!(BB.step && BB.key == key)) {
            if (BB.step) PB_HIP(hipGraphExecDestroy(BB.step));
            BB.step = nullptr;
            if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) == hipSuccess) {
                enqueue_step();
                hipGraph_t g = nullptr;
                PB_HIP(hipStreamEndCapture(s, &g));
                PB_HIP(hipGraphInstantiate(&BB.step, g, nullptr, nullptr, 0));
                PB_HIP(hipGraphDestroy(g));
                BB.key = key;
            } else {
                (void)hipGetLastError(); // a stream that cannot be captured: launch one by one
                graph = false;
            }
        }
    }
    // Enqueue steps until the control kernel's word reports every instance
    // ended, at most DEPTH of them ahead of the step reported.  An instance
    // that converges on its estimate (FIN) ends with the next step, which is
    // enqueued by then, so no further one is.
    const int DEPTH = 2;
    auto running = [&](int enqueued, int &reported, int &ending) {
        const unsigned long long v = __atomic_load_n(BB.word, __ATOMIC_ACQUIRE);
        reported = int(v >> (2 * GCOUNT_BITS));
        ending = int((v >> GCOUNT_BITS) & GCOUNT_MAX);
        return int(v & GCOUNT_MAX) < nb && !(enqueued > maxiter_host && reported >= enqueued);
    };
    enqueue_end(); // INIT: w = b, V_0
    PB_HIP(hipGetLastError());
    int enqueued = 1, reported = 0, ending = 0;
    for (int spins = 0; running(enqueued, reported, ending);) {
        if (enqueued <= maxiter_host && enqueued - reported < DEPTH && (ending < nb || enqueued == reported)) {
            if (graph) PB_HIP(hipGraphLaunch(BB.step, s));
            else enqueue_step();
            PB_HIP(hipGetLastError());
            ++enqueued;
            spins = 0;
            continue;
        }
        if (++spins % 4096) {
            std::this_thread::yield();
            continue;
        }
        // a drained stream has reported its last step; a device error shows here.
        // A query of a busy stream leaves hipErrorNotReady as the thread's last
        // error, which the launch checks would report: it is cleared.
        const hipError_t q = hipStreamQuery(s);
        if (q == hipErrorNotReady) {
            (void)hipGetLastError();
            continue;
        }
        PB_HIP(q);
        running(enqueued, reported, ending);
        PB_CHECK(reported >= enqueued, PBFB_EDEVICE, "a Krylov step did not report its end");
    }
    PB_HIP(hipStreamSynchronize(s));
    std::copy(BB.state, BB.state + nb, st.begin());
    for (int q = 0; q < nb; ++q) {
        GmresJob &J = *jobs[q];
        J.iters = st[q].total;
        J.applies = st[q].napply;
        if (st[q].st == G_DONE) J.status = 0;
        else if (st[q].st == G_FAIL) J.status = st[q].code;
        else J.status = PBFB_ENOTCONV;
    }
}

} // namespace pbfb
