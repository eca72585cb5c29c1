// Matrix-free boundary-element apply, for instances whose dense Galerkin
// operators would not fit the device: every apply evaluates the regular
// (non-touching) part of [K' | V'] x as a quadrature-point N-body sum and
// adds the touching-pair blocks and 1/2 M from small resident tables
// (Sec. 2.2, eq. KV; the paper switches to a fast multipole method above
// 90k vertices for the same reason).
//
//   1. k_mf_src: per source triangle sigma and rule point y_q the strengths
//      s_V w_q |sigma| lambda_h(y_q) and s_K w_q |sigma| u_h(y_q);
//   2. k_mf_tile: the unordered pairs of 64-triangle blocks (a <= b).  The
//      kernels are symmetric in their two points, so a pair of triangles is
//      evaluated once and serves both directions (the double layers differ
//      only in the normal distance, which is the same for the six points of
//      one panel against a point of the other).  Sums over a triangle's six
//      points in the evaluation precision, as in the dense assembly, single
//      and double layer apart; the two are added, and the sums over triangles
//      formed, in FP64; each block pair leaves the corner values
//      |tau| / (4 pi) sum_p w_p b_p[a] (potential at x_p) it contributes to
//      either block in a slot of its own;
//   3. k_mf_sum: the slots of each block added in a fixed order;
//   4. k_mf_gather: per vertex, the corner values of its triangles, the
//      touching-pair blocks (Sauter-Schwab, FP64, computed once at setup)
//      and the P1 mass, in a fixed order.
// No atomics between workgroups, so the result is bitwise reproducible.
//
// The same integrals as the dense operator, summed in another order.
#include <algorithm>
#include <cmath>

#include "bem_quad.hpp"
#include "pbfb_internal.hpp"

namespace pbfb {

constexpr int MF_T = 64;                 // triangles per block
constexpr int MF_W = 4;                  // wavefronts per block pair
constexpr int MF_SLOT = 3 * MF_T;        // corner values one block pair leaves to a block
// Slots held at once: 32 MiB, which the per-request memory estimate covers
// with its constant part.  Surfaces of more than 147 blocks are swept in
// pairs of block groups.
constexpr int64_t MF_SLOTS = (int64_t(32) << 20) / (8 * MF_SLOT);

static inline unsigned nbk_(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }

// batched use: only an instance in its Arnoldi or restart-residual phase applies
__device__ inline bool mf_active(const int *st) { return !st || *st == G_ARN || *st == G_RES; }

__global__ void k_mf_src(int64_t nt, int64_t nv, const int32_t *__restrict__ m_tri, const double *__restrict__ m_area,
                         const double *__restrict__ x, double sV, double sK, QRule6 R, const int *__restrict__ st,
                         double *__restrict__ sl, double *__restrict__ su)
{
    if (!mf_active(st)) return;
    const int64_t m = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (m >= nt) return;
    const int32_t v0 = m_tri[3 * m], v1 = m_tri[3 * m + 1], v2 = m_tri[3 * m + 2];
    const double u0 = x[v0], u1 = x[v1], u2 = x[v2];
    const double l0 = x[nv + v0], l1 = x[nv + v1], l2 = x[nv + v2];
    const double ar = m_area[m];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const double wq = R.w[q] * ar;
        sl[6 * m + q] = sV * wq * (R.b[q][0] * l0 + R.b[q][1] * l1 + R.b[q][2] * l2);
        su[6 * m + q] = sK * wq * (R.b[q][0] * u0 + R.b[q][1] * u1 + R.b[q][2] * u2);
    }
}

// The tile of a block pair (a, b): blocks a0 + .. and b0 + .. of one pair of
// groups (tri: the two groups are the same and only a <= b is launched, tile
// k = bl (bl + 1) / 2 + al; otherwise k = bl * na + al).  Lane i of every
// wavefront holds target triangle i of block a; wavefront w takes the steps
// s = 16 w .. 16 w + 15, in which lane i meets source triangle (i + s) mod 64
// of block b, read from LDS.  In one step the lanes of a wavefront meet 64
// different source triangles, so what they add to the sources' potentials
// (one LDS array per wavefront) never collides within a step; the next step
// moves every source on to the next lane, so a wavefront fence separates the
// steps.  Targets accumulate in registers.  Both are added over the wavefronts
// in a fixed order at the end.
// fwd: slots [bl][al] of the targets (row length na), rev: slots [al][bl] of
// the sources (row length nb); a diagonal tile meets every ordered pair as a
// target and leaves no reverse slot.
//
// Bound by FP64 / FP32 vector issue (about 21 instruction slots per
// quadrature pair and two directions for FP64 Laplace, 43 for Yukawa).
// Whole products of both surfaces: 13.6 -> 5.5 ms (FP64, 11 520 triangles)
// and 17.6 -> 8.0 ms (FP32 evaluation, 20 480 triangles) against one thread
// per target and source triangle that read the source from LDS at every
// quadrature pair (five LDS reads a pair) and served one direction.
//
// RT = double: FP64 positions (xq, nq: Morton-ordered points and normals)
// RT = float : FP32 offsets from FP64 centroids (cen)
template <bool YUK, typename RT>
__global__ void __launch_bounds__(64 * MF_W, sizeof(RT) == 8 ? 3 : 4)
    k_mf_tile(int64_t nt, int64_t a0, int64_t b0, int64_t na, int64_t nb, int tri, const int32_t *__restrict__ m_tri,
              const RT *__restrict__ xq, const RT *__restrict__ nq, const double *__restrict__ cen,
              const double *__restrict__ m_area, const double *__restrict__ sl, const double *__restrict__ su,
              double kappa, QRule6 R, const int *__restrict__ st, double *__restrict__ fwd, double *__restrict__ rev)
{
    if (!mf_active(st)) return;
    constexpr bool F32 = sizeof(RT) == 4;
    constexpr int NSRC = 33; // values per source triangle: 18 coordinates, 6 + 6 strengths, normal
    constexpr size_t SRC = sizeof(RT) * NSRC * MF_T, FW = sizeof(double) * MF_W * 6 * MF_T;
    __shared__ alignas(16) unsigned char raw[SRC > FW ? SRC : FW]; // the sources, later the targets' sums
    __shared__ double sC[F32 ? 3 : 1][MF_T];
    __shared__ int sV[3][MF_T];
    __shared__ double acc[MF_W][6][MF_T]; // what the sources collect
    RT(*src)[MF_T] = reinterpret_cast<RT(*)[MF_T]>(raw);

    int64_t al, bl;
    {
        const int64_t k = blockIdx.x;
        if (tri) {
            bl = int64_t((sqrt(8.0 * double(k) + 1.0) - 1.0) * 0.5);
            while (bl * (bl + 1) / 2 > k) --bl;
            while ((bl + 1) * (bl + 2) / 2 <= k) ++bl;
            al = k - bl * (bl + 1) / 2;
        } else {
            bl = k / na;
            al = k - bl * na;
        }
    }
    const int64_t a = a0 + al, b = b0 + bl;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // a block's data are contiguous; triangles past the end get zeros and meet nothing
    const int64_t eB = nt - b * MF_T;
    for (int k = tid; k < 18 * MF_T; k += 64 * MF_W) {
        const int t = k / 18, c = k % 18;
        src[c][t] = t < eB ? xq[18 * b * MF_T + k] : RT(0);
    }
    for (int k = tid; k < 6 * MF_T; k += 64 * MF_W) {
        const int t = k / 6, c = k % 6;
        src[18 + c][t] = t < eB ? RT(sl[6 * b * MF_T + k]) : RT(0);
        src[24 + c][t] = t < eB ? RT(su[6 * b * MF_T + k]) : RT(0);
    }
    if (tid < 3 * MF_T) {
        const int t = tid / 3, c = tid % 3;
        src[30 + c][t] = t < eB ? nq[3 * b * MF_T + tid] : RT(0);
        sV[c][t] = t < eB ? m_tri[3 * b * MF_T + tid] : -1;
        if constexpr (F32) sC[c][t] = t < eB ? cen[3 * b * MF_T + tid] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) acc[w][q][lane] = 0.0;

    // this lane's target triangle
    const int64_t mA = a * MF_T + lane;
    const bool inA = mA < nt;
    const int64_t mt = inA ? mA : 0;
    RT X[18], tl[6], tu[6], m0, m1, m2;
#pragma unroll
    for (int k = 0; k < 18; ++k) X[k] = xq[18 * mt + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        tl[k] = RT(sl[6 * mt + k]);
        tu[k] = RT(su[6 * mt + k]);
    }
    m0 = nq[3 * mt];
    m1 = nq[3 * mt + 1];
    m2 = nq[3 * mt + 2];
    const int v0 = inA ? m_tri[3 * mt] : -2, v1 = inA ? m_tri[3 * mt + 1] : -2, v2 = inA ? m_tri[3 * mt + 2] : -2;
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    if constexpr (F32) {
        g0 = cen[3 * mt];
        g1 = cen[3 * mt + 1];
        g2 = cen[3 * mt + 2];
    }
    const RT kap = RT(kappa);
    const RT kl2 = RT(-1.44269504088896341 * kappa); // FP32: e^{-kappa r} = 2^{kl2 r}
    double P[6];
#pragma unroll
    for (int p = 0; p < 6; ++p) P[p] = 0.0;
    __syncthreads();

#pragma unroll 1
    for (int k = 0; k < MF_T / MF_W; ++k) {
        const int j = (lane + w * (MF_T / MF_W) + k) & 63;
        const int u0 = sV[0][j], u1 = sV[1][j], u2 = sV[2][j];
        bool skip = !inA || u0 < 0;
        skip |= (v0 == u0) | (v0 == u1) | (v0 == u2) | (v1 == u0) | (v1 == u1) | (v1 == u2) | (v2 == u0) |
                (v2 == u1) | (v2 == u2);
        if (!skip) {
            RT c0 = 0, c1 = 0, c2 = 0; // FP32: target centroid relative to the source's
            if constexpr (F32) {
                c0 = float(g0 - sC[0][j]);
                c1 = float(g1 - sC[1][j]);
                c2 = float(g2 - sC[2][j]);
            }
            RT av[6], ak[6]; // the target points' sums (av: FP32 only)
#pragma unroll
            for (int p = 0; p < 6; ++p) av[p] = ak[p] = RT(0);
#pragma unroll 1
            for (int q = 0; q < 6; ++q) {
                RT y0 = src[3 * q][j], y1 = src[3 * q + 1][j], y2 = src[3 * q + 2][j];
                if constexpr (F32) {
                    y0 -= c0;
                    y1 -= c1;
                    y2 -= c2;
                }
                const RT ql = src[18 + q][j], qu = src[24 + q][j];
                // (y_q - x).n_tau, the same for the six target points
                const RT dm = (y0 - X[0]) * m0 + (y1 - X[1]) * m1 + (y2 - X[2]) * m2;
                RT bv = RT(0), bk = RT(0);
#pragma unroll
                for (int p = 0; p < 6; ++p) {
                    const RT d0 = X[3 * p] - y0, d1 = X[3 * p + 1] - y1, d2 = X[3 * p + 2] - y2;
                    const RT r2 = d0 * d0 + d1 * d1 + d2 * d2;
                    const RT ri = rsqrt_pos(r2);
                    RT gv, hk; // single-layer kernel, double-layer kernel / normal distance
                    if constexpr (YUK) {
                        const RT r = r2 * ri;
                        RT e;
                        if constexpr (F32) e = __builtin_amdgcn_exp2f(kl2 * r);
                        else e = exp_neg(kap * r);
                        gv = e * ri;
                        hk = gv * ri * (ri + kap); // e (1 + kappa r) / r^3
                    } else {
                        gv = ri;
                        hk = ri * ri * ri;
                    }
                    if constexpr (F32) av[p] = fma(gv, ql, av[p]);
                    else P[p] = fma(gv, ql, P[p]);
                    ak[p] = fma(hk, qu, ak[p]);
                    bv = fma(gv, tl[p], bv);
                    bk = fma(hk, tu[p], bk);
                }
                if constexpr (F32) acc[w][q][j] += double(bv) + double(bk * dm);
                else acc[w][q][j] += fma(bk, dm, bv);
            }
            RT y0 = src[0][j], y1 = src[1][j], y2 = src[2][j];
            if constexpr (F32) {
                y0 -= c0;
                y1 -= c1;
                y2 -= c2;
            }
            const RT n0 = src[30][j], n1 = src[31][j], n2 = src[32][j];
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                const RT dn = (X[3 * p] - y0) * n0 + (X[3 * p + 1] - y1) * n1 + (X[3 * p + 2] - y2) * n2;
                if constexpr (F32) P[p] += double(av[p]) + double(ak[p] * dn);
                else P[p] = fma(ak[p], dn, P[p]);
            }
        }
        // lane i - 1 adds to this source next: no access to acc may cross the
        // steps (a wavefront's LDS operations complete in order, so the fence
        // binds the compiler only and costs no instruction)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads(); // the sources are no longer read: their space takes the targets' sums
    double(*fw)[6][MF_T] = reinterpret_cast<double(*)[6][MF_T]>(raw);
#pragma unroll
    for (int p = 0; p < 6; ++p) fw[w][p][lane] = P[p];
    __syncthreads();
    if (tid >= MF_SLOT) return;
    const int t = tid & 63, corner = tid >> 6;
    auto out = [&](const double(*s)[6][MF_T], int64_t m) {
        double y = 0.0;
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            const double v = (s[0][p][t] + s[1][p][t]) + (s[2][p][t] + s[3][p][t]);
            y += (corner == 0 ? R.wb[p][0] : corner == 1 ? R.wb[p][1] : R.wb[p][2]) * v;
        }
        return m < nt ? m_area[m] * INV4PI * y : 0.0;
    };
    static_assert(MF_W == 4, "four partial sums");
    fwd[(bl * na + al) * MF_SLOT + tid] = out(fw, a * MF_T + t);
    if (!(tri && al == bl)) rev[(al * nb + bl) * MF_SLOT + tid] = out(acc, b * MF_T + t);
}

// Yc of the blocks x0 + .. (one workgroup of 256 threads per 64 corner
// values): the slots [row][block] of `rows` rows, four interleaved partial
// sums per value, added to Yc (add) or stored
__global__ void __launch_bounds__(256)
    k_mf_sum(int64_t nt, int64_t x0, int64_t nx, int64_t rows, int add, const double *__restrict__ slots,
             const int *__restrict__ st, double *__restrict__ Yc)
{
    if (!mf_active(st)) return;
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t x = blockIdx.x / 3;
    const int corner = int(blockIdx.x % 3);
    double s = 0.0;
#pragma unroll 8
    for (int64_t r = g; r < rows; r += 4) s += slots[(r * nx + x) * MF_SLOT + corner * 64 + lane];
    red[g][lane] = s;
    __syncthreads();
    const int64_t m = (x0 + x) * MF_T + lane;
    if (g != 0 || m >= nt) return;
    const double v = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    double &y = Yc[3 * m + corner];
    y = add ? y + v : v;
}

// y_i = corner values of the triangles at i + touching-pair blocks + 1/2 M:
// eight lanes per vertex, each taking every eighth triangle at it, added by
// a fixed xor-shuffle tree (one thread per vertex walks about 80 blocks one
// after the other: 89 us per surface of 11 520 triangles)
__global__ void __launch_bounds__(256)
    k_mf_gather(int64_t nv, const int32_t *__restrict__ v2t_ptr, const int32_t *__restrict__ v2t,
                const int32_t *__restrict__ tri, const int32_t *__restrict__ mpos, const int32_t *__restrict__ tp_ptr,
                const int32_t *__restrict__ tp_sig, const double *__restrict__ tpv, const double *__restrict__ area,
                const double *__restrict__ Yc, const double *__restrict__ x, double sV, double sK,
                const int *__restrict__ st, double *__restrict__ y)
{
    if (!mf_active(st)) return;
    const int64_t i = (blockIdx.x * int64_t(256) + threadIdx.x) >> 3;
    const int l = threadIdx.x & 7;
    double acc = 0.0;
    if (i < nv)
        for (int32_t e = v2t_ptr[i] + l; e < v2t_ptr[i + 1]; e += 8) {
            const int32_t ta = v2t[e] / 3, a = v2t[e] % 3;
            acc += Yc[3 * int64_t(mpos[ta]) + a];
            for (int32_t pp = tp_ptr[ta]; pp < tp_ptr[ta + 1]; ++pp) {
                const int32_t sb = tp_sig[pp];
                const double *blk = tpv + 18 * int64_t(pp);
                for (int b = 0; b < 3; ++b) {
                    const int32_t j = tri[3 * sb + b];
                    acc += sV * blk[3 * a + b] * x[nv + j] + sK * blk[9 + 3 * a + b] * x[j];
                }
            }
            for (int b = 0; b < 3; ++b) acc += 0.5 * area[ta] * (a == b ? 2.0 : 1.0) / 12.0 * x[tri[3 * ta + b]];
        }
    for (int off = 4; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 8);
    if (l == 0 && i < nv) y[i] = acc;
}

void mf_apply(Problem &p, int w, const double *x, double *y, const int *st, hipStream_t s)
{
    const SurfaceDev &S = p.surf[w];
    const int64_t nt = S.nt, nv = S.nv;
    const bool yuk = (w == 1) && p.kappa > 0.0;
    const double kappa = (w == 1) ? p.kappa : 0.0;
    const double sV = (w == 0) ? -1.0 : 1.0, sK = (w == 0) ? 1.0 : -1.0;
    const int base = w == 0 ? SCR_MF0 : SCR_MF1;
    double *sl = scratch<double>(p, base, 15 * size_t(nt));
    double *su = sl + 6 * nt, *Yc = su + 6 * nt;
    const QRule6 R = q6arg();
    hipLaunchKernelGGL(k_mf_src, dim3(nbk_(nt, 256)), dim3(256), 0, s, nt, nv, S.m_tri, S.m_area, x, sV, sK, R, st,
                       sl, su);
    // One group of all blocks if its nb x nb slots fit; else groups of G
    // blocks, first each with itself (which stores Yc), then each pair of
    // groups with the slots of both directions (which adds)
    const int64_t nb = nbk_(nt, MF_T);
    int64_t G = nb;
    if (nb * nb > MF_SLOTS)
        for (G = 1; 2 * (G + 1) * (G + 1) <= MF_SLOTS;) ++G;
    const int64_t ng = (nb + G - 1) / G;
    double *slots = scratch<double>(p, SCR_MF2, size_t(std::min(ng > 1 ? 2 * G * G : G * G, MF_SLOTS)) * MF_SLOT);
    auto tiles = [&](int64_t ga, int64_t gb) {
        const int64_t a0 = ga * G, b0 = gb * G, na = std::min(G, nb - a0), nbb = std::min(G, nb - b0);
        const int tri = ga == gb ? 1 : 0;
        // the same group: both directions in one slot array (rows and columns are the same blocks)
        double *fwd = slots, *rev = tri ? slots : slots + na * nbb * MF_SLOT;
        const dim3 grid(unsigned(tri ? na * (na + 1) / 2 : na * nbb));
#define PB_MF(Y, RT, xq, nq, cen)                                                                                  \
    hipLaunchKernelGGL((k_mf_tile<Y, RT>), grid, dim3(64 * MF_W), 0, s, nt, a0, b0, na, nbb, tri, S.m_tri, xq, nq, \
                       cen, S.m_area, sl, su, kappa, R, st, fwd, rev)
        if (p.precision == PBFB_MIXED) {
            if (yuk) PB_MF(true, float, S.m_qf, S.m_nf, S.m_cen);
            else PB_MF(false, float, S.m_qf, S.m_nf, S.m_cen);
        } else {
            if (yuk) PB_MF(true, double, S.m_qp, S.m_nrm, (const double *)nullptr);
            else PB_MF(false, double, S.m_qp, S.m_nrm, (const double *)nullptr);
        }
#undef PB_MF
        hipLaunchKernelGGL(k_mf_sum, dim3(unsigned(3 * na)), dim3(256), 0, s, nt, a0, na, nbb, tri ? 0 : 1, fwd, st, Yc);
        if (!tri)
            hipLaunchKernelGGL(k_mf_sum, dim3(unsigned(3 * nbb)), dim3(256), 0, s, nt, b0, nbb, na, 1, rev, st, Yc);
    };
    for (int64_t ga = 0; ga < ng; ++ga) tiles(ga, ga);
    for (int64_t ga = 0; ga < ng; ++ga)
        for (int64_t gb = ga + 1; gb < ng; ++gb) tiles(ga, gb);
    hipLaunchKernelGGL(k_mf_gather, dim3(nbk_(nv * 8, 256)), dim3(256), 0, s, nv, S.v2t_ptr, S.v2t, S.tri, S.mpos,
                       S.tp_ptr, S.tp_sig, S.tpv, S.area, Yc, x, sV, sK, st, y);
    PB_HIP(hipGetLastError());
}

} // namespace pbfb

namespace pbfb {

// diagonal of the signed single layer V': only touching pairs (every pair of
// triangles at a vertex shares it) reach the diagonal
__global__ void k_mf_vdiag(int64_t nv, const int32_t *__restrict__ v2t_ptr, const int32_t *__restrict__ v2t,
                           const int32_t *__restrict__ tri, const int32_t *__restrict__ tp_ptr,
                           const int32_t *__restrict__ tp_sig, const double *__restrict__ tpv, double sV,
                           double *__restrict__ vdiag)
{
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i >= nv) return;
    double acc = 0.0;
    for (int32_t e = v2t_ptr[i]; e < v2t_ptr[i + 1]; ++e) {
        const int32_t ta = v2t[e] / 3, a = v2t[e] % 3;
        for (int32_t pp = tp_ptr[ta]; pp < tp_ptr[ta + 1]; ++pp) {
            const int32_t sb = tp_sig[pp];
            for (int b = 0; b < 3; ++b)
                if (tri[3 * sb + b] == i) acc += tpv[18 * int64_t(pp) + 3 * a + b];
        }
    }
    vdiag[i] = sV * acc;
}

void mf_vdiag(Problem &p, int w, hipStream_t s)
{
    const SurfaceDev &S = p.surf[w];
    hipLaunchKernelGGL(k_mf_vdiag, dim3(nbk_(S.nv, 256)), dim3(256), 0, s, S.nv, S.v2t_ptr, S.v2t, S.tri, S.tp_ptr,
                       S.tp_sig, S.tpv, (w == 0) ? -1.0 : 1.0, S.vdiag);
    PB_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// preconditioner of the single layers without stored rows: the 1-ring
// sparse approximate inverse (row i minimises || m^T V' - e_i^T ||_2 over m
// on the 1-ring P(i)) built from the near field of V' instead of its full
// rows.  The near field keeps, for every row a, the columns within three
// rings of a, each entry the same Galerkin integral as the dense operator
// (touching pairs from the resident blocks, the others by the 6 x 6 rule).
// ---------------------------------------------------------------------------
// entry e = (a, c): sum over triangles tau at a and sigma at c (one thread per entry)
template <bool YUK>
__global__ void k_mf_near(int64_t nnz, const int32_t *__restrict__ nf_row, const int32_t *__restrict__ nf_col,
                          const int32_t *__restrict__ v2t_ptr, const int32_t *__restrict__ v2t,
                          const int32_t *__restrict__ tp_ptr, const int32_t *__restrict__ tp_sig,
                          const double *__restrict__ tpv, const double *__restrict__ qp,
                          const double *__restrict__ area, double kappa, double sV, QRule6 R,
                          double *__restrict__ nf_val)
{
    const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (e >= nnz) return;
    const int32_t a = nf_row[e], c = nf_col[e];
    double acc = 0.0;
    for (int32_t ea = v2t_ptr[a]; ea < v2t_ptr[a + 1]; ++ea) {
        const int32_t ta = v2t[ea] / 3, la = v2t[ea] % 3;
        for (int32_t ec = v2t_ptr[c]; ec < v2t_ptr[c + 1]; ++ec) {
            const int32_t sc = v2t[ec] / 3, lc = v2t[ec] % 3;
            int32_t pp = -1;
            for (int32_t k = tp_ptr[ta]; k < tp_ptr[ta + 1]; ++k)
                if (tp_sig[k] == sc) {
                    pp = k;
                    break;
                }
            if (pp >= 0) { // touching pair: the resident V block
                acc += tpv[18 * int64_t(pp) + 3 * la + lc];
                continue;
            }
            const double *X = qp + 18 * int64_t(ta), *Y = qp + 18 * int64_t(sc);
            double sum = 0.0;
            for (int p = 0; p < 6; ++p) {
                double sp = 0.0;
                for (int q = 0; q < 6; ++q) {
                    const double d0 = X[3 * p] - Y[3 * q], d1 = X[3 * p + 1] - Y[3 * q + 1],
                                 d2 = X[3 * p + 2] - Y[3 * q + 2];
                    const double r = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
                    const double g = YUK ? exp(-kappa * r) / r : 1.0 / r;
                    sp += R.w[q] * R.b[q][lc] * g;
                }
                sum += R.w[p] * R.b[p][la] * sp;
            }
            acc += area[ta] * area[sc] * INV4PI * sum;
        }
    }
    nf_val[e] = sV * acc;
}

// one 64-thread workgroup per row i: lanes take the (a, b) pairs of the Gram
// matrix of the near-field rows P(i), each a merge of two ascending sparse
// rows; lane 0 solves the normal equations by Cholesky
__global__ void __launch_bounds__(64)
    k_mf_spai(int64_t nv, const int32_t *__restrict__ ring_ptr, const int32_t *__restrict__ ring,
              const int32_t *__restrict__ nf_ptr, const int32_t *__restrict__ nf_col,
              const double *__restrict__ nf_val, double *__restrict__ val, int *__restrict__ bad)
{
    __shared__ double G[MAXRING][MAXRING + 1];
    __shared__ double rhs[MAXRING];
    const int lane = threadIdx.x;
    const int64_t i = blockIdx.x;
    if (i >= nv) return;
    const int p0 = ring_ptr[i], m = ring_ptr[i + 1] - p0;
    const int npair = m * (m + 1) / 2;
    for (int pr = lane; pr < npair; pr += 64) {
        int a = int((sqrt(8.0 * pr + 1.0) - 1.0) * 0.5);
        while (a * (a + 1) / 2 > pr) --a;
        while ((a + 1) * (a + 2) / 2 <= pr) ++a;
        const int b = pr - a * (a + 1) / 2;
        const int32_t ra = ring[p0 + a], rb = ring[p0 + b];
        int32_t ka = nf_ptr[ra], kb = nf_ptr[rb];
        const int32_t ea = nf_ptr[ra + 1], eb = nf_ptr[rb + 1];
        double sum = 0.0;
        while (ka < ea && kb < eb) {
            const int32_t ca = nf_col[ka], cb = nf_col[kb];
            if (ca == cb) sum = fma(nf_val[ka++], nf_val[kb++], sum);
            else if (ca < cb) ++ka;
            else ++kb;
        }
        G[a][b] = G[b][a] = sum;
    }
    for (int a = lane; a < m; a += 64) {
        const int32_t ra = ring[p0 + a];
        double v = 0.0; // V'(P_a, i): i is in the 1-ring of P_a, hence in its pattern
        for (int32_t k = nf_ptr[ra]; k < nf_ptr[ra + 1]; ++k)
            if (nf_col[k] == int32_t(i)) v = nf_val[k];
        rhs[a] = v;
    }
    __syncthreads();
    if (lane != 0) return;
    bool ok = true;
    for (int a = 0; a < m && ok; ++a) {
        double d = G[a][a];
        for (int k = 0; k < a; ++k) d -= G[a][k] * G[a][k];
        if (!(d > 0.0)) {
            ok = false;
            break;
        }
        G[a][a] = sqrt(d);
        for (int b = a + 1; b < m; ++b) {
            double t = G[b][a];
            for (int k = 0; k < a; ++k) t -= G[b][k] * G[a][k];
            G[b][a] = t / G[a][a];
        }
    }
    if (!ok) {
        atomicOr(bad, 4);
        for (int a = 0; a < m; ++a) val[p0 + a] = 0.0;
        return;
    }
    for (int a = 0; a < m; ++a) {
        double t = rhs[a];
        for (int k = 0; k < a; ++k) t -= G[a][k] * rhs[k];
        rhs[a] = t / G[a][a];
    }
    for (int a = m - 1; a >= 0; --a) {
        double t = rhs[a];
        for (int k = a + 1; k < m; ++k) t -= G[k][a] * rhs[k];
        rhs[a] = t / G[a][a];
    }
    for (int a = 0; a < m; ++a) val[p0 + a] = rhs[a];
}

void mf_spai(Problem &p, int w, hipStream_t s)
{
    const SurfaceDev &S = p.surf[w];
    const bool yuk = (w == 1) && p.kappa > 0.0;
    const double kappa = (w == 1) ? p.kappa : 0.0, sV = (w == 0) ? -1.0 : 1.0;
    const QRule6 R = q6arg();
    const dim3 g(nbk_(S.nf_nnz, 256));
    if (yuk)
        hipLaunchKernelGGL(k_mf_near<true>, g, dim3(256), 0, s, S.nf_nnz, S.nf_row, S.nf_col, S.v2t_ptr, S.v2t,
                           S.tp_ptr, S.tp_sig, S.tpv, S.qp, S.area, kappa, sV, R, S.nf_val);
    else
        hipLaunchKernelGGL(k_mf_near<false>, g, dim3(256), 0, s, S.nf_nnz, S.nf_row, S.nf_col, S.v2t_ptr, S.v2t,
                           S.tp_ptr, S.tp_sig, S.tpv, S.qp, S.area, kappa, sV, R, S.nf_val);
    hipLaunchKernelGGL(k_mf_spai, dim3(unsigned(S.nv)), dim3(64), 0, s, S.nv, S.ring_ptr, S.ring, S.nf_ptr, S.nf_col,
                       S.nf_val, S.spai, p.d_bad);
    PB_HIP(hipGetLastError());
}

} // namespace pbfb
