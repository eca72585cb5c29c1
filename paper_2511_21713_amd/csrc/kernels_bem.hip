// Dense Galerkin P1 boundary operators on one surface:
//   V_ij = int int zeta_i(x) g(x,y) zeta_j(y),   K_ij = int int zeta_i(x) dg/dn_y zeta_j(y),
//   g = exp(-kappa r) / (4 pi r)   (Sec. 2.2 Yukawa kernel; kappa = 0: Sec. 2.3 Laplace kernel)
// stored as one row-major matrix per surface, row i = [K'_i | V'_i] with
//   Gamma_m: K' = 1/2 M + K0,  V' = -V0   (interior Laplace equation)
//   Gamma_s: K' = 1/2 M - Kk,  V' = +Vk   (exterior Yukawa equation)
// so the Galerkin rows of the coupled operator are one dense GEMV each.
//
// Rows and columns follow the Morton vertex order (first appearance along
// the Morton-ordered triangles; SurfaceTopo::mvert), so the vertices of a
// block of consecutive triangles are nearby rows and columns.
//
// Assembly, deterministic and free of atomics, straight into that storage:
//  1. regular tiles: a workgroup takes TA target x TB source Morton-ordered
//     triangles (shape chosen by an autotuner), evaluates the 6 x 6 product
//     rule for every non-touching pair, reduces the 3x3 pair blocks to the
//     blocks' vertices in LDS and adds the result into the stored operator.
//     The triangle blocks are coloured so that blocks of one colour share no
//     vertex; one launch per colour pair then has tiles that touch disjoint
//     entries, and the launches run one after the other, so every entry
//     receives its contributions in a fixed order.  Square shapes evaluate
//     each unordered pair once and also add the double layer of the
//     mirrored pair to an nv x nv matrix T in the context's workspace.  Small
//     surfaces run every tile in one launch, each into entries of its own in
//     planes over the blocks' local vertices, and a second one adds them up in
//     the colour pairs' order (k_bem_gather; the same bits);
//  2. square shapes: a transpose pass completes V' = U + U^T and K' += T^T
//     (the regular part of V' bitwise symmetric);
//  3. touching pairs (identical, common edge, common vertex) are integrated
//     with the Sauter-Schwab rules (one lane per pair) and added, with
//     the 1/2 M term, by a row-owned scatter.
//
// In mixed precision the regular tiles evaluate the kernels in FP32: each
// quadrature point is held as an FP32 offset from its triangle's centroid,
// the centroid difference of a pair is formed in FP64 and rounded once, so
// x - y never cancels large coordinates in FP32.  A pair's 3x3 V and K
// blocks are summed over its 36 quadrature pairs in FP32, and so are the
// fold's corner sums onto a tile's vertices (at most MAXS terms each); each
// tile's sum is added to the FP32 stored entry in FP64 and rounded once (an
// entry receives one tile's sum for each pair of blocks holding its two
// vertices).  The touching pairs stay FP64 throughout.
#include <chrono>
#include <cmath>
#include <thread>
#include <type_traits>

#include "bem_quad.hpp"
#include "gemv_rows.hpp"
#include "pbfb_internal.hpp"

namespace pbfb {

static inline unsigned nblk(int64_t n, int bs) { return unsigned((n + bs - 1) / bs); }



// Morton-ordered copies of the triangle data used by the regular assembly.
// FP64 evaluation reads m_qp/m_nrm; FP32 evaluation reads m_cen/m_qf/m_nf
// (whichever pointers are non-null are written).
__global__ void k_tri_morton(int64_t nt, const int32_t *__restrict__ morton, const int32_t *__restrict__ tri,
                             const double *__restrict__ qp, const double *__restrict__ nrm,
                             const double *__restrict__ area, const int32_t *__restrict__ g,
                             const double *__restrict__ x, int32_t *__restrict__ m_tri, double *__restrict__ m_qp,
                             double *__restrict__ m_nrm, double *__restrict__ m_area, double *__restrict__ m_cen,
                             float *__restrict__ m_qf, float *__restrict__ m_nf)
{
    int64_t m = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (m >= nt) return;
    int32_t t = morton[m];
    for (int k = 0; k < 3; ++k) m_tri[3 * m + k] = tri[3 * t + k];
    m_area[m] = area[t];
    if (m_qp) {
        for (int k = 0; k < 3; ++k) m_nrm[3 * m + k] = nrm[3 * t + k];
        for (int k = 0; k < 18; ++k) m_qp[18 * m + k] = qp[18 * t + k];
    }
    if (m_cen) {
        double c[3];
        for (int d = 0; d < 3; ++d)
            c[d] = (x[3 * g[tri[3 * t]] + d] + x[3 * g[tri[3 * t + 1]] + d] + x[3 * g[tri[3 * t + 2]] + d]) / 3.0;
        for (int d = 0; d < 3; ++d) {
            m_cen[3 * m + d] = c[d];
            m_nf[3 * m + d] = float(nrm[3 * t + d]);
        }
        for (int q = 0; q < 6; ++q)
            for (int d = 0; d < 3; ++d) m_qf[18 * m + 3 * q + d] = float(qp[18 * t + 3 * q + d] - c[d]);
    }
}

// ---------------------------------------------------------------------------
// 1. regular tiles
// ---------------------------------------------------------------------------


// Read-modify-write of one folded operator entry into the stored operator
// (FP64 or FP32 storage; the sum is formed in FP64 and rounded once).  No
// other thread of the launch touches the same entry (the launch's tiles have
// vertex-disjoint target blocks and vertex-disjoint source blocks).
template <typename MT> __device__ inline void add_entry(MT *__restrict__ U, int64_t at, double v)
{
    U[at] = MT(double(U[at]) + v);
}

// The fold of a tile's 3x3 pair blocks onto the blocks' vertices, in LDS
// planes of one block per pair.  Rows and columns are permuted so that the
// corners of one local vertex lie side by side (BlockSide::cpos; seg: first
// position and number of each vertex), which gives both passes exact,
// wavefront-uniform trip counts and addresses:
//  1. a wavefront takes a source vertex at a time, a lane per tile row: its
//     columns are added up into the first of them, in place (a vertex with one
//     corner in the block needs nothing);
//  2. a wavefront takes a target vertex at a time, a lane per (plane, source
//     vertex): its rows are added up and the sum goes into the operator.
// Corners are added in ascending order.  A fold over corner lists padded to
// the longest (6 of 2.6 on average, the absent ones reading a zero row or
// column) took a third of the tiles' vector instructions (1 324 per wavefront
// in FP32, now 1 050), and operator entries and inputs read under conditions
// or in loops, each with a wait of its own, most of the waiting.  Per surface
// (mean of Laplace and Yukawa): 10 242 vertices FP64 18.3 -> 16.2 ms, FP32
// 10.5 -> 8.8, 40 962 vertices FP32 152.9 -> 133.3.  FP32 tiles are now bound
// by vector issue (86 % busy), FP64 ones by that (56 % Laplace, 74 % Yukawa)
// and by what four wavefronts per SIMD leave waiting.
//
// Operator entries: plane V to U + offV, plane K to U, the mirrored K to T.
template <typename MT> struct FoldOut {
    MT *U, *T;
    int64_t offV, ld, ldT;
    double sV, sK;
};
template <int TB> constexpr int fold_rs() { return TB * 3 + 1; } // row stride, odd
template <int TA, int TB> constexpr int fold_ps() { return TA * 3 * fold_rs<TB>(); }
// FP64 V and K alternate, so that a pair of values moves at once: the first
// store's columns, in no order, collide less (LDS conflicts 598 -> 172 cycles
// per wavefront, 10 242 vertices 17.2 -> 16.2 ms).  FP32, three planes and
// bound by vector issue, has them one after the other.
template <int NP, typename ST> constexpr bool fold_pairs() { return NP == 2 && sizeof(ST) == 8; }

// lane t of the second pass over NP planes from plane FIRST (0: V, 1: K, 2: mirrored K)
template <typename MT> struct FoldLane {
    MT *at;
    int64_t stride;
    double sc;
    int col;
    bool on;
};
template <int TA, int TB, int FIRST, int NP, typename ST, typename MT>
__device__ inline FoldLane<MT> fold_lane(int t, int nB, const int *sIb, const int *sSb, const FoldOut<MT> &o)
{
    int q = 0, jb = t;
#pragma unroll
    for (int k = 1; k < NP; ++k)
        if (jb >= nB) {
            jb -= nB;
            ++q;
        }
    FoldLane<MT> L;
    L.on = jb < nB;
    if (!L.on) jb = 0;
    L.col = fold_pairs<NP, ST>() ? 2 * (sSb[jb] & 255) + q : q * fold_ps<TA, TB>() + (sSb[jb] & 255);
    q += FIRST;
    L.at = (q == 2 ? o.T : o.U) + (q == 0 ? o.offV : 0) + sIb[jb];
    L.stride = q == 2 ? o.ldT : o.ld;
    L.sc = q == 0 ? o.sV : o.sK;
    return L;
}

// Vertices of a wavefront's round (of 4.6 in all on average): their list
// entries come through independent scalar loads and, of a round of target
// vertices, a lane's operator entries together: the first round's before the
// quadrature (FP32) or, where they would spill, right after it (FP64), so that
// their latency hides.  No other workgroup of the launch touches them.  Six
// rows cover most blocks in one round; FP64 has registers for four.
template <typename MT> constexpr int fold_rnd() { return sizeof(MT) == 4 ? 6 : 4; }
template <bool SLOT, int NW, typename MT>
__device__ inline void fold_read(int i0, int nA, const int32_t *__restrict__ vA, const FoldLane<MT> &L,
                                 MT (&pre)[fold_rnd<MT>()])
{
    // past the end: the last row again, not used (a read under a condition
    // would be waited for where the condition ends)
#pragma unroll
    for (int k = 0; k < fold_rnd<MT>(); ++k)
        pre[k] = SLOT ? MT(0) : L.at[int64_t(vA[min(i0 + k * NW, nA - 1)]) * L.stride];
}

// sum of n values (uniform n) at q, q + step, ...
template <int STEP, typename ST> __device__ inline ST fold_sum(const ST *q, int n)
{
    auto sum = [&](auto N) {
        ST v[decltype(N)::value];
#pragma unroll
        for (int k = 0; k < decltype(N)::value; ++k) v[k] = q[k * STEP];
        ST t = v[0];
#pragma unroll
        for (int k = 1; k < decltype(N)::value; ++k) t += v[k];
        return t;
    };
    switch (n) {
    case 1: return sum(std::integral_constant<int, 1>{});
    case 2: return sum(std::integral_constant<int, 2>{});
    case 3: return sum(std::integral_constant<int, 3>{});
    case 4: return sum(std::integral_constant<int, 4>{});
    case 5: return sum(std::integral_constant<int, 5>{});
    case 6: return sum(std::integral_constant<int, 6>{});
    }
    ST t = sum(std::integral_constant<int, 6>{});
    for (int k = 6; k < n; ++k) t += q[k * STEP];
    return t;
}

// acc: NP planes, free; blk: the pair's blocks; pa, pb: the packed positions of
// the pair's triangles; segA, vA, segB: lists of the two blocks; pre: the
// entries of this wavefront's first rows (fold_read)
template <bool SLOT, int TA, int TB, int FIRST, int NP, typename ST, typename MT>
__device__ inline void fold_tile(int tid, int nA, int nB, const int32_t *__restrict__ segA,
                                 const int32_t *__restrict__ vA, const int32_t *__restrict__ segB, const int *sIb,
                                 const int *sSb, int pa, int pb, ST *acc, const ST (&blk)[NP][9],
                                 const FoldOut<MT> &o, MT (&pre)[fold_rnd<MT>()])
{
    constexpr int RND = fold_rnd<MT>();
    constexpr int NW = TA * TB / 64, RS = fold_rs<TB>(), PS = fold_ps<TA, TB>();
    constexpr bool PAIRS = fold_pairs<NP, ST>();
    constexpr int NV = PAIRS ? 1 : NP, UN = PAIRS ? 2 : 1; // vectors of UN values
    typedef ST vec __attribute__((ext_vector_type(2)));
    using V = std::conditional_t<PAIRS, vec, ST>;
    V *const accv = reinterpret_cast<V *>(acc);
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            V *q = accv + ((pa >> (8 * a)) & 255) * RS + ((pb >> (8 * b)) & 255);
            if constexpr (PAIRS) {
                *q = V{blk[0][3 * a + b], blk[1][3 * a + b]};
            } else {
#pragma unroll
                for (int pl = 0; pl < NP; ++pl) q[pl * PS] = blk[pl][3 * a + b];
            }
        }
    __syncthreads();
    for (int j0 = w; j0 < nB; j0 += NW * RND) {
        int seg[RND];
#pragma unroll
        for (int k = 0; k < RND; ++k) seg[k] = segB[min(j0 + k * NW, nB - 1)];
#pragma unroll
        for (int k = 0; k < RND; ++k) {
            const int n = seg[k] >> 8;
            if (j0 + k * NW < nB && n > 1 && lane < TA * 3) {
                V *q = accv + lane * RS + (seg[k] & 255);
                V t[NV];
#pragma unroll
                for (int pl = 0; pl < NV; ++pl) t[pl] = fold_sum<1>(q + pl * PS, n);
#pragma unroll
                for (int pl = 0; pl < NV; ++pl) q[pl * PS] = t[pl];
            }
        }
    }
    __syncthreads();
    for (int t0 = 0; t0 < NP * nB; t0 += 64) {
        const FoldLane<MT> L = fold_lane<TA, TB, FIRST, NP, ST>(t0 + lane, nB, sIb, sSb, o);
        for (int i0 = w; i0 < nA; i0 += NW * RND) {
            if (t0 > 0 || i0 > w) fold_read<SLOT, NW>(i0, nA, vA, L, pre);
            int seg[RND], v[RND];
            ST t[RND];
#pragma unroll
            for (int k = 0; k < RND; ++k) {
                seg[k] = segA[min(i0 + k * NW, nA - 1)];
                v[k] = SLOT ? i0 + k * NW : vA[min(i0 + k * NW, nA - 1)];
            }
#pragma unroll
            for (int k = 0; k < RND; ++k)
                if (i0 + k * NW < nA) {
                    t[k] = fold_sum<UN * RS>(acc + L.col + (seg[k] & 255) * (UN * RS), seg[k] >> 8);
                    if (L.on) L.at[int64_t(v[k]) * L.stride] = MT(double(pre[k]) + L.sc * double(t[k]));
                }
        }
    }
}

// occupancy asked of the compiler: FP32 tiles fit in 96 VGPRs (five
// wavefronts per SIMD, as many as the LDS of five workgroups leaves), FP64
// tiles in 128 (four)
constexpr int TILE_F32_WAVES = 5;
constexpr int TILE_F64_WAVES = 4;

// RT = double: positions and normals in FP64 (xq, nq: m_qp, m_nrm; cen unused)
// RT = float : FP32 offsets from FP64 centroids (xq, nq: m_qf, m_nf; cen: m_cen)
// MT: storage of the operator (double, or float in mixed precision)
// TA x TB: target x source triangles of the tile, one pair per thread.  The
// tile of workgroup (x, y) is target block listA[y] x source block listB[x]
// (skip_lower: tiles whose source block precedes the target block return).
// The tile's V and K blocks are folded onto its vertices and added into the
// stored operator U (rows: [K' | V'] in the Morton vertex order, sK K and sV
// V) -- the launch's tiles touch disjoint entries, see BlockSide.
// SYM (square tiles): each unordered pair is evaluated once (the launches
// cover each unordered block pair once, in either orientation, and a
// diagonal tile only its pairs with the source after the target).  Besides
// V and K of (tau, sigma) a pair also yields K of (sigma, tau): the kernel
// values are shared, only the normal distance changes ((y_q - x).n_tau, the
// same for the six target points, which lie in the plane of tau).  It is
// added, transposed, to T (nv x nv: T[i][j] collects sK K(j, i)); V of
// (sigma, tau) is the transpose of V of (tau, sigma).  k_bem_symm then
// completes the operator: V' = U_V + U_V^T, K' = U_K + T^T.
//
// Every lane runs the quadrature: a pair that is not evaluated (padding
// triangle, shared vertex, or the mirror of a diagonal-tile pair) has its
// target moved 1e4 away and a zero factor, so its terms are exact zeros.
template <bool YUK, typename RT, typename MT, int TA, int TB, bool SYM, bool SLOT>
__global__ void __launch_bounds__(TA * TB) __attribute__((amdgpu_waves_per_eu(sizeof(RT) == 4 ? TILE_F32_WAVES : TILE_F64_WAVES)))
    k_bem_regular(int64_t nt, const int32_t *__restrict__ m_tri, const RT *__restrict__ xq,
                  const RT *__restrict__ nq, const double *__restrict__ cen, const double *__restrict__ m_area,
                  const int32_t *__restrict__ A_pref, const int32_t *__restrict__ A_nv,
                  const int32_t *__restrict__ A_seg, const int32_t *__restrict__ A_vid,
                  const int32_t *__restrict__ A_cpos,
                  const int32_t *__restrict__ B_pref, const int32_t *__restrict__ B_nv,
                  const int32_t *__restrict__ B_seg, const int32_t *__restrict__ B_vid,
                  const int32_t *__restrict__ B_cpos,
                  const int32_t *__restrict__ listA, const int32_t *__restrict__ listB, int skip_lower,
                  MT *__restrict__ U, MT *__restrict__ T, int64_t ld, int64_t nv, double sV, double sK,
                  double kappa, QRule6 R, QRule6F RF)
{
    static_assert(!SYM || TA == TB, "symmetric evaluation needs square tiles");
    static_assert(!SLOT || SYM, "slots hold the upper block pairs");
    // SLOT: U holds three ld x ld planes over the local vertices, K, V and the mirrored K (T)
    const int64_t offV = SLOT ? ld * ld : nv, ldT = SLOT ? ld : nv;
    constexpr bool F32 = sizeof(RT) == 4;
    constexpr int NT = TA * TB;
    const int64_t bA = listA[blockIdx.y], bB = listB[blockIdx.x];
    // evaluated as (bB, bA); SLOT: the lists are in the order of the colours,
    // and the block of the lower one is the target, as in the colour pairs' launches
    if (SYM && skip_lower && (SLOT ? blockIdx.x < blockIdx.y : bB < bA)) return;
    // quadrature inputs, then in the same memory the planes of the fold: FP32
    // all of them, FP64 V and K, then the mirrored K (four workgroups per CU)
    struct In {
        RT X[TA * 18], Y[TB * 18]; // quadrature points, 18 values per triangle
        RT N[TB][3], Na[SYM ? TA : 1][3];
        double Ca[F32 ? TA : 1][3], Cb[F32 ? TB : 1][3], Aa[TA], Ab[TB];
        int Va[TA][3], Vb[TB][3];
    };
    constexpr int NPL = F32 && SYM ? 3 : 2, NW = NT / 64;
    __shared__ union alignas(16) {
        In in;
        RT acc[NPL * fold_ps<TA, TB>()];
    } sh;
    RT *const sX = sh.in.X, *const sY = sh.in.Y;
    auto &sN = sh.in.N;
    auto &sNa = sh.in.Na;
    auto &sCa = sh.in.Ca;
    auto &sCb = sh.in.Cb;
    auto &sAa = sh.in.Aa;
    auto &sAb = sh.in.Ab;
    auto &sVa = sh.in.Va;
    auto &sVb = sh.in.Vb;
    __shared__ int sIb[TB * 3], sSb[TB * 3]; // operator index and segment of each source vertex

    const int tid = threadIdx.x;
    const int nA = A_nv[bA], nB = B_nv[bB];
    const int64_t pA = A_pref[bA], pB = B_pref[bB];

    // Every input is read at once, at an index within its array, and waited for
    // together; in loops and under conditions, each with a wait of its own,
    // the inputs took longer than the quadrature.
    {
        constexpr int NX = (TA * 18 + NT - 1) / NT, NY = (TB * 18 + NT - 1) / NT;
        const int64_t xa = 18 * bA * TA, xb = 18 * bB * TB, xe = 18 * nt; // a block's points are contiguous
        RT x[NX], y[NY];
#pragma unroll
        for (int k = 0; k < NX; ++k) x[k] = xq[min(xa + tid + k * NT, xe - 1)];
#pragma unroll
        for (int k = 0; k < NY; ++k) y[k] = xq[min(xb + tid + k * NT, xe - 1)];
        const int64_t ka = 3 * bA * TA + tid, kb = 3 * bB * TB + tid; // triangle * 3 + corner / component
        const int64_t la = min(ka, 3 * nt - 1), lb = min(kb, 3 * nt - 1);
        int va = m_tri[la], vb = m_tri[lb];
        RT nb = nq[lb], na = RT(0);
        if constexpr (SYM) na = nq[la];
        double ca = 0.0, cb = 0.0;
        if constexpr (F32) ca = cen[la], cb = cen[lb];
        double aa = m_area[min(bA * TA + tid, nt - 1)], ab = m_area[min(bB * TB + tid, nt - 1)];
        int ib = SLOT ? int(pB) + tid : B_vid[pB + min(tid, nB - 1)], sb = B_seg[pB + min(tid, nB - 1)];
        // (keeps the reads out of the conditions below)
        asm volatile("" : "+v"(va), "+v"(vb), "+v"(nb), "+v"(na), "+v"(aa), "+v"(ab), "+v"(ib), "+v"(sb), "+v"(ca), "+v"(cb));
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            asm volatile("" : "+v"(x[k]));
            if (tid + k * NT < TA * 18) sX[tid + k * NT] = xa + tid + k * NT < xe ? x[k] : RT(0);
        }
#pragma unroll
        for (int k = 0; k < NY; ++k) {
            asm volatile("" : "+v"(y[k]));
            if (tid + k * NT < TB * 18) sY[tid + k * NT] = xb + tid + k * NT < xe ? y[k] : RT(0);
        }
        const bool ina = ka < 3 * nt, inb = kb < 3 * nt;
        if (tid < TB * 3) {
            (&sN[0][0])[tid] = inb ? nb : RT(0);
            (&sVb[0][0])[tid] = inb ? vb : -1;
            if constexpr (F32) (&sCb[0][0])[tid] = inb ? cb : 0.0;
            sIb[tid] = ib;
            sSb[tid] = sb;
        }
        if (tid < TA * 3) {
            (&sVa[0][0])[tid] = ina ? va : -2;
            if constexpr (F32) (&sCa[0][0])[tid] = ina ? ca : 0.0;
            if constexpr (SYM) (&sNa[0][0])[tid] = ina ? na : RT(0);
        }
        if (tid < TA) sAa[tid] = bA * TA + tid < nt ? aa : 0.0;
        if (tid < TB) sAb[tid] = bB * TB + tid < nt ? ab : 0.0;
    }
    __syncthreads();

    // this thread's pair (target tl, source sl)
    const int tl = tid / TB, sl = tid % TB;
    // (FP32: every read at once; FP64: one after the other, for its registers)
    bool live = sVa[tl][0] >= 0 && sVb[sl][0] >= 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            if constexpr (F32) live &= sVa[tl][a] != sVb[sl][b];
            else live = live && sVa[tl][a] != sVb[sl][b];
        }
    if (SYM && bA == bB && sl <= tl) live = false; // the mirror pair carries it
    RT c0 = RT(0), c1 = RT(0), c2 = RT(0); // FP32: target frame relative to the source centroid
    if constexpr (F32) {
        c0 = float(sCa[tl][0] - sCb[sl][0]);
        c1 = float(sCa[tl][1] - sCb[sl][1]);
        c2 = float(sCa[tl][2] - sCb[sl][2]);
    }
    if (!live) c0 += RT(1.0e4);
    const RT sc = live ? RT(sAa[tl] * sAb[sl] * INV4PI) : RT(0);
    const RT *xt = sX + 18 * tl, *ys = sY + 18 * sl;
    const RT n0 = sN[sl][0], n1 = sN[sl][1], n2 = sN[sl][2];
    RT y0n = RT(0); // FP32: y_0.n (offsets from the source centroid are small)
    if constexpr (F32) y0n = ys[0] * n0 + ys[1] * n1 + ys[2] * n2;
    RT dm[SYM ? 6 : 1]; // (y_q - x).n_tau, the same for every target point x
    if constexpr (SYM) {
        const RT m0 = sNa[tl][0], m1 = sNa[tl][1], m2 = sNa[tl][2];
        const RT xa0 = xt[0] + c0, xa1 = xt[1] + c1, xa2 = xt[2] + c2;
#pragma unroll
        for (int q = 0; q < 6; ++q)
            dm[q] = (ys[3 * q] - xa0) * m0 + (ys[3 * q + 1] - xa1) * m1 + (ys[3 * q + 2] - xa2) * m2;
    }
    RT oA0, oA1, oD0, oD1;
    if constexpr (F32) {
        oA0 = RF.oA[0], oA1 = RF.oA[1], oD0 = RF.oD[0], oD1 = RF.oD[1];
    } else {
        oA0 = R.oA[0], oA1 = R.oA[1], oD0 = R.oD[0], oD1 = R.oD[1];
    }
    const RT kap = RT(kappa);
    const RT kl2 = RT(-1.44269504088896341 * kappa); // FP32: e^{-kappa r} = 2^{kl2 r}

    // Target point p: the kernels at its 6 source points and their sums with
    // the source rule's orbits.  The source points lie in the plane of the
    // source triangle, so the normal distance (x - y_q).n is the same for all
    // six: it is taken once per target point and factored out of the
    // double-layer sums.  s: single layer, t: double layer / (x - y).n, u:
    // mirrored double layer (SYM).
    auto point = [&](int p, RT (&s)[3], RT (&t)[3], RT (&u)[3], RT &dn) {
        const RT x0 = xt[3 * p] + c0;
        RT x1 = xt[3 * p + 1], x2 = xt[3 * p + 2];
        if constexpr (F32) {
            x1 += c1;
            x2 += c2;
            dn = x0 * n0 + x1 * n1 + x2 * n2 - y0n;
        } else {
            dn = (x0 - ys[0]) * n0 + (x1 - ys[1]) * n1 + (x2 - ys[2]) * n2;
        }
        RT gv[6], hk[6]; // single-layer kernel, double-layer kernel / (x - y).n
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const RT d0 = x0 - ys[3 * q], d1 = x1 - ys[3 * q + 1], d2 = x2 - ys[3 * q + 2];
            const RT r2 = d0 * d0 + d1 * d1 + d2 * d2;
            const RT ri = rsqrt_pos(r2);
            if constexpr (YUK) {
                const RT r = r2 * ri;
                RT e;
                if constexpr (F32) e = __builtin_amdgcn_exp2f(kl2 * r);
                else e = exp_neg(kap * r);
                gv[q] = e * ri;
                hk[q] = gv[q] * ri * (ri + kap); // e (1 + kappa r) / r^3
            } else {
                gv[q] = ri;
                hk[q] = ri * ri * ri;
            }
        }
        auto orb = [&](const RT (&g)[6], RT (&o)[3]) {
            const RT c = oA0 * (g[0] + g[1] + g[2]) + oA1 * (g[3] + g[4] + g[5]);
            o[0] = c + oD0 * g[0] + oD1 * g[3];
            o[1] = c + oD0 * g[1] + oD1 * g[4];
            o[2] = c + oD0 * g[2] + oD1 * g[5];
        };
        orb(gv, s);
        orb(hk, t);
        if constexpr (SYM) {
            RT hm[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) hm[q] = hk[q] * dm[q];
            orb(hm, u);
        }
    };

    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // SLOT: rows are the block's own local vertices
    FoldOut<MT> out{U, T, offV, ld, ldT, sV, sK};
    if constexpr (SLOT) {
        out.U += pA * ld;
        out.T += pA * ldT;
    }
    MT pre[fold_rnd<MT>()];
    if constexpr (F32)
        fold_read<SLOT, NW>(w, nA, A_vid + pA, fold_lane<TA, TB, 0, NPL, RT>(lane, nB, sIb, sSb, out), pre);

    // the pair's 3x3 blocks, summed over its 36 quadrature pairs; the first
    // target point assigns them
    RT Vl[9] = {}, Kl[9] = {}, Ktl[SYM ? 9 : 1] = {};
    auto accumulate = [&](auto first, int p) {
        // the source points are read from LDS at every target point rather
        // than held in registers (a compiler-only fence): fewer registers,
        // more wavefronts per SIMD
        asm volatile("" ::: "memory");
        RT s[3], t[3], u[3], dn;
        point(p, s, t, u, dn);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            RT wa;
            if constexpr (F32) wa = sc * RF.wb[p][a];
            else wa = sc * R.wb[p][a];
            const RT wk = wa * dn;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                Vl[3 * a + b] = decltype(first)::value ? wa * s[b] : fma(wa, s[b], Vl[3 * a + b]);
                Kl[3 * a + b] = decltype(first)::value ? wk * t[b] : fma(wk, t[b], Kl[3 * a + b]);
                if constexpr (SYM)
                    Ktl[3 * a + b] = decltype(first)::value ? wa * u[b] : fma(wa, u[b], Ktl[3 * a + b]);
            }
        }
    };
    accumulate(std::true_type{}, 0);
    // not unrolled: the 6 source points of one target point are the unit of ILP
#pragma unroll 1
    for (int p = 1; p < 6; ++p) accumulate(std::false_type{}, p);

    RT vk[NPL][9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        vk[0][k] = Vl[k];
        vk[1][k] = Kl[k];
        if constexpr (NPL == 3) vk[NPL - 1][k] = Ktl[k];
    }
    const int pa = A_cpos[bA * TA + tl], pb = B_cpos[bB * TB + sl];
    const int32_t *segA = A_seg + pA, *vA = A_vid + pA, *segB = B_seg + pB;
    __syncthreads();
    if constexpr (!F32) fold_read<SLOT, NW>(w, nA, vA, fold_lane<TA, TB, 0, NPL, RT>(lane, nB, sIb, sSb, out), pre);
    fold_tile<SLOT, TA, TB, 0, NPL>(tid, nA, nB, segA, vA, segB, sIb, sSb, pa, pb, sh.acc, vk, out, pre);
    if constexpr (SYM && !F32) {
        RT kt[1][9];
#pragma unroll
        for (int k = 0; k < 9; ++k) kt[0][k] = Ktl[k];
        fold_read<SLOT, NW>(w, nA, vA, fold_lane<TA, TB, 2, 1, RT>(lane, nB, sIb, sSb, out), pre);
        __syncthreads();
        fold_tile<SLOT, TA, TB, 2, 1>(tid, nA, nB, segA, vA, segB, sIb, sSb, pa, pb, sh.acc, kt, out, pre);
    }
}

// ---------------------------------------------------------------------------
// 2. completion of a symmetric evaluation
// ---------------------------------------------------------------------------
// On 32 x 32 tiles (I <= J, both mirror tiles handled by one workgroup):
// V'(i, j) = U_V(i, j) + U_V(j, i) and K'(i, j) = U_K(i, j) + T(j, i), where
// B holds [U_K | U_V] per row (signed; the regular part of V' comes out
// bitwise symmetric).
constexpr int SYMT = 32;
template <typename MT>
__global__ void __launch_bounds__(256) k_bem_symm(int64_t nv, int64_t ld, MT *__restrict__ B, const MT *__restrict__ T)
{
    const int64_t I = blockIdx.y, J = blockIdx.x;
    if (J < I) return;
    __shared__ double a[SYMT][SYMT + 1], b[SYMT][SYMT + 1], t1[SYMT][SYMT + 1], t2[SYMT][SYMT + 1];
    const int tx = threadIdx.x % SYMT, ty = threadIdx.x / SYMT;
    for (int r = ty; r < SYMT; r += 256 / SYMT) {
        const int64_t i = I * SYMT + r, j = J * SYMT + tx;   // tile (I, J)
        const int64_t i2 = J * SYMT + r, j2 = I * SYMT + tx; // tile (J, I)
        const bool in1 = i < nv && j < nv, in2 = i2 < nv && j2 < nv;
        a[r][tx] = in1 ? double(B[i * ld + nv + j]) : 0.0;
        t2[r][tx] = in1 ? double(T[i * nv + j]) : 0.0;
        b[r][tx] = in2 ? double(B[i2 * ld + nv + j2]) : 0.0;
        t1[r][tx] = in2 ? double(T[i2 * nv + j2]) : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < SYMT; r += 256 / SYMT) {
        const int64_t i = I * SYMT + r, j = J * SYMT + tx;
        if (i < nv && j < nv) {
            B[i * ld + nv + j] = MT(a[r][tx] + b[tx][r]);
            add_entry(B, i * ld + j, t1[tx][r]);
        }
        const int64_t i2 = J * SYMT + r, j2 = I * SYMT + tx;
        if (I != J && i2 < nv && j2 < nv) {
            B[i2 * ld + nv + j2] = MT(b[r][tx] + a[tx][r]);
            add_entry(B, i2 * ld + j2, t2[tx][r]);
        }
    }
}

// The same completion for an even nv (every row offset of B and T is then
// even, so each thread moves aligned pairs of entries), launched over the
// tile pairs I <= J only (block k = J (J + 1) / 2 + I), with the stored K'
// entries read together with the other inputs, before the exchange.  The
// sums are those of k_bem_symm, so the results are identical.
template <typename MT>
__global__ void __launch_bounds__(256) k_bem_symm2(int64_t nv, int64_t ld, MT *__restrict__ B,
                                                   const MT *__restrict__ T)
{
    typedef MT pair_t __attribute__((ext_vector_type(2)));
    const int64_t k = blockIdx.x;
    int64_t J = int64_t((sqrt(8.0 * double(k) + 1.0) - 1.0) * 0.5);
    while (J * (J + 1) / 2 > k) --J;
    while ((J + 1) * (J + 2) / 2 <= k) ++J;
    const int64_t I = k - J * (J + 1) / 2;
    __shared__ double a[SYMT][SYMT + 1], b[SYMT][SYMT + 1], t1[SYMT][SYMT + 1], t2[SYMT][SYMT + 1];
    constexpr int TXN = SYMT / 2, RP = 256 / TXN; // threads per tile row, rows per pass
    const int tx = threadIdx.x % TXN, ty = threadIdx.x / TXN, c = 2 * tx;
    pair_t k1[SYMT / RP], k2[SYMT / RP]; // stored K' of tile (I, J) and of tile (J, I)
#pragma unroll
    for (int h = 0; h < SYMT / RP; ++h) {
        const int r = ty + h * RP;
        const int64_t i = I * SYMT + r, j = J * SYMT + c;   // tile (I, J)
        const int64_t i2 = J * SYMT + r, j2 = I * SYMT + c; // tile (J, I)
        // nv even and c even: the pair (j, j + 1) lies entirely inside or outside
        const bool in1 = i < nv && j < nv, in2 = i2 < nv && j2 < nv;
        const pair_t z = {MT(0), MT(0)};
        const pair_t va = in1 ? *reinterpret_cast<const pair_t *>(B + i * ld + nv + j) : z;
        const pair_t vt2 = in1 ? *reinterpret_cast<const pair_t *>(T + i * nv + j) : z;
        const pair_t vb = in2 ? *reinterpret_cast<const pair_t *>(B + i2 * ld + nv + j2) : z;
        const pair_t vt1 = in2 ? *reinterpret_cast<const pair_t *>(T + i2 * nv + j2) : z;
        k1[h] = in1 ? *reinterpret_cast<const pair_t *>(B + i * ld + j) : z;
        k2[h] = in2 && I != J ? *reinterpret_cast<const pair_t *>(B + i2 * ld + j2) : z;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            a[r][c + e] = double(va[e]);
            t2[r][c + e] = double(vt2[e]);
            b[r][c + e] = double(vb[e]);
            t1[r][c + e] = double(vt1[e]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < SYMT / RP; ++h) {
        const int r = ty + h * RP;
        const int64_t i = I * SYMT + r, j = J * SYMT + c;
        if (i < nv && j < nv) {
            pair_t v, w;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                v[e] = MT(a[r][c + e] + b[c + e][r]);
                w[e] = MT(double(k1[h][e]) + t1[c + e][r]);
            }
            *reinterpret_cast<pair_t *>(B + i * ld + nv + j) = v;
            *reinterpret_cast<pair_t *>(B + i * ld + j) = w;
        }
        const int64_t i2 = J * SYMT + r, j2 = I * SYMT + c;
        if (I != J && i2 < nv && j2 < nv) {
            pair_t v, w;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                v[e] = MT(b[r][c + e] + a[c + e][r]);
                w[e] = MT(double(k2[h][e]) + t2[c + e][r]);
            }
            *reinterpret_cast<pair_t *>(B + i2 * ld + nv + j2) = v;
            *reinterpret_cast<pair_t *>(B + i2 * ld + j2) = w;
        }
    }
}

// Small surfaces (launch_slots): one launch holds every tile, each storing its
// folded values to its own entries of three S x S planes over the blocks'
// local vertices (K, V, mirrored K; block pairs A <= B in the order of the
// colours only), and this adds them up for the completion above: U(k, l) and
// T(k, l) take, over the local vertices a of k and b of l with block(a) <=
// block(b), what the tile left at (a, b).  A vertex's blocks are all of
// different colours, so walking them in that order adds the tiles as the colour
// pairs' launches do, rounded to the storage after each: the two ways give the
// same bits, and which one is taken may depend on the memory there is.  Three
// launches instead of one per colour pair (28 to 36, 12-15 us each however few
// tiles they hold), the completion and the clears: a 642-vertex surface 0.50 ->
// 0.105 ms (FP64), 0.40 -> 0.067 (FP32); a 320-triangle solve 5.9 -> 5.0 ms,
// 1 280 triangles mixed 14.5 -> 13.7.
//
// Bound by the latency of the plane reads and of the lists before them.  A
// workgroup takes 256 columns of one row, so that its reads are rows of the
// planes, whose lines the lanes share (1 212 vertices FP64 67 us and 15 of
// completion, 1 692 FP32 82 and 17); a thread that adds up both entries of a
// pair and completes them itself reads every second block by columns (137 and
// 216 us).
template <typename MT>
__global__ void __launch_bounds__(256)
    k_bem_gather(int64_t nv, int64_t ld, int64_t S, const int32_t *__restrict__ occ_ptr,
                 const int32_t *__restrict__ occ, const MT *__restrict__ W, MT *__restrict__ U, MT *__restrict__ T)
{
    struct Occ { // a local vertex and the place of its block in the order of the colours
        int32_t at, rank;
    };
    const Occ *O = reinterpret_cast<const Occ *>(occ);
    const int64_t k = blockIdx.y, l = blockIdx.x * int64_t(256) + threadIdx.x;
    if (blockIdx.x == 0) // the row padding, read by the dense apply against zero inputs
        for (int64_t c = 2 * nv + threadIdx.x; c < ld; c += 256) U[k * ld + c] = MT(0);
    if (l >= nv) return;
    const int32_t j0 = occ_ptr[l], j1 = occ_ptr[l + 1];
    MT u[3] = {}; // K, V, mirrored K
    constexpr int N = 4; // local vertices of l read at a time
    for (int32_t i = occ_ptr[k]; i < occ_ptr[k + 1]; ++i) {
        const Occ a = O[i];
        const MT *row = W + a.at * S;
        for (int32_t j = j0; j < j1; j += N) {
            bool take[N];
            MT d[N][3];
#pragma unroll
            for (int t = 0; t < N; ++t) { // unconditional reads; past the end the last again
                const Occ b = O[min(j + t, j1 - 1)];
                take[t] = j + t < j1 && a.rank <= b.rank;
#pragma unroll
                for (int q = 0; q < 3; ++q) d[t][q] = row[q * S * S + b.at];
            }
#pragma unroll
            for (int t = 0; t < N; ++t)
#pragma unroll
                for (int q = 0; q < 3; ++q) u[q] = take[t] ? MT(double(u[q]) + double(d[t][q])) : u[q];
        }
    }
    U[k * ld + l] = u[0];
    U[k * ld + nv + l] = u[1];
    T[k * nv + l] = u[2];
}

// ---------------------------------------------------------------------------
// 3. touching pairs: Sauter-Schwab (Sauter & Schwab, Boundary Element
//    Methods, Sec. 5.2) on the reference triangle {0 <= xi2 <= xi1 <= 1},
//    chi(xi) = P0 + xi1 (P1 - P0) + xi2 (P2 - P1), shape functions
//    (1 - xi1, xi1 - xi2, xi2); vertices reordered so that the shared
//    vertex is P0 (common vertex) or the shared edge is P0 P1 (common edge).
// ---------------------------------------------------------------------------
struct RefPair {
    double x1, x2, y1, y2;
};

// the r-th region map for `kind` shared vertices; the Jacobian is ss_jac
static RefPair ss_region(int kind, int r, double xi, double e1, double e2, double e3)
{
    if (kind == 3) {
        switch (r) {
        case 0: return {xi, xi * (1 - e1 + e1 * e2), xi * (1 - e1 * e2 * e3), xi * (1 - e1)};
        case 1: return {xi * (1 - e1 * e2 * e3), xi * (1 - e1), xi, xi * (1 - e1 + e1 * e2)};
        case 2: return {xi, xi * e1 * (1 - e2 + e2 * e3), xi * (1 - e1 * e2), xi * e1 * (1 - e2)};
        case 3: return {xi * (1 - e1 * e2), xi * e1 * (1 - e2), xi, xi * e1 * (1 - e2 + e2 * e3)};
        case 4: return {xi * (1 - e1 * e2 * e3), xi * e1 * (1 - e2 * e3), xi, xi * e1 * (1 - e2)};
        default: return {xi, xi * e1 * (1 - e2), xi * (1 - e1 * e2 * e3), xi * e1 * (1 - e2 * e3)};
        }
    }
    if (kind == 2) {
        switch (r) {
        case 0: return {xi, xi * e1 * e3, xi * (1 - e1 * e2), xi * e1 * (1 - e2)};
        case 1: return {xi, xi * e1, xi * (1 - e1 * e2 * e3), xi * e1 * e2 * (1 - e3)};
        case 2: return {xi * (1 - e1 * e2), xi * e1 * (1 - e2), xi, xi * e1 * e2 * e3};
        case 3: return {xi * (1 - e1 * e2 * e3), xi * e1 * e2 * (1 - e3), xi, xi * e1};
        default: return {xi * (1 - e1 * e2 * e3), xi * e1 * (1 - e2 * e3), xi, xi * e1 * e2};
        }
    }
    if (r == 0) return {xi, xi * e1, xi * e2, xi * e2 * e3};
    return {xi * e2, xi * e2 * e3, xi, xi * e1};
}

static double ss_jac(int kind, int r, double xi, double e1, double e2)
{
    const double x3 = xi * xi * xi;
    if (kind == 3) return x3 * e1 * e1 * e2;
    if (kind == 2) return r == 0 ? x3 * e1 * e1 : x3 * e1 * e1 * e2;
    return x3 * e2;
}

// The points of the three rules, kind 3, 2, 1 after each other, SS_STRIDE
// doubles each: x1, x2, y1, y2, then the nine weights w phi_a(x) phi_b(y)
constexpr int SS_STRIDE = 16; // 13 used; one aligned 128-byte line
constexpr int SS_NPT[3] = {6 * 256, 5 * 256, 2 * 256}, SS_OFF[3] = {0, 6 * 256, 11 * 256}, SS_ALL = 13 * 256;

// device copy of the table, once per context, uploaded on the stream of the
// setup that comes first; other streams may use it when this returns
static const double *ss_points(Ctx &C, hipStream_t s)
{
    std::lock_guard<std::mutex> lk(C.setup_mu);
    if (C.ss_points) return C.ss_points;
    const Rules &R = rules();
    std::vector<double> t(size_t(SS_ALL) * SS_STRIDE, 0.0);
    for (int g = 0; g < 3; ++g)
        for (int i = 0; i < SS_NPT[g]; ++i) {
            const int kind = 3 - g, r = i >> 8, i0 = (i >> 6) & 3, i1 = (i >> 4) & 3, i2 = (i >> 2) & 3, i3 = i & 3;
            const double xi = R.gl_x[i0], e1 = R.gl_x[i1], e2 = R.gl_x[i2], e3 = R.gl_x[i3];
            const RefPair m = ss_region(kind, r, xi, e1, e2, e3);
            const double w = R.gl_w[i0] * R.gl_w[i1] * R.gl_w[i2] * R.gl_w[i3] * ss_jac(kind, r, xi, e1, e2);
            const double fx[3] = {1.0 - m.x1, m.x1 - m.x2, m.x2}, fy[3] = {1.0 - m.y1, m.y1 - m.y2, m.y2};
            double *o = t.data() + size_t(SS_OFF[g] + i) * SS_STRIDE;
            o[0] = m.x1;
            o[1] = m.x2;
            o[2] = m.y1;
            o[3] = m.y2;
            for (int k = 0; k < 9; ++k) o[4 + k] = w * fx[k / 3] * fy[k % 3];
        }
    double *dev = nullptr;
    PB_HIP(hipMalloc(&dev, sizeof(double) * t.size()));
    hipError_t e = hipMemcpyAsync(dev, t.data(), sizeof(double) * t.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(dev);
        PB_HIP(e);
    }
    C.ss_points = dev;
    return dev;
}

// One lane per touching ordered pair (tau, sigma), 64 pairs of one kind per
// workgroup (ord: the pairs by kind, cnt of each); its SING_W wavefronts split
// the rule's points, which are uniform and come through scalar loads, and
// their sums are added in wavefront order.  The 3x3 V and K blocks (in the
// triangles' own vertex order) go to out[18 * pair].  Both panels start at a
// shared vertex, so x - y is formed from edge vectors alone, and its normal
// distance from x's edges (y and the shared vertex lie in sigma's plane).
//
// Bound by FP64 vector issue: about 47 instruction slots per point (Yukawa
// 71), 9 984 points per triangle.  One wavefront per pair, which formed the
// region maps, shape products and 18 cross-lane sums for every pair, took
// 1.53 ms at 20 480 triangles and 0.40 at 5 120 (mean of Laplace and Yukawa);
// this 0.47 and 0.13.
constexpr int SING_W = 8;
template <bool YUK>
__global__ void __launch_bounds__(64 * SING_W)
    k_bem_singular(int64_t n3, int64_t n2, int64_t n1, const int32_t *__restrict__ ord,
                   const int32_t *__restrict__ tp_tau, const int32_t *__restrict__ tp_sig,
                   const int32_t *__restrict__ tri, const double *__restrict__ vx, const double *__restrict__ nrm,
                   const double *__restrict__ area, double kappa, const double *__restrict__ points,
                   double *__restrict__ out)
{
    constexpr int RND = 6; // sums exchanged at a time
    __shared__ double red[SING_W][RND][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t g3 = (n3 + 63) / 64, g2 = (n2 + 63) / 64;
    int64_t bi = blockIdx.x, seg = 0, n = n3;
    int g = 0; // kind 3 - g
    if (bi >= g3) {
        bi -= g3;
        seg = n3;
        n = n2;
        g = 1;
        if (bi >= g2) {
            bi -= g2;
            seg = n3 + n2;
            n = n1;
            g = 2;
        }
    }
    const int64_t i = bi * 64 + lane;
    const bool in = i < n;
    const int64_t pair = ord[seg + (in ? i : n - 1)];
    const int32_t ta = tp_tau[pair], sb = tp_sig[pair];
    int A[3], B[3];
    for (int k = 0; k < 3; ++k) {
        A[k] = tri[3 * ta + k];
        B[k] = tri[3 * sb + k];
    }
    int shared = 0, ia0 = 0, ia1 = 0, ib0 = 0, ib1 = 0; // the first two shared corners
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            if (A[a] == B[b]) {
                if (shared == 0) {
                    ia0 = a;
                    ib0 = b;
                } else if (shared == 1) {
                    ia1 = a;
                    ib1 = b;
                }
                ++shared;
            }
    int pa[3], pb[3];
    if (g == 0) { // identical
        pa[0] = pb[0] = 0;
        pa[1] = pb[1] = 1;
        pa[2] = pb[2] = 2;
    } else if (g == 1) { // common edge: first
        pa[0] = ia0;
        pa[1] = ia1;
        pa[2] = 3 - ia0 - ia1;
        pb[0] = ib0;
        pb[1] = ib1;
        pb[2] = 3 - ib0 - ib1;
    } else { // common vertex first
        pa[0] = ia0;
        pa[1] = (ia0 + 1) % 3;
        pa[2] = (ia0 + 2) % 3;
        pb[0] = ib0;
        pb[1] = (ib0 + 1) % 3;
        pb[2] = (ib0 + 2) % 3;
    }
    auto corner = [](const int(&T)[3], int k) { return k == 0 ? T[0] : k == 1 ? T[1] : T[2]; };
    double E1[3], E2[3], F1[3], F2[3], a1 = 0.0, a2 = 0.0;
    for (int d = 0; d < 3; ++d) {
        const double p0 = vx[3 * corner(A, pa[0]) + d], p1 = vx[3 * corner(A, pa[1]) + d],
                     p2 = vx[3 * corner(A, pa[2]) + d];
        const double q0 = vx[3 * corner(B, pb[0]) + d], q1 = vx[3 * corner(B, pb[1]) + d],
                     q2 = vx[3 * corner(B, pb[2]) + d], ny = nrm[3 * sb + d];
        E1[d] = p1 - p0;
        E2[d] = p2 - p1;
        F1[d] = q1 - q0;
        F2[d] = q2 - q1;
        a1 = fma(E1[d], ny, a1);
        a2 = fma(E2[d], ny, a2);
    }
    double V[9], K[9];
    for (int k = 0; k < 9; ++k) V[k] = K[k] = 0.0;
    const int npt = (g == 0 ? SS_NPT[0] : g == 1 ? SS_NPT[1] : SS_NPT[2]) / SING_W;
    const double *T = points + int64_t((g == 0 ? SS_OFF[0] : g == 1 ? SS_OFF[1] : SS_OFF[2]) + w * npt) * SS_STRIDE;
#pragma unroll 4 // several points' scalar loads in flight
    for (int k = 0; k < npt; ++k, T += SS_STRIDE) {
        const double x1 = T[0], x2 = T[1], y1 = T[2], y2 = T[3];
        double r2 = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double dd = fma(x1, E1[d], x2 * E2[d]) - fma(y1, F1[d], y2 * F2[d]);
            r2 = fma(dd, dd, r2);
        }
        const double ri = rsqrt_pos(r2);
        double gv = ri, gk = ri * ri * ri;
        if constexpr (YUK) {
            gv = exp_neg(kappa * (r2 * ri)) * ri;
            gk = gv * ri * (ri + kappa); // e (1 + kappa r) / r^3
        }
#pragma unroll
        for (int c = 0; c < 9; ++c) V[c] = fma(T[4 + c], gv, V[c]);
        if (g == 0) continue; // (x - y).n_y vanishes on a flat panel
        gk *= fma(x1, a1, x2 * a2);
#pragma unroll
        for (int c = 0; c < 9; ++c) K[c] = fma(T[4 + c], gk, K[c]);
    }
    const double sc = 4.0 * area[ta] * area[sb] * INV4PI;
#pragma unroll
    for (int r0 = 0; r0 < 18; r0 += RND) {
#pragma unroll
        for (int k = 0; k < RND; ++k) red[w][k][lane] = r0 + k < 9 ? V[(r0 + k) % 9] : K[(r0 + k) % 9];
        __syncthreads();
        if (w < RND) {
            double s = 0.0;
#pragma unroll
            for (int v = 0; v < SING_W; ++v) s += red[v][w][lane];
            const int c = (r0 + w) % 9, a = c / 3, b = c % 3;
            if (in) out[18 * pair + (r0 + w < 9 ? 0 : 9) + 3 * corner(pa, a) + corner(pb, b)] = sc * s;
        }
        __syncthreads();
    }
}

// Row-owned scatter of the touching-pair blocks and of the 1/2 M term into
// the stored operator (Morton vertex order: vertex i is row minv[i]).  One
// wavefront per row: what the pairs at the vertex contribute (about 240
// values of V' and K') is staged in LDS with its column; the wavefront then
// walks the contributions in order, a lane per distinct column adding its own,
// and adds each column's sum to the stored entry once.  (One thread per row
// that added every contribution into global memory took 140-330 us whatever
// the surface's size.)
constexpr int SCAT_CAP = 640; // staged at once: more than the pairs of any one triangle give
template <typename MT>
__global__ void __launch_bounds__(64)
    k_bem_scatter(int64_t nv, int64_t ld, const int32_t *__restrict__ minv, const int32_t *__restrict__ v2t_ptr,
                  const int32_t *__restrict__ v2t, const int32_t *__restrict__ tri,
                  const int32_t *__restrict__ tp_ptr, const int32_t *__restrict__ tp_sig,
                  const double *__restrict__ tpv, const double *__restrict__ area, double sV, double sK,
                  MT *__restrict__ Bo)
{
    __shared__ int cj[SCAT_CAP];
    __shared__ double cv[SCAT_CAP], ck[SCAT_CAP];
    const int lane = threadIdx.x;
    const int64_t i = blockIdx.x;
    MT *row = Bo + int64_t(minv[i]) * ld;
    int m = 0; // staged
    auto flush = [&]() {
        __syncthreads();
        int col = -1, nu = 0; // this lane's column, columns in use
        double v = 0.0, k = 0.0;
        auto store = [&]() {
            if (lane < nu) {
                add_entry(row, nv + col, v);
                add_entry(row, int64_t(col), k);
            }
            col = -1;
            nu = 0;
            v = k = 0.0;
            __threadfence_block(); // a column may come back to another lane
            __syncthreads();
        };
        for (int c0 = 0; c0 < m; c0 += 64) {
            const int cn = min(m - c0, 64);
            const int jj = lane < cn ? cj[c0 + lane] : -1;
            for (int e = 0; e < cn; ++e) {
                const int j = __builtin_amdgcn_readlane(jj, e);
                if (__ballot(col == j) == 0) { // a new column
                    if (nu == 64) store();
                    if (lane == nu) col = j;
                    ++nu;
                }
                const double ev = cv[c0 + e], ek = ck[c0 + e]; // one address: broadcast
                if (col == j) {
                    v += ev;
                    k += ek;
                }
            }
        }
        store();
        m = 0;
    };
    for (int32_t e = v2t_ptr[i]; e < v2t_ptr[i + 1]; ++e) {
        const int32_t ta = v2t[e] / 3, a = v2t[e] % 3, p0 = tp_ptr[ta];
        const int np = tp_ptr[ta + 1] - p0;
        for (int c0 = 0; c0 < 3 * np + 3; c0 += SCAT_CAP) { // one round, except at extreme valences
            const int cn = min(3 * np + 3 - c0, SCAT_CAP);
            if (m + cn > SCAT_CAP) flush();
            for (int c = lane; c < cn; c += 64) {
                const int q = c0 + c, b = q % 3;
                int j;
                double v = 0.0, k;
                if (q < 3 * np) {
                    const int64_t pp = p0 + q / 3;
                    j = tri[3 * tp_sig[pp] + b];
                    v = sV * tpv[18 * pp + 3 * a + b];
                    k = sK * tpv[18 * pp + 9 + 3 * a + b];
                } else {
                    j = tri[3 * ta + b];
                    k = 0.5 * area[ta] * (a == b ? 2.0 : 1.0) / 12.0;
                }
                cj[m + c] = minv[j];
                cv[m + c] = v;
                ck[m + c] = k;
            }
            m += cn;
        }
    }
    flush();
}

__global__ void k_gather_coords(int64_t nv, const int32_t *__restrict__ g, const double *__restrict__ x,
                                double *__restrict__ vx)
{
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i >= nv) return;
    for (int d = 0; d < 3; ++d) vx[3 * i + d] = x[3 * g[i] + d];
}

// diagonal of V' in the ascending vertex order
template <typename MT>
__global__ void k_vdiag(int64_t nv, int64_t ld, const int32_t *__restrict__ mvert, const MT *__restrict__ B,
                        double *__restrict__ vdiag)
{
    const int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (k < nv) vdiag[mvert[k]] = double(B[k * ld + nv + k]);
}

// ---------------------------------------------------------------------------
// sparse approximate inverse of the single-layer block (GMRES preconditioner)
// ---------------------------------------------------------------------------
constexpr int SPAI_SMALL = 8; // largest 1-ring of the one-wavefront path
// Row i minimises || m^T V' - e_i^T ||_2 over m supported on the 1-ring P(i)
// of vertex i, V' = columns [nv, 2nv) of the stored rows (the signed
// single-layer block of the operator; vertex v is row / column minv[v]).  Normal equations
// (V'_P V'_P^T) m = V'_P e_i, solved by Cholesky.  One workgroup per row;
// the Gram matrix accumulates over 64-column tiles of the rows P staged in
// LDS, one thread per (a, b) pair, in a fixed order.
template <typename MT>
__global__ void __launch_bounds__(256)
    k_spai(int64_t nv, const MT *__restrict__ B, int64_t ld, const int32_t *__restrict__ minv,
           const int32_t *__restrict__ ring_ptr, const int32_t *__restrict__ ring, double *__restrict__ val,
           int *__restrict__ bad)
{
    __shared__ double T[MAXRING][65];
    __shared__ double G[MAXRING][MAXRING + 1];
    __shared__ double rhs[MAXRING];
    __shared__ int P[MAXRING];
    const int tid = threadIdx.x;
    const int64_t i = blockIdx.x;
    const int p0 = ring_ptr[i], m = ring_ptr[i + 1] - p0;
    if (m <= SPAI_SMALL) return; // handled by k_spai_small
    for (int a = tid; a < m; a += 256) P[a] = minv[ring[p0 + a]];
    __syncthreads();
    const int npair = m * (m + 1) / 2;
    constexpr int PPT = (MAXRING * (MAXRING + 1) / 2 + 255) / 256; // pairs per thread
    double acc[PPT];
    int pa[PPT], pb[PPT];
#pragma unroll
    for (int q = 0; q < PPT; ++q) {
        acc[q] = 0.0;
        const int pr = tid + 256 * q;
        int a = int((sqrt(8.0 * pr + 1.0) - 1.0) * 0.5);
        while (a * (a + 1) / 2 > pr) --a;
        while ((a + 1) * (a + 2) / 2 <= pr) ++a;
        pa[q] = a;
        pb[q] = pr - a * (a + 1) / 2;
    }
    for (int64_t c0 = 0; c0 < nv; c0 += 64) {
        for (int k = tid; k < m * 64; k += 256) {
            const int a = k >> 6, c = k & 63;
            T[a][c] = c0 + c < nv ? double(B[int64_t(P[a]) * ld + nv + c0 + c]) : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            if (tid + 256 * q < npair) {
                const int a = pa[q], b = pb[q];
                double s = 0.0;
                for (int c = 0; c < 64; ++c) s = fma(T[a][c], T[b][c], s);
                acc[q] += s;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < PPT; ++q)
        if (tid + 256 * q < npair) G[pa[q]][pb[q]] = G[pb[q]][pa[q]] = acc[q];
    for (int a = tid; a < m; a += 256) rhs[a] = double(B[int64_t(P[a]) * ld + nv + minv[i]]);
    __syncthreads();
    if (tid == 0) {
        // Cholesky G = L L^T (lower triangle), then L y = rhs, L^T m = y
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
                double s = G[b][a];
                for (int k = 0; k < a; ++k) s -= G[b][k] * G[a][k];
                G[b][a] = s / G[a][a];
            }
        }
        if (!ok) {
            atomicOr(bad, 4);
            for (int a = 0; a < m; ++a) val[p0 + a] = 0.0;
        } else {
            for (int a = 0; a < m; ++a) {
                double s = rhs[a];
                for (int k = 0; k < a; ++k) s -= G[a][k] * rhs[k];
                rhs[a] = s / G[a][a];
            }
            for (int a = m - 1; a >= 0; --a) {
                double s = rhs[a];
                for (int k = a + 1; k < m; ++k) s -= G[k][a] * rhs[k];
                rhs[a] = s / G[a][a];
            }
            for (int a = 0; a < m; ++a) val[p0 + a] = rhs[a];
        }
    }
}

// Rows whose 1-ring has at most SPAI_SMALL vertices (every vertex of the
// usual surface meshes): one wavefront per row, each lane streams W
// consecutive columns at a time (one 16-byte load per row: W = 4 for FP32,
// 2 for FP64) of the m rows and keeps the m (m + 1) / 2 Gram partial sums in
// registers; a fixed xor-shuffle tree then sums them across the lanes.  The
// V' columns start at column nv of rows of ld (a multiple of 256) entries,
// so the first head = (-nv) mod W columns are taken one per lane and the
// W-wide loads start at an aligned column.
template <typename MT, int W> struct alignas(W * sizeof(MT)) SpaiVec {
    MT v[W];
};
template <typename MT, int W>
__global__ void __launch_bounds__(256)
    k_spai_small(int64_t nv, const MT *__restrict__ B, int64_t ld, const int32_t *__restrict__ minv,
                 const int32_t *__restrict__ ring_ptr, const int32_t *__restrict__ ring, double *__restrict__ val,
                 int *__restrict__ bad)
{
    constexpr int NP = SPAI_SMALL * (SPAI_SMALL + 1) / 2;
    const int lane = threadIdx.x & 63;
    const int64_t i = blockIdx.x * int64_t(4) + (threadIdx.x >> 6);
    if (i >= nv) return;
    const int p0 = ring_ptr[i], m = ring_ptr[i + 1] - p0;
    if (m > SPAI_SMALL) return; // handled by k_spai
    const MT *rows[SPAI_SMALL];
#pragma unroll
    for (int a = 0; a < SPAI_SMALL; ++a) rows[a] = B + int64_t(minv[ring[p0 + (a < m ? a : 0)]]) * ld + nv;
    double g[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) g[k] = 0.0;
    const int head = int((W - nv % W) % W);
    if (lane < head) {
        double x[SPAI_SMALL];
#pragma unroll
        for (int a = 0; a < SPAI_SMALL; ++a) x[a] = a < m ? double(rows[a][lane]) : 0.0;
        int k = 0;
#pragma unroll
        for (int a = 0; a < SPAI_SMALL; ++a)
#pragma unroll
            for (int b = 0; b <= a; ++b, ++k) g[k] = fma(x[a], x[b], g[k]);
    }
    for (int64_t c = head + int64_t(W) * lane; c < nv; c += 64 * W) {
        if constexpr (sizeof(MT) == 4) {
            // FP32 storage: the loaded values stay FP32 and each column is
            // widened when its products are formed (162 instead of 181 VGPRs,
            // three wavefronts per SIMD instead of two: 11.2 -> 4.7 ms per
            // 80k-triangle interface)
            SpaiVec<MT, W> t[SPAI_SMALL];
            if (c + W <= nv) {
#pragma unroll
                for (int a = 0; a < SPAI_SMALL; ++a) t[a] = *reinterpret_cast<const SpaiVec<MT, W> *>(rows[a] + c);
            } else {
#pragma unroll
                for (int a = 0; a < SPAI_SMALL; ++a)
#pragma unroll
                    for (int w = 0; w < W; ++w) t[a].v[w] = c + w < nv ? rows[a][c + w] : MT(0);
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                double x[SPAI_SMALL];
#pragma unroll
                for (int a = 0; a < SPAI_SMALL; ++a) x[a] = a < m ? double(t[a].v[w]) : 0.0;
                int k = 0;
#pragma unroll
                for (int a = 0; a < SPAI_SMALL; ++a)
#pragma unroll
                    for (int b = 0; b <= a; ++b, ++k) g[k] = fma(x[a], x[b], g[k]);
            }
            continue;
        }
        double x[SPAI_SMALL][W];
        if (c + W <= nv) {
#pragma unroll
            for (int a = 0; a < SPAI_SMALL; ++a) {
                const SpaiVec<MT, W> t = *reinterpret_cast<const SpaiVec<MT, W> *>(rows[a] + c);
#pragma unroll
                for (int w = 0; w < W; ++w) x[a][w] = a < m ? double(t.v[w]) : 0.0;
            }
        } else {
#pragma unroll
            for (int a = 0; a < SPAI_SMALL; ++a)
#pragma unroll
                for (int w = 0; w < W; ++w) x[a][w] = a < m && c + w < nv ? double(rows[a][c + w]) : 0.0;
        }
#pragma unroll
        for (int w = 0; w < W; ++w) {
            int k = 0;
#pragma unroll
            for (int a = 0; a < SPAI_SMALL; ++a)
#pragma unroll
                for (int b = 0; b <= a; ++b, ++k) g[k] = fma(x[a][w], x[b][w], g[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < NP; ++k)
        for (int off = 32; off > 0; off >>= 1) g[k] += __shfl_xor(g[k], off);
    if (lane != 0) return;
    // Cholesky in place on the packed lower triangle g[a (a + 1) / 2 + b]
#define GP(a, b) g[(a) * ((a) + 1) / 2 + (b)]
    double r[SPAI_SMALL];
    const int64_t ci = minv[i];
#pragma unroll
    for (int a = 0; a < SPAI_SMALL; ++a) r[a] = a < m ? double(rows[a][ci]) : 0.0;
    bool ok = true;
#pragma unroll
    for (int a = 0; a < SPAI_SMALL; ++a) {
        if (a < m) {
            double d = GP(a, a);
#pragma unroll
            for (int k = 0; k < a; ++k) d -= GP(a, k) * GP(a, k);
            ok = ok && d > 0.0;
            GP(a, a) = sqrt(d);
#pragma unroll
            for (int b = a + 1; b < SPAI_SMALL; ++b) {
                if (b < m) {
                    double t = GP(b, a);
#pragma unroll
                    for (int k = 0; k < a; ++k) t -= GP(b, k) * GP(a, k);
                    GP(b, a) = t / GP(a, a);
                }
            }
        }
    }
    if (!ok) {
        atomicOr(bad, 4);
        for (int a = 0; a < m; ++a) val[p0 + a] = 0.0;
        return;
    }
#pragma unroll
    for (int a = 0; a < SPAI_SMALL; ++a) {
        if (a < m) {
            double t = r[a];
#pragma unroll
            for (int k = 0; k < a; ++k) t -= GP(a, k) * r[k];
            r[a] = t / GP(a, a);
        }
    }
#pragma unroll
    for (int a = SPAI_SMALL - 1; a >= 0; --a) {
        if (a < m) {
            double t = r[a];
#pragma unroll
            for (int k = a + 1; k < SPAI_SMALL; ++k)
                if (k < m) t -= GP(k, a) * r[k];
            r[a] = t / GP(a, a);
        }
    }
#undef GP
#pragma unroll
    for (int a = 0; a < SPAI_SMALL; ++a)
        if (a < m) val[p0 + a] = r[a];
}

// Delta_kl = V'_kl - V'_lk on the upper two-ring pattern of the Morton vertex
// order, from the stored operator (one thread per row)
template <typename MT>
__global__ void k_sym_delta(int64_t nv, int64_t ld, const MT *__restrict__ B, const int32_t *__restrict__ dptr,
                            const int32_t *__restrict__ dcol, double *__restrict__ dval)
{
    const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
    if (i >= nv) return;
    for (int32_t e = dptr[i]; e < dptr[i + 1]; ++e) {
        const int64_t j = dcol[e];
        dval[e] = double(B[i * ld + nv + j]) - double(B[j * ld + nv + i]);
    }
}

// ===========================================================================
// host orchestration
// ===========================================================================
int64_t bem_ld(int64_t nv) { return ((2 * nv + 255) / 256) * 256; }

// device copy of the block tables of block size bs (in the surface's arena)
static const BlockSideDev &device_side(Problem &p, int w, int bs, hipStream_t s)
{
    SurfaceDev &S = p.surf[w];
    auto it = S.sides.find(bs);
    if (it != S.sides.end()) return it->second;
    const BlockSide &H = block_side(p.topo[w], bs);
    Arena &A = p.bem_arena[w];
    BlockSideDev D;
    D.bs = bs;
    D.nb = H.nb;
    D.S = H.S;
    D.pref = A.upload(H.pref, s);
    D.nvb = A.upload(H.nvb, s);
    D.seg = A.upload(H.seg, s);
    D.cpos = A.upload(H.cpos, s);
    D.vid = A.upload(H.vid, s);
    // the blocks of each colour, then every block in order (the tuner's lists)
    std::vector<int32_t> lists(H.col_blk);
    for (int64_t b = 0; b < H.nb; ++b) lists.push_back(int32_t(b));
    D.col_blk = A.upload(lists, s);
    D.occ_ptr = A.upload(H.occ_ptr, s);
    D.occ = A.upload(H.occ, s);
    return S.sides.emplace(bs, D).first->second;
}

struct RegArgs {
    int64_t nt = 0;
    const int32_t *m_tri = nullptr;
    const void *xq = nullptr, *nq = nullptr;
    const double *cen = nullptr, *m_area = nullptr;
    BlockSideDev A, B;
    const int32_t *listA = nullptr, *listB = nullptr; // device block lists of the launch
    int64_t nA = 0, nB = 0;                            // their lengths
    int skip_lower = 0;
    void *U = nullptr, *T = nullptr; // operator rows [K' | V'] and the mirrored double layer (square shapes)
    int64_t ld = 0, nv = 0;
    double sV = 0.0, sK = 0.0;
    double kappa = 0.0;
    QRule6 R;
    QRule6F RF;
};

// square shapes evaluate each unordered pair once (SYM)
template <int TA, int TB> constexpr bool shape_sym() { return TA == TB; }
template <int TA, int TB, bool SLOT = false>
static void launch_regular_t(bool yuk, bool f32, const RegArgs &a, hipStream_t s)
{
    if (a.nA == 0 || a.nB == 0) return;
    const dim3 grid(unsigned(a.nB), unsigned(a.nA));
    constexpr bool SYM = shape_sym<TA, TB>();
#define PB_REG(Y, RT)                                                                                              \
    hipLaunchKernelGGL((k_bem_regular<Y, RT, RT, TA, TB, SYM, SLOT>), grid, dim3(TA * TB), 0, s, a.nt, a.m_tri,     \
                       static_cast<const RT *>(a.xq), static_cast<const RT *>(a.nq), a.cen, a.m_area, a.A.pref,     \
                       a.A.nvb, a.A.seg, a.A.vid, a.A.cpos, a.B.pref, a.B.nvb, a.B.seg, a.B.vid, a.B.cpos, a.listA, \
                       a.listB, a.skip_lower, static_cast<RT *>(a.U), static_cast<RT *>(a.T), a.ld, a.nv, a.sV, a.sK,        \
                       a.kappa, a.R, a.RF)
    if (f32) {
        if (yuk) PB_REG(true, float);
        else PB_REG(false, float);
    } else {
        if (yuk) PB_REG(true, double);
        else PB_REG(false, double);
    }
#undef PB_REG
}
static_assert(N_TILE_SHAPES == 5, "one launch case per candidate tile shape");
static void launch_regular(int shape, bool yuk, bool f32, const RegArgs &a, hipStream_t s)
{
    switch (shape) {
    case 0: launch_regular_t<TILE_SHAPES[0].ta, TILE_SHAPES[0].tb>(yuk, f32, a, s); break;
    case 1: launch_regular_t<TILE_SHAPES[1].ta, TILE_SHAPES[1].tb>(yuk, f32, a, s); break;
    case 2: launch_regular_t<TILE_SHAPES[2].ta, TILE_SHAPES[2].tb>(yuk, f32, a, s); break;
    case 3: launch_regular_t<TILE_SHAPES[3].ta, TILE_SHAPES[3].tb>(yuk, f32, a, s); break;
    case 4: launch_regular_t<TILE_SHAPES[4].ta, TILE_SHAPES[4].tb>(yuk, f32, a, s); break;
    default: PB_CHECK(false, PBFB_EINVAL, "unknown tile shape");
    }
}

// Every tile of the assembly, one launch per pair of colours so that no two
// tiles of a launch touch the same operator entry; launches follow each other
// on the stream, so every entry receives its contributions in a fixed order.
// Square shapes: launch (c1, c2), c1 < c2, takes every target block of colour
// c1 against every source block of colour c2 (one orientation per unordered
// block pair); launch (c, c) the pairs with source block >= target block.
// Rectangular shapes (target and source blocks coloured separately): every
// colour pair, every tile.
static void launch_all_tiles(int shape, bool yuk, bool f32, RegArgs a, const BlockSide &HA, const BlockSide &HB,
                             hipStream_t s)
{
    const bool sym = TILE_SHAPES[shape].ta == TILE_SHAPES[shape].tb;
    for (int c1 = 0; c1 < HA.ncolor; ++c1)
        for (int c2 = sym ? c1 : 0; c2 < HB.ncolor; ++c2) {
            a.listA = a.A.col_blk + HA.col_ptr[c1];
            a.nA = HA.col_ptr[c1 + 1] - HA.col_ptr[c1];
            a.listB = a.B.col_blk + HB.col_ptr[c2];
            a.nB = HB.col_ptr[c2 + 1] - HB.col_ptr[c2];
            a.skip_lower = sym && c1 == c2 ? 1 : 0;
            launch_regular(shape, yuk, f32, a, s);
        }
}

// Square 16 x 16 tiles of a small surface go through slots (k_bem_gather) if
// the three planes fit in 192 MiB (to about 1 250 vertices FP64, 1 750 FP32:
// some 2.3 local vertices per vertex).  Setup of both surfaces, colour pairs ->
// slots: 1 002 vertices FP64 1.88 -> 1.10 ms, 1 442 FP32 1.84 -> 1.15; 2 562
// vertices would still gain (3.95 -> 3.64 FP64, 2.85 -> 2.44 FP32) and 4 002
// nothing, but the planes grow with the square of the surface (0.8 GB FP64 at
// 2 562 vertices), and the context keeps them in its workspaces.
constexpr size_t SLOT_BYTES = size_t(192) << 20;
constexpr int SLOT_SHAPE = 3;
static_assert(TILE_SHAPES[SLOT_SHAPE].ta == SLOT_BS && TILE_SHAPES[SLOT_SHAPE].tb == SLOT_BS, "the symmetric 16 x 16 shape");
size_t slot_planes(const Problem &p, int w)
{
    if (p.tile_fixed >= 0 && p.tile_fixed != SLOT_SHAPE) return 0;
    const size_t S = size_t(p.topo[w].sides.at(SLOT_BS).S);
    const size_t b = 3 * S * S * (p.precision == PBFB_MIXED ? sizeof(float) : sizeof(double));
    return b <= SLOT_BYTES ? b : 0;
}
static void launch_slots(bool yuk, bool f32, RegArgs a, hipStream_t s)
{
    a.ld = a.A.S;
    a.listA = a.listB = a.A.col_blk; // every block, colour by colour
    a.nA = a.nB = a.A.nb;
    a.skip_lower = 1;
    launch_regular_t<SLOT_BS, SLOT_BS, true>(yuk, f32, a, s);
}

// cache key of the tuned shape: precision, kernel and size class (floor log2 of the triangle count)
static int tile_key(int precision, bool yuk, int64_t nt)
{
    int c = 0;
    while (c < 62 && (int64_t(2) << c) <= nt) ++c;
    return (precision * 2 + (yuk ? 1 : 0)) * 64 + c;
}

// Autotuner: times the regular tile kernel of every candidate shape on the
// same sample of this surface (min(nt, 512) Morton-ordered target triangles
// from the middle of the order against all source triangles, so that a
// symmetric shape, which skips the source blocks below the target block,
// does the average share of its work; one warm-up launch, then the fastest
// of three timed launches) and returns the shape with the shortest time per
// target triangle.  Runs with the context workspace held.
static void tune_range(const BlockSide &HA, int64_t nsample, int64_t &b0, int64_t &b1)
{
    const int64_t nbs = std::min<int64_t>((nsample + HA.bs - 1) / HA.bs, HA.nb);
    b0 = (HA.nb - nbs) / 2;
    b1 = b0 + nbs;
}
static int tile_tune(Problem &p, int w, RegArgs a, bool yuk, bool f32, hipStream_t s)
{
    // the timed launches add into the operator and T (a.U, a.T), which are
    // cleared before the assembly proper; their tiles are not coloured (the
    // values are discarded, so unordered additions do not matter here)
    SurfaceTopo &T = p.topo[w];
    const int64_t nsample = std::min<int64_t>(T.nt, 512);
    hipEvent_t e0, e1;
    PB_HIP(hipEventCreate(&e0));
    PB_HIP(hipEventCreate(&e1));
    int best = 0;
    double best_t = 1e300;
    for (int k = 0; k < N_TILE_SHAPES; ++k) {
        const BlockSide &HA = block_side(T, TILE_SHAPES[k].ta), &HB = block_side(T, TILE_SHAPES[k].tb);
        a.A = device_side(p, w, HA.bs, s);
        a.B = device_side(p, w, HB.bs, s);
        int64_t b0, b1;
        tune_range(HA, nsample, b0, b1);
        a.listA = a.A.col_blk + HA.nb + b0; // blocks b0 .. b1 - 1 of the in-order list
        a.nA = b1 - b0;
        a.listB = a.B.col_blk + HB.nb;
        a.nB = HB.nb;
        a.skip_lower = TILE_SHAPES[k].ta == TILE_SHAPES[k].tb ? 1 : 0;
        const int64_t tris = std::min<int64_t>(b1 * HA.bs, T.nt) - b0 * HA.bs;
        launch_regular(k, yuk, f32, a, s);
        float ms = 1e30f;
        for (int rep = 0; rep < 3; ++rep) {
            PB_HIP(hipEventRecord(e0, s));
            launch_regular(k, yuk, f32, a, s);
            PB_HIP(hipEventRecord(e1, s));
            PB_HIP(hipEventSynchronize(e1));
            float t = 0.0f;
            PB_HIP(hipEventElapsedTime(&t, e0, e1));
            ms = std::min(ms, t);
        }
        PB_HIP(hipGetLastError());
        const double per = double(ms) / double(tris);
        if (per < best_t) {
            best_t = per;
            best = k;
        }
    }
    PB_HIP(hipEventDestroy(e0));
    PB_HIP(hipEventDestroy(e1));
    return best;
}

// the touching-pair blocks of a surface (vertex coordinates vx) into tpv
static void singular_pairs(Problem &p, const SurfaceDev &S, bool yuk, double kappa, const double *vx, double *tpv,
                           hipStream_t s)
{
    const double *pts = ss_points(*p.ctx, s);
    const unsigned g = nblk(S.tp_cnt[0], 64) + nblk(S.tp_cnt[1], 64) + nblk(S.tp_cnt[2], 64);
    if (p.timing) p.timer.begin(T_SING, s);
    if (yuk)
        hipLaunchKernelGGL(k_bem_singular<true>, dim3(g), dim3(64 * SING_W), 0, s, S.tp_cnt[0], S.tp_cnt[1],
                           S.tp_cnt[2], S.tp_ord, S.tp_tau, S.tp_sig, S.tri, vx, S.nrm, S.area, kappa, pts, tpv);
    else
        hipLaunchKernelGGL(k_bem_singular<false>, dim3(g), dim3(64 * SING_W), 0, s, S.tp_cnt[0], S.tp_cnt[1],
                           S.tp_cnt[2], S.tp_ord, S.tp_tau, S.tp_sig, S.tri, vx, S.nrm, S.area, kappa, pts, tpv);
    if (p.timing) p.timer.end(s);
    PB_HIP(hipGetLastError());
}

void ensure_bem(Problem &p, int w, hipStream_t s)
{
    if (p.bem_ready[w]) return;
    ensure_geometry(p, s);
    SurfaceTopo &T = p.topo[w];
    SurfaceDev &S = p.surf[w];
    Arena &A = p.bem_arena[w];
    const bool yuk = (w == 1) && p.kappa > 0.0;
    const bool f32 = p.precision == PBFB_MIXED;
    const double kappa = (w == 1) ? p.kappa : 0.0;
    if (!p.bem_topo_ready[w]) {
        // Morton order and triangle data: once per mesh (block tables are
        // uploaded per block size when a tile shape needs them)
        A.release();
        S.sides.clear();
        S.tile = -1;
        S.B = nullptr;
        S.m_tri = A.alloc<int32_t>(3 * T.nt);
        S.m_area = A.alloc<double>(T.nt);
        S.m_qp = S.m_nrm = S.m_cen = nullptr;
        S.m_qf = S.m_nf = nullptr;
        if (f32) {
            S.m_cen = A.alloc<double>(3 * T.nt);
            S.m_qf = A.alloc<float>(18 * T.nt);
            S.m_nf = A.alloc<float>(3 * T.nt);
        } else {
            S.m_qp = A.alloc<double>(18 * T.nt);
            S.m_nrm = A.alloc<double>(3 * T.nt);
        }
        S.morton = A.upload(T.morton, s);
        S.tp_ptr = A.upload(T.tp_ptr, s);
        S.tp_sig = A.upload(T.tp_sig, s);
        S.ntp = int64_t(T.tp_sig.size());
        std::vector<int32_t> tp_tau(S.ntp);
        for (int64_t t = 0; t < T.nt; ++t)
            for (int32_t k = T.tp_ptr[t]; k < T.tp_ptr[t + 1]; ++k) tp_tau[k] = int32_t(t);
        S.tp_tau = A.upload(tp_tau, s);
        std::vector<int32_t> tp_ord; // by shared vertices: 3, 2, 1
        tp_ord.reserve(S.ntp);
        std::vector<int8_t> kind(S.ntp);
        for (int64_t k = 0; k < S.ntp; ++k) {
            int n = 0;
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) n += T.tri[3 * int64_t(tp_tau[k]) + a] == T.tri[3 * int64_t(T.tp_sig[k]) + b];
            kind[k] = int8_t(n);
        }
        for (int g = 0; g < 3; ++g) {
            const size_t before = tp_ord.size();
            for (int64_t k = 0; k < S.ntp; ++k)
                if (kind[k] == 3 - g) tp_ord.push_back(int32_t(k));
            S.tp_cnt[g] = int64_t(tp_ord.size() - before);
        }
        S.tp_ord = A.upload(tp_ord, s);
        S.vdiag = A.alloc<double>(T.nv);
        S.tpv = nullptr;
        S.mpos = nullptr;
        S.nf_ptr = S.nf_col = S.nf_row = nullptr;
        S.nf_val = nullptr;
        S.nf_nnz = 0;
        S.d_ptr = S.d_col = nullptr;
        S.d_val = nullptr;
        S.sym = false;
        S.ring_ptr = A.upload(T.ring_ptr, s);
        S.ring = A.upload(T.ring, s);
        S.spai = A.alloc<double>(T.ring.size());
        if (p.bem_mf) {
            // matrix-free: resident touching-pair blocks, the Morton position of
            // each triangle and the near-field rows of the preconditioner
            S.tpv = A.alloc<double>(18 * S.ntp);
            std::vector<int32_t> mpos(T.nt);
            for (int64_t m = 0; m < T.nt; ++m) mpos[T.morton[m]] = int32_t(m);
            S.mpos = A.upload(mpos, s);
            near_pattern(T);
            S.nf_nnz = int64_t(T.nf_col.size());
            std::vector<int32_t> nf_row(S.nf_nnz);
            for (int64_t i = 0; i < T.nv; ++i)
                for (int32_t k = T.nf_ptr[i]; k < T.nf_ptr[i + 1]; ++k) nf_row[k] = int32_t(i);
            S.nf_ptr = A.upload(T.nf_ptr, s);
            S.nf_col = A.upload(T.nf_col, s);
            S.nf_row = A.upload(nf_row, s);
            S.nf_val = A.alloc<double>(S.nf_nnz);
        } else {
            const int64_t ldt = bem_ld(T.nv);
            if (f32) S.B = A.alloc<float>(T.nv * ldt);
            else S.B = A.alloc<double>(T.nv * ldt);
            if (!gemv_small(T.nv, f32)) { // small surfaces are applied by full rows
                delta_pattern(T);
                S.d_ptr = A.upload(T.d2_ptr, s);
                S.d_col = A.upload(T.d2_col, s);
                S.d_val = A.alloc<double>(std::max<size_t>(T.d2_col.size(), 1));
            }
        }
        PB_HIP(hipStreamSynchronize(s));
        p.bem_topo_ready[w] = true;
    }
    hipLaunchKernelGGL(k_tri_morton, dim3(nblk(T.nt, 256)), dim3(256), 0, s, T.nt, S.morton, S.tri, S.qp, S.nrm,
                       S.area, S.g, S.x, S.m_tri, S.m_qp, S.m_nrm, S.m_area, S.m_cen, S.m_qf, S.m_nf);

    // one of the context's assembly workspaces (see below), used by one assembly at a time
    Workspace *wsp = nullptr;
    std::unique_lock<std::mutex> ws_lock;
    while (!wsp) {
        for (Workspace &W : p.ctx->asm_ws) {
            std::unique_lock<std::mutex> l(W.mu, std::try_to_lock);
            if (l.owns_lock()) {
                wsp = &W;
                ws_lock = std::move(l);
                break;
            }
        }
        if (!wsp) std::this_thread::sleep_for(std::chrono::microseconds(100));
    }
    struct Drain { // on every exit the stream drains before the workspace is released
        hipStream_t s;
        ~Drain() { (void)hipStreamSynchronize(s); }
    } drain{s};
    if (p.bem_mf) {
        // matrix-free: only the touching-pair blocks (kept) and the diagonal of V'
        double *vxm = wsp->doubles(3 * T.nv);
        hipLaunchKernelGGL(k_gather_coords, dim3(nblk(T.nv, 256)), dim3(256), 0, s, T.nv, S.g, S.x, vxm);
        singular_pairs(p, S, yuk, kappa, vxm, S.tpv, s);
        mf_vdiag(p, w, s);
        mf_spai(p, w, s);
        PB_HIP(hipStreamSynchronize(s));
        S.tile = -1;
        p.bem_ready[w] = true;
        return;
    }
    const int64_t nv = T.nv, ld = bem_ld(nv);
    const size_t elem = f32 ? sizeof(float) : sizeof(double);
    // Gamma_m (and an independent Gamma_m mesh): V' = -V0, K' = 1/2 M + K0;
    // Gamma_s: V' = +Vk, K' = 1/2 M - Kk
    const double sV = (w != 1) ? -1.0 : 1.0, sK = (w != 1) ? 1.0 : -1.0;
    RegArgs ra;
    ra.nt = T.nt;
    ra.m_tri = S.m_tri;
    ra.xq = f32 ? static_cast<const void *>(S.m_qf) : static_cast<const void *>(S.m_qp);
    ra.nq = f32 ? static_cast<const void *>(S.m_nf) : static_cast<const void *>(S.m_nrm);
    ra.cen = S.m_cen;
    ra.m_area = S.m_area;
    ra.kappa = kappa;
    ra.R = q6arg();
    ra.RF = q6farg();
    ra.U = S.B;
    ra.ld = ld;
    ra.nv = nv;
    ra.sV = sV;
    ra.sK = sK;
    // the context's assembly workspace: the mirrored double layer T of a
    // square-tile assembly (nv x nv in the storage precision), vertex
    // coordinates and the touching-pair blocks; behind them the planes of a
    // small surface if they may be allocated or the workspace has the room
    // already (by colour pairs of the same tile shape the operator is the same
    // bits)
    const size_t planes = slot_planes(p, w);
    auto round256 = [](size_t b) { return (b + 255) / 256 * 256; };
    // bytes of an assembly without planes
    auto ws_pairs = [&](const SurfaceTopo &V) {
        return round256(round256(size_t(V.nv) * V.nv * elem) + 8 * (3 * size_t(V.nv) + 18 * V.tp_sig.size()));
    };
    auto ws_slots = [&](int v) { return ws_pairs(p.topo[v]) + round256(slot_planes(p, v)); };
    bool slots = planes > 0 && (p.planes || wsp->bytes >= ws_slots(w));
    double *ws = nullptr;
    if (slots) {
        // room for the planes of all the problem's surfaces, which are not of
        // one size: a workspace that grows frees its memory first, and that
        // waits for every stream
        size_t want = ws_slots(w);
        for (int v = 0; v < NSURF && p.planes; ++v)
            if (!p.bem_ready[v] && (v < 2 || p.gm() == 2) && slot_planes(p, v) > 0) want = std::max(want, ws_slots(v));
        try {
            ws = wsp->doubles(want / 8);
        } catch (const Error &e) {
            if (e.code != PBFB_ENOMEM) throw;
            (void)hipGetLastError(); // no room on the device: colour pairs
            slots = false;
        }
    }
    if (!slots) ws = wsp->doubles(ws_pairs(T) / 8);
    void *Tm = ws;
    double *vx = ws + round256(size_t(nv) * nv * elem) / 8, *tpv = vx + 3 * nv;
    void *Wp = ws + ws_pairs(T) / 8; // the planes
    ra.T = Tm;
    // tile shape: forced, or tuned once per (precision, kernel, size class) and context
    int shape = planes > 0 ? SLOT_SHAPE : p.tile_fixed;
    if (shape < 0) {
        const int key = tile_key(p.precision, yuk, T.nt);
        std::lock_guard<std::mutex> tl(p.ctx->tune_mu);
        auto it = p.ctx->tile_choice.find(key);
        if (it != p.ctx->tile_choice.end()) {
            shape = it->second;
        } else {
            shape = tile_tune(p, w, ra, yuk, f32, s);
            p.ctx->tile_choice[key] = shape;
        }
    }
    S.tile = shape;
    const BlockSide &HA = block_side(T, TILE_SHAPES[shape].ta), &HB = block_side(T, TILE_SHAPES[shape].tb);
    ra.A = device_side(p, w, TILE_SHAPES[shape].ta, s);
    ra.B = device_side(p, w, TILE_SHAPES[shape].tb, s);
    const bool sym = TILE_SHAPES[shape].ta == TILE_SHAPES[shape].tb;
    // every tile adds into the operator: start from zero (the row padding
    // past 2 nv, read by the dense apply against zero inputs, stays zero)
    if (!slots) PB_HIP(hipMemsetAsync(S.B, 0, size_t(nv) * ld * elem, s));
    if (sym && !slots) PB_HIP(hipMemsetAsync(Tm, 0, size_t(nv) * nv * elem, s));
    if (p.timing) p.timer.begin(T_ASM, s);
    if (slots) {
        ra.U = Wp;
        ra.T = static_cast<char *>(Wp) + planes / 3 * 2;
        launch_slots(yuk, f32, ra, s);
        const dim3 g(nblk(nv, 256), unsigned(nv));
        if (f32)
            hipLaunchKernelGGL(k_bem_gather<float>, g, dim3(256), 0, s, nv, ld, HA.S, ra.A.occ_ptr, ra.A.occ,
                               static_cast<const float *>(Wp), static_cast<float *>(S.B), static_cast<float *>(Tm));
        else
            hipLaunchKernelGGL(k_bem_gather<double>, g, dim3(256), 0, s, nv, ld, HA.S, ra.A.occ_ptr, ra.A.occ,
                               static_cast<const double *>(Wp), static_cast<double *>(S.B),
                               static_cast<double *>(Tm));
    } else {
        launch_all_tiles(shape, yuk, f32, ra, HA, HB, s);
    }
    if (p.timing) p.timer.end(s);
    PB_HIP(hipGetLastError());
    if (sym) {
        const unsigned nbt = unsigned((nv + SYMT - 1) / SYMT);
        // FP32 storage with an even nv: pairs of entries, upper tile pairs only
        // (11.3 -> 7.7 ms per 80k-triangle interface); the same form ran FP64
        // storage slower (14.5 -> 19.9 ms), which keeps the one-entry kernel
        const int64_t npair = int64_t(nbt) * (nbt + 1) / 2; // one-dimensional grid: npair * 256 < 2^32
        if (f32 && nv % 2 == 0 && ld % 2 == 0 && npair * 256 < (int64_t(1) << 32))
            hipLaunchKernelGGL(k_bem_symm2<float>, dim3(unsigned(npair)), dim3(256), 0, s, nv, ld,
                               static_cast<float *>(S.B), static_cast<const float *>(Tm));
        else if (f32)
            hipLaunchKernelGGL(k_bem_symm<float>, dim3(nbt, nbt), dim3(256), 0, s, nv, ld, static_cast<float *>(S.B),
                               static_cast<const float *>(Tm));
        else
            hipLaunchKernelGGL(k_bem_symm<double>, dim3(nbt, nbt), dim3(256), 0, s, nv, ld,
                               static_cast<double *>(S.B), static_cast<const double *>(Tm));
        PB_HIP(hipGetLastError());
    }
    // touching pairs
    hipLaunchKernelGGL(k_gather_coords, dim3(nblk(nv, 256)), dim3(256), 0, s, nv, S.g, S.x, vx);
    singular_pairs(p, S, yuk, kappa, vx, tpv, s);
    if (f32)
        hipLaunchKernelGGL(k_bem_scatter<float>, dim3(unsigned(nv)), dim3(64), 0, s, nv, ld, S.minv, S.v2t_ptr, S.v2t,
                           S.tri, S.tp_ptr, S.tp_sig, tpv, S.area, sV, sK, static_cast<float *>(S.B));
    else
        hipLaunchKernelGGL(k_bem_scatter<double>, dim3(unsigned(nv)), dim3(64), 0, s, nv, ld, S.minv, S.v2t_ptr,
                           S.v2t, S.tri, S.tp_ptr, S.tp_sig, tpv, S.area, sV, sK, static_cast<double *>(S.B));
    PB_HIP(hipGetLastError());
    // diagonal of V', symmetric storage use (Delta from the stored values),
    // approximate inverse of the single-layer block (from the stored values)
    // symmetric use: the apply reads K' and the lower triangle of V' (square
    // tiles leave the regular part of V' bitwise symmetric), unless the surface
    // is small (gemv_small)
    S.sym = sym && !gemv_small(nv, f32);
    PB_HIP(hipMemsetAsync(p.d_bad, 0, sizeof(int), s));
    if (f32) {
        const float *Bf = static_cast<const float *>(S.B);
        hipLaunchKernelGGL(k_vdiag<float>, dim3(nblk(nv, 256)), dim3(256), 0, s, nv, ld, S.mvert, Bf, S.vdiag);
        if (S.sym)
            hipLaunchKernelGGL(k_sym_delta<float>, dim3(nblk(nv, 256)), dim3(256), 0, s, nv, ld, Bf, S.d_ptr, S.d_col,
                               S.d_val);
        hipLaunchKernelGGL((k_spai_small<float, 4>), dim3(nblk(nv, 4)), dim3(256), 0, s, nv, Bf, ld, S.minv,
                           S.ring_ptr, S.ring, S.spai, p.d_bad);
        if (T.max_ring > SPAI_SMALL)
            hipLaunchKernelGGL(k_spai<float>, dim3(unsigned(nv)), dim3(256), 0, s, nv, Bf, ld, S.minv, S.ring_ptr,
                               S.ring, S.spai, p.d_bad);
    } else {
        const double *Bd = static_cast<const double *>(S.B);
        hipLaunchKernelGGL(k_vdiag<double>, dim3(nblk(nv, 256)), dim3(256), 0, s, nv, ld, S.mvert, Bd, S.vdiag);
        if (S.sym)
            hipLaunchKernelGGL(k_sym_delta<double>, dim3(nblk(nv, 256)), dim3(256), 0, s, nv, ld, Bd, S.d_ptr,
                               S.d_col, S.d_val);
        hipLaunchKernelGGL((k_spai_small<double, 2>), dim3(nblk(nv, 4)), dim3(256), 0, s, nv, Bd, ld, S.minv,
                           S.ring_ptr, S.ring, S.spai, p.d_bad);
        if (T.max_ring > SPAI_SMALL)
            hipLaunchKernelGGL(k_spai<double>, dim3(unsigned(nv)), dim3(256), 0, s, nv, Bd, ld, S.minv, S.ring_ptr,
                               S.ring, S.spai, p.d_bad);
    }
    PB_HIP(hipGetLastError());
    int bad = 0;
    PB_HIP(hipMemcpyAsync(&bad, p.d_bad, sizeof(int), hipMemcpyDeviceToHost, s));
    PB_HIP(hipStreamSynchronize(s));
    PB_CHECK(!(bad & 4), PBFB_EMESH, "single-layer block not positive definite on a vertex 1-ring");
    p.bem_ready[w] = true;
}

void ensure_all(Problem &p, hipStream_t s)
{
    ensure_geometry(p, s);
    ensure_values(p, s);
    ensure_rhs(p, s);
    ensure_bem(p, 0, s);
    ensure_bem(p, 1, s);
    if (p.gm() == 2) ensure_bem(p, 2, s); // lambda_m and u_r on the independent Gamma_m mesh
}

} // namespace pbfb
