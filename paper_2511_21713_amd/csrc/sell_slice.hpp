// FEM rows of the coupled operator in sliced ELL: a slice is 64 consecutive
// rows (one wavefront wide); entry k of row 64 q + l is stored at
// sptr[q] + 64 k + l for k below the slice width w_q = (sptr[q+1] - sptr[q]) / 64,
// columns ascending, padding entries column = row and value 0.  Row lengths
// of the layered shell mesh are nearly uniform, so the padding is about 1 %
// of the entries and every value and column load of a wavefront is one
// contiguous 512- or 256-byte segment, with no row-pointer load in front of
// it.
//
// A workgroup of four wavefronts owns one slice: wavefront v takes the
// entries k = v, v + 4, v + 8, ... of its 64 rows, issuing SELL_U value and
// column loads and then SELL_U gathers of the input before it waits, so a
// slice of width 16 is read by one round of loads.  The four partial sums of
// a row are added in wavefront order through LDS (bitwise reproducible).
// FP32 values are widened; products and sums are FP64.
//
// A row of more than LONG_ROW entries (a node where a coarse fan of tets
// meets, such as the centre of a meshed solute) would set the width of its
// whole slice and be walked by one lane.  Such rows hold padding only in their
// slice; their entries follow the slices, contiguous, and the workgroup of the
// slice adds each of them with all its lanes (sell_long).
//
// This is the bandwidth-bound sparse kernel of every coupled apply and of
// every Chebyshev term of the FEM-block preconditioner.  Its loads are plain
// (cached): the Chebyshev terms read the same slices many times in a row.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pbfb {

constexpr int SELL_W = 4; // wavefronts per slice (one workgroup of 256 threads)
constexpr int SELL_U = 4; // entries per lane in flight

// long rows of a matrix: those of slice q are ptr[q] .. ptr[q + 1] - 1 (null:
// the matrix has none), long row l is row[l] with entries off[l] .. off[l + 1] - 1
struct SellLong {
    const int32_t *ptr = nullptr, *row = nullptr, *off = nullptr;
};

// Partial sum of row 64 q + lane over the entries k = wv, wv + 4, ... of
// slice q (entries from b0, width w) with input entry x(column).  FEM_ONLY skips the coupling columns
// (index >= nn).
template <typename VT, bool FEM_ONLY, typename XF>
__device__ inline double sell_part_of(int32_t b0, int32_t w, const int32_t *__restrict__ col,
                                      const VT *__restrict__ val, XF &&x, int lane, int wv, int64_t nn)
{
    double acc = 0.0;
    for (int k0 = wv; k0 < w; k0 += SELL_W * SELL_U) {
        int32_t c[SELL_U];
        VT v[SELL_U];
#pragma unroll
        for (int j = 0; j < SELL_U; ++j) {
            // a clamped index keeps the load in bounds; its term is dropped below
            const int k = min(k0 + SELL_W * j, w - 1);
            const int64_t at = b0 + int64_t(k) * 64 + lane;
            c[j] = col[at];
            v[j] = val[at];
        }
        double xv[SELL_U];
#pragma unroll
        for (int j = 0; j < SELL_U; ++j) xv[j] = (FEM_ONLY && c[j] >= nn) ? 0.0 : x(c[j]);
#pragma unroll
        for (int j = 0; j < SELL_U; ++j)
            if (k0 + SELL_W * j < w) acc = fma(double(v[j]), xv[j], acc);
    }
    return acc;
}

// Sum of the four wavefront partials of each row of the slice, in order;
// valid in wavefront 0 (every thread of the workgroup must call it).
__device__ inline double sell_reduce(double part, int lane, int wv)
{
    __shared__ double red[SELL_W][64];
    red[wv][lane] = part;
    __syncthreads();
    double s = 0.0;
    if (wv == 0) {
        s = red[0][lane];
#pragma unroll
        for (int v = 1; v < SELL_W; ++v) s += red[v][lane];
    }
    return s;
}

// The long rows of slice q into acc of their lanes of wavefront 0 (every thread
// of the workgroup must call it; x and FEM_ONLY as in sell_part_of)
template <typename VT, bool FEM_ONLY, typename XF>
__device__ inline void sell_long(const SellLong &L, const int32_t *__restrict__ col, const VT *__restrict__ val, XF &&x,
                                 int64_t q, int lane, int wv, int64_t nn, double &acc)
{
    if (!L.ptr) return;
    __shared__ double red[SELL_W];
    for (int32_t l = L.ptr[q]; l < L.ptr[q + 1]; ++l) {
        double t = 0.0;
        for (int32_t e = L.off[l] + 64 * wv + lane; e < L.off[l + 1]; e += 64 * SELL_W) {
            const int32_t c = col[e];
            if (!FEM_ONLY || c < nn) t = fma(double(val[e]), x(c), t);
        }
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
        if (lane == 0) red[wv] = t;
        __syncthreads();
        if (wv == 0 && lane == int(L.row[l] - q * 64)) acc = (red[0] + red[1]) + (red[2] + red[3]);
        __syncthreads();
    }
}

// One row product per lane of wavefront 0 for the 64 rows of slice q, long
// rows included
template <typename VT, bool FEM_ONLY, typename XF>
__device__ inline double sell_rows(int32_t b0, int32_t w, const SellLong &L, const int32_t *__restrict__ col,
                                   const VT *__restrict__ val, XF &&x, int64_t q, int lane, int wv, int64_t nn)
{
    double acc = sell_reduce(sell_part_of<VT, FEM_ONLY>(b0, w, col, val, x, lane, wv, nn), lane, wv);
    sell_long<VT, FEM_ONLY>(L, col, val, x, q, lane, wv, nn, acc);
    return acc;
}

} // namespace pbfb
