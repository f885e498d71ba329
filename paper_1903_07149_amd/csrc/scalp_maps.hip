// scalp_maps.hip -- per-pixel maps around the clustering path.
//
//   k_boundary_frequency  fraction of a stack of label maps in which a pixel
//                         is a superpixel boundary pixel (a 4-neighbour inside
//                         the image carries another label): the multi-scale
//                         boundary map whose thresholds give the
//                         precision-recall curves of Sec. III-A.2.
//   k_gradient_*          a soft contour prior computed on the device: the
//                         central-difference gradient magnitude of the Lab
//                         image (replicated borders), divided by its maximum,
//                         in FP64 and rounded once to FP32.  The paper feeds
//                         the contour map C of Sec. II-D from an external
//                         detector (Sec. II-E); this is a detector-free
//                         stand-in that needs no trained model.
//   k_prepare_gradient    the same prior fused into the packing of
//                         (l, a, b, w): C never reaches memory.
#include <algorithm>

#include "scalp_device.h"

namespace scalp {
namespace {

using namespace dev;

// The boundary map runs 256-thread blocks over row segments: x from the block
// column, rows strided by the grid's height (no per-pixel division).
#define FOR_PIXELS(W, H)                                                     \
    const int x = blockIdx.x * 256 + threadIdx.x;                            \
    for (int y = blockIdx.y; y < (H); y += gridDim.y)                        \
        if (x < (W))

__global__ __launch_bounds__(256) void k_boundary_frequency(int W, int H, int n,
                                                            const int* __restrict__ labels,
                                                            float* __restrict__ out) {
    const long long N = (long long)W * H;
    FOR_PIXELS(W, H) {
        const long long p = (long long)y * W + x;
        int c = 0;
        for (int s = 0; s < n; ++s) {
            const int* L = labels + N * s;
            const int v = L[p];
            c += ((x + 1 < W && L[p + 1] != v) || (x > 0 && L[p - 1] != v) ||
                  (y + 1 < H && L[p + W] != v) || (y > 0 && L[p - W] != v)) ? 1 : 0;
        }
        out[p] = (float)c / (float)n;
    }
}

// The gradient kernels give a wave kGradCols columns of kGradRows rows: a lane
// loads its column's kGradRows + 2 texels, 12 bytes a load and all in flight
// together, and takes the left and right neighbours from the next lanes (lanes 0
// and 63 only hold the columns beside).  A lane per pixel made 12 loads of 4
// bytes for each pixel; with the neighbours loaded too (14 loads of 12 bytes for
// 4 rows) the kernels took as long as with those.
constexpr int kGradRows = 4, kGradCols = 62;
constexpr int kGradWG = 512, kGradWaves = kGradWG / 64;

struct Texel {
    float c[3];
};

__device__ __forceinline__ Texel texel(const float* __restrict__ lab, long long p) {
    Texel t;
    __builtin_memcpy(&t, lab + 3 * p, sizeof(t));
    return t;
}

// Item t of a wave: rows y0 ... and the lane's column x, -1 and W included for
// the columns beside.
__device__ __forceinline__ void grad_item(int t, int wx, int& x, int& y0) {
    const int rg = t / wx;
    y0 = kGradRows * rg;
    x = kGradCols * (t - rg * wx) + (int)(threadIdx.x & 63) - 1;
}

// Whether the lane's column is one of the item's own.
__device__ __forceinline__ bool grad_own(int x, int W) {
    const int lane = threadIdx.x & 63;
    return lane >= 1 && lane <= kGradCols && x < W;
}

// Rows y0 - 1 ... of column x; beyond the image the border repeats.
__device__ __forceinline__ void grad_load(const float* __restrict__ lab, int W, int H, int x, int y0,
                                          Texel mid[kGradRows + 2]) {
    const int xc = min(max(x, 0), W - 1);
#pragma unroll
    for (int i = 0; i < kGradRows + 2; ++i)
        mid[i] = texel(lab, (long long)min(max(y0 + i - 1, 0), H - 1) * W + xc);
}

// The next lane's value, below (DPP wave_shr:1) or above (wave_shl:1).
template <int CTRL>
__device__ __forceinline__ float beside(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Four times the squared gradient magnitude of row i in FP64: central
// differences, replicated borders, channels summed in order.  The differences
// are not halved: a factor 4 is exact, as no square of a difference of two
// floats is subnormal.  All lanes call.
__device__ __forceinline__ double grad_sq4(const Texel mid[kGradRows + 2], int i) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float v = mid[i + 1].c[c];
        const double gx = (double)beside<0x130>(v) - (double)beside<0x138>(v);
        const double gy = (double)mid[i + 2].c[c] - (double)mid[i].c[c];
        s = s + (gx * gx + gy * gy);
    }
    return s;
}

template <int CTRL>
__device__ __forceinline__ unsigned long long max_dpp(unsigned long long v) {
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
    const unsigned long long w = ((unsigned long long)hi << 32) | lo;
    return w > v ? w : v;
}

// Largest v of the workgroup, to all its lanes.  All call, once.
__device__ __forceinline__ unsigned long long block_max(unsigned long long v,
                                                        unsigned long long red[kGradWaves]) {
    v = max_dpp<0x111>(v);   // row_shr 1, 2, 4, 8: lane 15 of a row has its largest
    v = max_dpp<0x112>(v);
    v = max_dpp<0x114>(v);
    v = max_dpp<0x118>(v);
    v = max_dpp<0x142>(v);   // row_bcast 15, 31: lane 63 has the wave's
    v = max_dpp<0x143>(v);
    if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int i = 1; i < kGradWaves; ++i) v = red[i] > v ? red[i] : v;
    return v;
}

// First item of the wave: a band of rows per XCD, the same in both passes.
__device__ __forceinline__ int grad_first() {
    return xcd_remap(blockIdx.x, gridDim.x) * kGradWaves +
           __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
}

// mx[block] = the largest of the block's grad_sq4 (at most kGradSlots blocks, each
// with a slot of its own: nothing to clear before, and no atomics).  Squares are
// >= 0, so their FP64 bit patterns order like the values; the correctly rounded
// square root is monotone, so the root of the largest square is the largest
// magnitude.
//
// What bounds it: the memory and a launch's fixed cost.  1920x1080: 12.9 us and
// 1.5 us of clearing before, 7.4 now (25 MB); without a band of rows per XCD,
// whose neighbours then share an L2, 10.9.
__global__ __launch_bounds__(kGradWG) void k_gradient_max(const float* __restrict__ lab, int W,
                                                             int H, int wx, int items,
                                                             unsigned long long* __restrict__ mx) {
    __shared__ unsigned long long red[kGradWaves];
    unsigned long long m = 0;
    for (int t = grad_first(); t < items; t += gridDim.x * kGradWaves) {
        int x, y0;
        grad_item(t, wx, x, y0);
        Texel mid[kGradRows + 2];
        grad_load(lab, W, H, x, y0, mid);
#pragma unroll
        for (int i = 0; i < kGradRows; ++i) {
            const unsigned long long b = (unsigned long long)__double_as_longlong(grad_sq4(mid, i));
            m = y0 + i < H && grad_own(x, W) && b > m ? b : m;
        }
    }
    m = block_max(m, red);
    if (threadIdx.x == 0) mx[blockIdx.x] = m;
}

// Contour value of a pixel as the standalone map stores it: sqrt(sq4 / 4) / m
// in FP64, rounded once to FP32 (m > 0).  Sets `exact` unless its estimate is that
// value: with half_inv = 0.5 / m, v_rsq_f64 and one Newton step are within 2^-44
// of the quotient, which rounds to the same FP32 unless the 29 bits that the
// rounding drops lie within 2^13 (2^-39) of half.  Subnormal results, zeros, NaN
// and infinities are left to the root and the division, too.
__device__ __forceinline__ float contour_near(double sq4, double half_inv, bool& exact) {
    const double y = __builtin_amdgcn_rsq(sq4);
    const double g = sq4 * y;
    const double q = fma(g, fma(-0.5 * y, g, 0.5), g) * half_inv;
    const unsigned long long b = (unsigned long long)__double_as_longlong(q);
    const unsigned hi = (unsigned)(b >> 32), low = (unsigned)b & 0x1fffffffu;
    exact = hi - 0x38700000u >= 0x07900000u || low - 0x0fffe000u < 0x4000u;   // hi: 2^-120 <= q < 2
    return (float)q;
}

__device__ __forceinline__ float contour_exact(double sq4, double m) {
    return m > 0.0 ? (float)(sqrt(0.25 * sq4) / m) : 0.0f;
}

// Rows y0 ... of the lane's column; those that need contour_exact go through one
// rolled loop, as a copy of the root and the division per row costs more in
// instruction fetches than their arithmetic.
__device__ __forceinline__ void contour_rows(const Texel mid[kGradRows + 2], double m, double half_inv,
                                             float v[kGradRows]) {
    unsigned need = 0;
    double sq[kGradRows];
#pragma unroll
    for (int i = 0; i < kGradRows; ++i) {
        bool exact;
        sq[i] = grad_sq4(mid, i);
        v[i] = contour_near(sq[i], half_inv, exact);
        need |= exact ? 1u << i : 0u;
    }
    if (!(m > 0.0)) need = (1u << kGradRows) - 1u;
#pragma unroll 1
    for (int r = 0; __ballot(need) != 0ULL; need &= ~(1u << r), ++r) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < kGradRows; ++i) s = r == i ? sq[i] : s;
        const float e = contour_exact(s, m);
#pragma unroll
        for (int i = 0; i < kGradRows; ++i) v[i] = r == i && (need >> i & 1u) ? e : v[i];
    }
}

// 1920x1080: 11.2 us before, 9.5 now (25 MB in, 8 MB out; 7.6 with no root and
// division at all).
__global__ __launch_bounds__(kGradWG) void k_gradient_normalise(const float* __restrict__ lab, int W,
                                                            int H, int wx, int items,
                                                            const unsigned long long* __restrict__ mx,
                                                            int n, float* __restrict__ out) {
    __shared__ unsigned long long red[kGradWaves];
    unsigned long long top = (int)threadIdx.x < n ? mx[threadIdx.x] : 0ULL;
    int t = grad_first(), x, y0;
    Texel mid[kGradRows + 2];
    grad_item(min(t, items - 1), wx, x, y0);
    grad_load(lab, W, H, x, y0, mid);
    top = block_max(top, red);                               // while the texels come
    const double m = sqrt(0.25 * __longlong_as_double((long long)top)), half_inv = 0.5 / m;
    while (t < items) {
        float v[kGradRows];
        contour_rows(mid, m, half_inv, v);
#pragma unroll
        for (int i = 0; i < kGradRows; ++i) {
            if (grad_own(x, W) && y0 + i < H) out[(long long)(y0 + i) * W + x] = v[i];
        }
        t += gridDim.x * kGradWaves;
        if (t >= items) break;
        grad_item(t, wx, x, y0);
        grad_load(lab, W, H, x, y0, mid);
    }
}

__global__ __launch_bounds__(kGradWG) void k_prepare_gradient(const float* __restrict__ lab, int W,
                                                          int H, int wx, int items, float sigma,
                                                          const unsigned long long* __restrict__ mx,
                                                          int n, float4* __restrict__ packed) {
    __shared__ unsigned long long red[kGradWaves];
    unsigned long long top = (int)threadIdx.x < n ? mx[threadIdx.x] : 0ULL;
    int t = grad_first(), x, y0;
    Texel mid[kGradRows + 2];
    grad_item(min(t, items - 1), wx, x, y0);
    grad_load(lab, W, H, x, y0, mid);
    top = block_max(top, red);
    const double m = sqrt(0.25 * __longlong_as_double((long long)top)), half_inv = 0.5 / m;
    const double s2 = (double)sigma * (double)sigma;
    while (t < items) {
        float v[kGradRows];
        contour_rows(mid, m, half_inv, v);
#pragma unroll
        for (int i = 0; i < kGradRows; ++i) {
            if (!grad_own(x, W) || y0 + i >= H) continue;
            const double c = (double)v[i];
            const float w = (float)(1.0 - exp(-(c * c) / s2));
            const Texel q = mid[i + 1];
            packed[(long long)(y0 + i) * W + x] = make_float4(q.c[0], q.c[1], q.c[2], w);
        }
        t += gridDim.x * kGradWaves;
        if (t >= items) break;
        grad_item(t, wx, x, y0);
        grad_load(lab, W, H, x, y0, mid);
    }
}

struct GradGrid {
    int wx, items;      // wave items along a row, in all
    unsigned maxima;    // blocks of k_gradient_max
    unsigned blocks;    // blocks of the second pass
};

// W H < 2^31, so there are at most 2^29 items.
GradGrid grad_grid(int W, int H) {
    GradGrid g;
    g.wx = (W + kGradCols - 1) / kGradCols;
    g.items = g.wx * ((H + kGradRows - 1) / kGradRows);
    const int blocks = (g.items + kGradWaves - 1) / kGradWaves;
    g.maxima = (unsigned)std::min(blocks, kGradSlots);
    g.blocks = (unsigned)std::min(blocks, 65536);
    return g;
}

// About 2048 blocks of 256 threads: whole rows, the row stride set by the grid height.
dim3 grid_for(int W, int H) {
    const int bx = (W + 255) / 256;
    const int by = std::max(1, std::min(H, std::max(1, 2048 / bx)));
    return dim3((unsigned)bx, (unsigned)std::min(by, 65535));
}

}  // namespace

int launch_boundary_frequency(int W, int H, int n, const int* labels, float* out, hipStream_t s) {
    hipLaunchKernelGGL(k_boundary_frequency, grid_for(W, H), dim3(256), 0, s, W, H, n, labels, out);
    return hipGetLastError();
}

int launch_contour_from_lab(int W, int H, const float* lab, float* out, void* ws, hipStream_t s) {
    unsigned long long* mx = static_cast<unsigned long long*>(ws);
    const GradGrid g = grad_grid(W, H);
    hipLaunchKernelGGL(k_gradient_max, dim3(g.maxima), dim3(kGradWG), 0, s, lab, W, H, g.wx,
                       g.items, mx);
    hipLaunchKernelGGL(k_gradient_normalise, dim3(g.blocks), dim3(kGradWG), 0, s, lab, W, H, g.wx,
                       g.items, mx, (int)g.maxima, out);
    return hipGetLastError();
}

int launch_prepare_gradient(int W, int H, const float* lab, float sigma, float4* packed,
                            unsigned long long* mx, hipStream_t s) {
    const GradGrid g = grad_grid(W, H);
    hipLaunchKernelGGL(k_gradient_max, dim3(g.maxima), dim3(kGradWG), 0, s, lab, W, H, g.wx,
                       g.items, mx);
    hipLaunchKernelGGL(k_prepare_gradient, dim3(g.blocks), dim3(kGradWG), 0, s, lab, W, H, g.wx,
                       g.items, sigma, mx, (int)g.maxima, packed);
    return hipGetLastError();
}

}  // namespace scalp
