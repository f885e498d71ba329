// scalp_soft.hip -- soft (differentiable) SCALP on gfx950.
//
// An extension of the paper's method: the distance D of Eqs. (1)-(3) over the
// same 3x3 grid-neighbour candidates as Algorithm 1, a softmax with
// temperature T over the candidates instead of the argmin, and soft
// barycenters instead of the hard update.  Paths go to the rounded
// barycenter floor(X_k + 0.5) (no Eq. (4) projection, which needs hard
// membership); the rounding is piecewise constant, so it carries no gradient.
//
// Forward, per iteration:
//   k_soft_assign  workgroup per (image, cell, slice), one pixel per lane:
//                  the candidate with the smallest bound of D is walked first,
//                  then, by full waves, those whose softmax weight that bound
//                  does not prove to be 0; then the FP64 softmax of -D/T over
//                  the 9 slots.  Writes Q, the factors A (Eq. (1)) and B
//                  (Eq. (2)) of the walked slots, and which Q are not 0.
//   k_soft_tables  the same where most slots are walked (see soft_tables): over an
//                  LDS table per candidate.
//   k_soft_update  workgroup per (image, superpixel): gathers the Q that are not
//                  0 over the 3x3 cell block in a fixed order (FP64 partial
//                  sums, tree reduction): deterministic, no atomics.
// Backward, per iteration in reverse:
//   k_soft_bwd_update  workgroup per (image, cell, slice): soft-update and
//                      softmax backward of its pixels, and, per slot, the list
//                      of the (pixel, dL/dD) that are not 0.
//   k_soft_bwd_path    workgroup per (image, superpixel): re-walks the paths of
//                      the pixels listed under it (samples are recomputed,
//                      never stored), adding the path's two per-sample weights
//                      into LDS tiles; a fold over the tiles then forms dL/df
//                      and dL/dw (float atomics: not bit-reproducible) and the
//                      superpixel's centre gradient (FP64).
#include <algorithm>
#include <climits>

#include "scalp_device.h"

namespace scalp {
namespace {

using namespace dev;

struct SoftImg {
    int W, H, nx, ny, K, B;
    int spl;    // work items (slices) per cell of the assignment
    long long N;
    float spw, gamma, lambda, inv_t;
    double temp;
    int prune;   // 1: skip the walks of slots whose softmax weight is provably 0
    int near;    // 32-bit byte offsets reach every texel of an image
    int bspl;    // slices of a cell in the backward's lists
    double inv_w;      // 1 / W
    FastDiv dper[2];   // 8 x the two cell heights (see PixelMap)
};

// A superpixel whose soft mass is below a millionth of a pixel counts as
// empty and keeps its centre (as an empty one does in the hard update).
constexpr double kZMin = 1e-6;

// Softmax weight below which a slot's path terms are left out of the backward.
constexpr float kQMin = 0x1p-24f;

// ------------------------------------------------------------------ forward

template <int WG>
__global__ __launch_bounds__(WG) void k_soft_init(SoftImg s, const float4* __restrict__ packed,
                                                  float* __restrict__ theta0) {
    __shared__ double red[6][WG];
    const int tid = threadIdx.x;
    const int b = blockIdx.x / s.K, k = blockIdx.x - b * s.K;
    const int ci = k / s.nx, cj = k - ci * s.nx;
    const int x0 = cell_lo(cj, s.W, s.nx), x1 = cell_lo(cj + 1, s.W, s.nx);
    const int y0 = cell_lo(ci, s.H, s.ny), y1 = cell_lo(ci + 1, s.H, s.ny);
    const float4* img = packed + (long long)b * s.N;
    const int cw = x1 - x0, P = cw * (y1 - y0);
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int t = tid; t < P; t += WG) {
        const int r = t / cw;
        const int x = x0 + (t - r * cw), y = y0 + r;
        const float4 f = img[(long long)y * s.W + x];
        acc[0] += f.x; acc[1] += f.y; acc[2] += f.z; acc[3] += x; acc[4] += y; acc[5] += 1.0;
    }
    for (int v = 0; v < 6; ++v) red[v][tid] = acc[v];
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if (tid < h)
            for (int v = 0; v < 6; ++v) red[v][tid] += red[v][tid + h];
        __syncthreads();
    }
    if (tid < 5) theta0[(5LL * b) * s.K + 5LL * k + tid] = (float)(red[tid][0] / red[5][0]);
}

// Per work item, by pixel (lane of the first pass): D per slot, then Q; the
// coordinates; the (pixel, slot) pairs of the second pass; the first D, and
// the pixels with more than one walk.
template <int WG>
struct SoftItem {
    float D[9][WG];
    int2 xy[WG];
    unsigned short list[8 * WG];
    float best[WG];
    unsigned short multi[WG];
    int pairs, multis;
};

// Q_pj = softmax_j(-D_pj / T) in FP64, rounded once to FP32 (the FP32 distances differ
// by far more than FP32's exponent range allows at small T).  A slot with (D - Dmin) /
// T > 110 has exp < 2^-158: added to the sum (at least 1, the minimum's term) it
// changes nothing in FP64, and its Q rounds to 0 in FP32, so neither the exponential
// nor the quotient is computed (same results, most slots at low T).
__device__ __forceinline__ void softmax(float (&v)[9], double temp) {
    float dmin = INFINITY;
#pragma unroll
    for (int j = 0; j < 9; ++j) dmin = fminf(dmin, v[j]);
    double e[9], sum = 0.0;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        e[j] = 0.0;
        if (v[j] < INFINITY) {
            const double t = ((double)v[j] - (double)dmin) / temp;
            if (t <= 110.0) e[j] = exp(-t);
        }
        sum += e[j];
    }
#pragma unroll
    for (int j = 0; j < 9; ++j) v[j] = e[j] == 0.0 ? 0.0f : (float)(e[j] / sum);
}

// What a slot's bound must exceed to prove that its Q is 0, where the pixel has a
// candidate with D = best (see k_soft_assign).
__device__ __forceinline__ float soft_limit(float best, double temp) {
    return fmaxf((best + 111.0f * (float)temp) * (1.0f + 0x1p-15f), 0x1p-70f);
}

// A work item: pixels [t0, t1) of a cell of image b.
struct SoftCell {
    int b, ci, cj, x0, y0, cw, ch, t0, t1;
};

__device__ __forceinline__ SoftCell soft_cell(const SoftImg& s, int item) {
    SoftCell c;
    const int bc = item / s.spl, slice = item - bc * s.spl;
    c.b = bc / s.K;
    const int cell = bc - c.b * s.K;
    c.ci = cell / s.nx;
    c.cj = cell - c.ci * s.nx;
    c.x0 = cell_lo(c.cj, s.W, s.nx);
    c.y0 = cell_lo(c.ci, s.H, s.ny);
    c.cw = cell_lo(c.cj + 1, s.W, s.nx) - c.x0;
    c.ch = cell_lo(c.ci + 1, s.H, s.ny) - c.y0;
    const int P = c.cw * c.ch, chunks = (P + 63) >> 6;
    c.t0 = 64 * (int)((long long)chunks * slice / s.spl);
    c.t1 = min(P, 64 * (int)((long long)chunks * (slice + 1) / s.spl));
    return c;
}

template <bool NEAR>
__device__ __forceinline__ Eqs soft_eqs(const SoftImg& s, const SoftCell& c, const Neighbours& nb,
                                        const float4* __restrict__ img,
                                        const float* __restrict__ cen) {
    Eqs eqs;
    eqs.img = img;
    eqs.W = s.W;
    near_all(eqs);
    if (!NEAR) {
        Box box = {c.x0, c.y0, c.x0 + c.cw - 1, c.y0 + c.ch - 1};
        for (int j = 0; j < 9; ++j) {
            const ConstF k = (ConstF)(uintptr_t)cen + 5LL * (nb.row[j / 3] + nb.col[j % 3]);
            box.add(round_coord(k[3], s.W - 1), round_coord(k[4], s.H - 1));
        }
        near_box(eqs, box);
    }
    eqs.lambda = s.lambda;
    eqs.oml = 1.0f - s.lambda;
    eqs.gamma = s.gamma;
    eqs.spw = s.spw;
    return eqs;
}

// One workgroup per (image, cell, slice) work item, one pixel per lane, in two
// passes of walks as in the hard assignment (process_cell), and the softmax.
// The softmax gives a slot Q = 0 exactly when (D - Dmin) / T > 110 in FP64.
// With best the D of the candidate walked first, Dmin <= best, so a slot whose
// bound exceeds (best + 111 T) (1 + 2^-15) gets Q = 0 whatever its walk would
// give (the margins cover the bound's rounding and the FP64 division's); such
// a slot, and a walk whose partial sums exceed that, counts as D = +inf.  Its
// saved factors are not written: the backward reads them only where dL/dD, a
// multiple of Q, is not 0.
//
// The pixels that walked one candidate have one Q, 1; the others are listed
// and take the FP64 softmax by full waves.
//
// What bounds it: VALU issue, as in the hard assignment.  A softmax pass of its
// own (it read D and wrote Q back) took 64 us per iteration of 16 x 512x512.
// The update's sums could be taken here too, as FP64 matrix products of the Q
// and the features of each wave's pixels, but in another order than the
// gather's, and one centre in 10^5 then rounds to the other FP32 neighbour.
template <int WG, bool NEAR>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(8))) void k_soft_assign(
    SoftImg s, const float4* __restrict__ packed, const float* __restrict__ theta_prev,
    float* __restrict__ q, float* __restrict__ fa, float* __restrict__ fb,
    unsigned short* __restrict__ pmask) {
    __shared__ SoftItem<WG> sh;
    const SoftCell it = soft_cell(s, xcd_remap(blockIdx.x, gridDim.x));
    if (it.t1 <= it.t0) return;                                 // uniform: an empty slice
    const int tid = threadIdx.x, b = it.b, ci = it.ci, cj = it.cj;
    const int W = s.W, H = s.H;
    const float4* __restrict__ img = packed + (long long)b * s.N;
    const float* __restrict__ cen = theta_prev + 5LL * s.K * b;
    const Neighbours nb = neighbours_of(s.nx, s.ny, ci, cj);
    const Eqs eqs = soft_eqs<NEAR>(s, it, nb, img, cen);
    const int k0 = (ci - 1) * s.nx + cj - 1;
    const long long base = 9LL * s.N * b;
    // D of pixel (px, py) with texel fp to slot j, its factors saved unless the
    // walk was cut
    auto distance = [&](int j, float4 fp, int px, int py, bool cut, float thr) -> float {
        const int di = (j * 11) >> 5;                           // j / 3 for j <= 8
        const float* cp = cen + 5 * (k0 + di * s.nx + (j - 3 * di));
        const float ck[5] = {cp[0], cp[1], cp[2], cp[3], cp[4]};
        float A, B;
        const float D = path_distance(eqs, ck, fp, round_coord(ck[3], W - 1),
                                      round_coord(ck[4], H - 1), px, py, cut, thr, A, B);
        if (D < INFINITY) {
            const long long o = base + (long long)j * s.N + (long long)py * W + px;
            fa[o] = A;
            fb[o] = B;
        }
        return D;
    };
    auto limit = [&](float best) { return soft_limit(best, s.temp); };
    if (tid == 0) sh.pairs = sh.multis = 0;
    __syncthreads();
    const bool prune = s.prune != 0;
    const bool mine = tid < it.t1 - it.t0;
    int px = 0, py = 0, first = 9;
    float D = INFINITY;
    bool again = false;
    if (mine) {
        pixel_at(pixel_map(s.dper, it.cw, it.ch), it.t0 + tid, px, py);
        px += it.x0;
        py += it.y0;
        unsigned key[9];
        const float4 fp = img[py * W + px];
        bound_keys(nb, (ConstF)(uintptr_t)cen, s.spw, fp, px, py, s.lambda, key);
        unsigned nk = next_key(key, kNoKey);
        first = (int)(nk & 15u);
        D = distance(first, fp, px, py, false, 0.0f);
        const float best = D < INFINITY ? D : INFINITY;         // NaN: nothing is known
        const float thr = limit(best);
        for (;;) {
            nk = next_key(key, nk);
            const bool more = nk != kNoKey && !(prune && key_bound(nk) > thr);
            const unsigned long long m = __ballot(more);
            if (m == 0ULL) break;                               // uniform over the lanes still here
            const int at = wave_claim(&sh.pairs, m);
            if (!more) break;
            sh.list[at] = (unsigned short)(tid | ((nk & 15u) << 10));
            again = true;
        }
        const unsigned long long m = __ballot(again);
        if (m != 0ULL) {
            const int at = wave_claim(&sh.multis, m);
            if (again) {
                sh.multi[at] = (unsigned short)tid;
                sh.best[tid] = best;
            }
        }
    }
    // the D walked so far; or Q, where there is one walk only
    const float rest = again ? INFINITY : 0.0f;
    const float one = again ? D : (D < INFINITY ? 1.0f : 0.0f);
#pragma unroll
    for (int j = 0; j < 9; ++j) sh.D[j][tid] = j == first ? one : rest;
    sh.xy[tid] = make_int2(px, py);
    __syncthreads();
    const int pairs = __builtin_amdgcn_readfirstlane(sh.pairs);
    const bool cut = prune && s.gamma <= 0x1p40f;
    for (int i = tid; i < pairs; i += WG) {
        const unsigned e = sh.list[i];
        const int id = (int)(e & 1023u), j = (int)(e >> 10);
        const int2 xy = sh.xy[id];
        sh.D[j][id] = distance(j, img[xy.y * W + xy.x], xy.x, xy.y, cut, limit(sh.best[id]));
    }
    __syncthreads();
    if (tid < sh.multis) {
        const int id = (int)sh.multi[tid];
        float v[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) v[j] = sh.D[j][id];
        softmax(v, s.temp);
#pragma unroll
        for (int j = 0; j < 9; ++j) sh.D[j][id] = v[j];
    }
    __syncthreads();
    if (mine) {
        unsigned mask = 0;
        const long long o = base + (long long)py * W + px;
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const float Q = sh.D[j][tid];
            q[o + (long long)j * s.N] = Q;
            mask |= Q != 0.0f ? 1u << j : 0u;
        }
        pmask[(long long)b * s.N + (long long)py * W + px] = (unsigned short)mask;
    }
}

// Per work item of k_soft_tables: D by slot and pixel, and a candidate's table or two
// of half the size; 72 bytes a lane in all (see TableShared).
template <int WG>
struct SoftTables {
    static constexpr int kEntries = (9 * WG - 8) / 2;
    float D[9][WG];
    float2 table[kEntries];
    int box[4];
};

// The same results as k_soft_assign where most pixels walk most candidates (see
// soft_tables): candidate by candidate, own cell first, then edges, then corners, over
// LDS tables as in the hard form's assign_all, one pixel per lane; a candidate
// whose bound proves that its Q is 0 is left out.
//
// What bounds it: VALU issue.
template <int WG, bool NEAR>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(8))) void k_soft_tables(
    SoftImg s, const float4* __restrict__ packed, const float* __restrict__ theta_prev,
    float* __restrict__ q, float* __restrict__ fa, float* __restrict__ fb,
    unsigned short* __restrict__ pmask) {
    __shared__ SoftTables<WG> sh;
    const SoftCell it = soft_cell(s, xcd_remap(blockIdx.x, gridDim.x));
    if (it.t1 <= it.t0) return;                                 // uniform: an empty slice
    const int tid = threadIdx.x;
    const int W = s.W, H = s.H;
    const float4* __restrict__ img = packed + (long long)it.b * s.N;
    const float* __restrict__ cen = theta_prev + 5LL * s.K * it.b;
    const Neighbours nb = neighbours_of(s.nx, s.ny, it.ci, it.cj);
    const Eqs eqs = soft_eqs<NEAR>(s, it, nb, img, cen);
    if (tid == 0) {
        sh.box[0] = sh.box[1] = INT_MAX;
        sh.box[2] = sh.box[3] = 0;
    }
    __syncthreads();
    const bool mine = tid < it.t1 - it.t0;
    int px = INT_MAX, py = INT_MAX;
    if (mine) {
        pixel_at(pixel_map(s.dper, it.cw, it.ch), it.t0 + tid, px, py);
        px += it.x0;
        py += it.y0;
    }
    {
        const int lx = wave_min_i32(px), ly = wave_min_i32(py);
        const int hx = wave_max_i32(mine ? px : 0), hy = wave_max_i32(mine ? py : 0);
        if ((tid & 63) == 0) {
            atomicMin(&sh.box[0], lx);
            atomicMin(&sh.box[1], ly);
            atomicMax(&sh.box[2], hx);
            atomicMax(&sh.box[3], hy);
        }
    }
#pragma unroll
    for (int j = 0; j < 9; ++j) sh.D[j][tid] = INFINITY;
    __syncthreads();
    const Box own = {__builtin_amdgcn_readfirstlane(sh.box[0]), __builtin_amdgcn_readfirstlane(sh.box[1]),
                     __builtin_amdgcn_readfirstlane(sh.box[2]), __builtin_amdgcn_readfirstlane(sh.box[3])};
    const long long o = 9LL * s.N * it.b + (long long)py * W + px;
    const int k0 = (it.ci - 1) * s.nx + it.cj - 1;
    const bool prune = s.prune != 0, cut = prune && s.gamma <= 0x1p40f;
    float best = INFINITY;
    bool half = false, was_full = false;                        // uniform
#pragma unroll 1
    for (int i = 0; i < 9; ++i) {
        const int j = (int)((0x862075314ULL >> (4 * i)) & 15ULL);   // 4, 1, 3, 5, 7, 0, 2, 6, 8
        if (!((nb.inside >> j) & 1u)) continue;                 // uniform
        const int di = (j * 11) >> 5;
        const ConstF cp = (ConstF)(uintptr_t)cen + 5 * (k0 + di * s.nx + (j - 3 * di));
        const float ck[5] = {cp[0], cp[1], cp[2], cp[3], cp[4]};
        const int cx = __builtin_amdgcn_readfirstlane(round_coord(ck[3], W - 1));
        const int cy = __builtin_amdgcn_readfirstlane(round_coord(ck[4], H - 1));
        Box box = own;
        box.add(cx, cy);
        const Table t = table_of(box, SoftTables<WG>::kEntries, WG);
        if (t.fits) {
            const bool full = t.pitch * t.rows > SoftTables<WG>::kEntries / 2;
            if (full || was_full) __syncthreads();              // the table before was read
            half = !half && !full;
            was_full = full;
        }
        float2* table = sh.table + (half ? SoftTables<WG>::kEntries / 2 : 0);
        if (t.fits) {
            fill_table<WG>(table, t, img, W, ck[0], ck[1], ck[2]);
            __syncthreads();
        }
        if (!mine) continue;
        float4 fp = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float dcp;
        if (t.fits) {                                           // uniform
            dcp = table[(py - t.y0) * t.pitch + (px - t.x0)].x;
        } else {
            fp = img[py * W + px];
            dcp = colour_dist(fp, ck[0], ck[1], ck[2]);
        }
        const float ax = (float)px - ck[3], ay = (float)py - ck[4];
        const float lb = s.lambda * dcp + (ax * ax + ay * ay) * s.spw;   // <= D
        if (prune && lb > soft_limit(best, s.temp)) continue;
        float A, B;
        const float D = t.fits ? table_distance(eqs, ck, t, table, cx, cy, px, py, A, B)
                               : path_distance(eqs, ck, fp, cx, cy, px, py, cut,
                                               soft_limit(best, s.temp), A, B);
        if (D < INFINITY) {
            sh.D[j][tid] = D;
            fa[o + (long long)j * s.N] = A;
            fb[o + (long long)j * s.N] = B;
            best = fminf(best, D);
        }
    }
    if (mine) {
        float v[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) v[j] = sh.D[j][tid];
        softmax(v, s.temp);
        unsigned mask = 0;
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            q[o + (long long)j * s.N] = v[j];
            mask |= v[j] != 0.0f ? 1u << j : 0u;
        }
        pmask[(long long)it.b * s.N + (long long)py * W + px] = (unsigned short)mask;
    }
}

// Per-pixel soft kernels run a 3D grid: image in z, rows strided over y,
// 256-column segments in x (no per-pixel division to recover coordinates).
#define SOFT_FOR_PIXELS(s)                                                   \
    const int b = blockIdx.z;                                                \
    const int x = blockIdx.x * 256 + threadIdx.x;                            \
    for (int y = blockIdx.y; y < (s).H; y += gridDim.y)                      \
        if (x < (s).W)

template <int WG>
__device__ __forceinline__ void block_sum6(double (&v)[6], double (*red)[WG]) {
    const int tid = threadIdx.x;
    for (int i = 0; i < 6; ++i) red[i][tid] = v[i];
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if (tid < h)
            for (int i = 0; i < 6; ++i) red[i][tid] += red[i][tid + h];
        __syncthreads();
    }
    for (int i = 0; i < 6; ++i) v[i] = red[i][0];
}

// Soft update of superpixel k: Z = sum Q, f_k = sum Q f / Z, X_k = sum Q X / Z
// over the pixels of the 3x3 cell block around k, each read through the slot
// under which it sees k.
template <int WG>
__global__ __launch_bounds__(WG) void k_soft_update(SoftImg s, const float* __restrict__ q,
                                                    const unsigned short* __restrict__ pmask,
                                                    const float4* __restrict__ packed,
                                                    const float* __restrict__ theta_prev,
                                                    float* __restrict__ theta_next,
                                                    double* __restrict__ z) {
    __shared__ double red[6][WG];
    const int tid = threadIdx.x;
    const int b = blockIdx.x / s.K, k = blockIdx.x - b * s.K;
    const int ci = k / s.nx, cj = k - ci * s.nx;
    const int X0 = cell_lo(max(cj - 1, 0), s.W, s.nx), X1 = cell_lo(min(cj + 2, s.nx), s.W, s.nx);
    const int Y0 = cell_lo(max(ci - 1, 0), s.H, s.ny), Y1 = cell_lo(min(ci + 2, s.ny), s.H, s.ny);
    const int bw = X1 - X0, area = bw * (Y1 - Y0);
    const float4* img = packed + (long long)b * s.N;
    const float* qb = q + 9LL * s.N * b;
    const unsigned short* pm = pmask + (long long)b * s.N;
    // the block's inner cell boundaries: a pixel's cell row is ci - 1 + (y >= yb1)
    // + (y >= yb2), likewise for columns
    const int yb1 = cell_lo(ci, s.H, s.ny), yb2 = cell_lo(ci + 1, s.H, s.ny);
    const int xb1 = cell_lo(cj, s.W, s.nx), xb2 = cell_lo(cj + 1, s.W, s.nx);
    double acc[6] = {0, 0, 0, 0, 0, 0};
    // element e = r * bw + c; lanes step by WG elements = (dr rows, dc columns)
    const int dr = WG / bw, dc = WG - dr * bw;
    int r = tid / bw, c = tid - r * bw;
    // kU elements per trip (e, e + WG, ...), their masks loaded first; a Q is
    // read only where its mask says that it is not 0 (at low T one slot in
    // eight; 0 * f adds exactly nothing), and a texel only with it
    constexpr int kU = 8;
    for (int e = tid; e < area; e += kU * WG) {
        int xs[kU], ys[kU], js[kU];
        unsigned ms[kU];
        float Qs[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            xs[u] = X0 + c;
            ys[u] = Y0 + r;
            c += dc;
            const bool wrap = c >= bw;
            c -= wrap ? bw : 0;
            r += dr + (wrap ? 1 : 0);
            const int di = (ys[u] >= yb1 ? 1 : 0) + (ys[u] >= yb2 ? 1 : 0);
            const int dj = (xs[u] >= xb1 ? 1 : 0) + (xs[u] >= xb2 ? 1 : 0);
            js[u] = (2 - di) * 3 + (2 - dj);        // the pixel's slot that points at k
            ms[u] = e + u * WG < area ? pm[ys[u] * s.W + xs[u]] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            Qs[u] = (ms[u] >> js[u]) & 1u
                        ? qb[(long long)js[u] * s.N + (ys[u] * s.W + xs[u])] : 0.0f;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (Qs[u] == 0.0f) continue;
            const double Q = (double)Qs[u];
            const float4 f = img[ys[u] * s.W + xs[u]];
            acc[0] += Q;
            acc[1] += Q * f.x;
            acc[2] += Q * f.y;
            acc[3] += Q * f.z;
            acc[4] += Q * xs[u];
            acc[5] += Q * ys[u];
        }
    }
    block_sum6<WG>(acc, red);
    if (tid < 5) {
        const long long o = 5LL * s.K * b + 5LL * k + tid;
        theta_next[o] = acc[0] >= kZMin ? (float)(acc[tid + 1] / acc[0]) : theta_prev[o];
    }
    if (tid == 0) z[(long long)s.K * b + k] = acc[0];
}

// ------------------------------------------------------------------ backward

// Per superpixel, what the soft-update backward needs of it, in two float4:
// u = dL/dTheta_k / Z_k (5 values) and v = u . Theta_k, all zero when Z_k is
// below kZMin (such a superpixel kept its centre and passes no gradient to
// Q or f).
__device__ __forceinline__ void store_cand(double Z, const double (&g)[5],
                                           const float* __restrict__ theta,
                                           float4* __restrict__ cand) {
    float u[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    float v = 0.0f;
    if (Z >= kZMin) {
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            u[c] = (float)(g[c] / Z);
            v += u[c] * theta[c];
        }
    }
    cand[0] = make_float4(u[0], u[1], u[2], u[3]);
    cand[1] = make_float4(u[4], v, 0.0f, 0.0f);
}

// dL/dTheta_T from the caller, in FP64, and the terms of the first update.
__global__ void k_soft_bwd_start(SoftImg s, const float* __restrict__ grad_theta,
                                 const double* __restrict__ z, const float* __restrict__ theta,
                                 double* __restrict__ gth, float4* __restrict__ cand) {
    const long long total = (long long)s.B * s.K;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        double g[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            g[c] = (double)grad_theta[5 * i + c];
            gth[5 * i + c] = g[c];
        }
        store_cand(z[i], g, theta + 5 * i, cand + 2 * i);
    }
}

// Pixels [t0, t1) of slice `slice` of a cell of P pixels in the backward's
// lists, in whole 64-pixel chunks.
__device__ __forceinline__ void bwd_slice(const SoftImg& s, int P, int slice, int& t0, int& t1) {
    const int chunks = (P + 63) >> 6;
    t0 = 64 * (int)((long long)chunks * slice / s.bspl);
    t1 = min(P, 64 * (int)((long long)chunks * (slice + 1) / s.bspl));
}

constexpr int kUpdateWG = 256;

// Soft-update backward (theta_t = sum Q feat / Z) and softmax backward of the
// pixels of a slice of a cell: dL/dD_pj (0 where Q_pj < kQMin), and gf +=
// dL/df_p through the update.  With u, v of store_cand: dL/dQ_pk += u . feat_p
// - v and dL/df_p += Q_pk u[0..2].  The cell's 9 candidates are uniform, so
// their u, v come through the scalar cache.  The dL/dD that are not 0 (one
// pixel in ten at low T) are listed per slot as (pixel, value), in no
// particular order, from entry 9 N b + j N + (pixels of the cells before, in
// cell order) + t0 on, and counted: the path pass finds what it walks without
// a search.  first: gf is written, not added to.
__global__ __launch_bounds__(kUpdateWG) void k_soft_bwd_update(
    SoftImg s, int first, const float* __restrict__ q, const unsigned short* __restrict__ pmask,
    const float4* __restrict__ cand, const float4* __restrict__ packed,
    const float* __restrict__ gq_in, uint2* __restrict__ pairs, int* __restrict__ count,
    float4* __restrict__ gf) {
    __shared__ int cnt[9];
    const int tid = threadIdx.x;
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const int bc = item / s.bspl, slice = item - bc * s.bspl;
    const int b = bc / s.K, cell = bc - b * s.K;
    const int W = s.W, H = s.H;
    const int ci = cell / s.nx, cj = cell - ci * s.nx;
    const int x0 = cell_lo(cj, W, s.nx), cw = cell_lo(cj + 1, W, s.nx) - x0;
    const int y0 = cell_lo(ci, H, s.ny), ch = cell_lo(ci + 1, H, s.ny) - y0;
    int t0, t1;
    bwd_slice(s, cw * ch, slice, t0, t1);
    if (tid < 9) cnt[tid] = 0;
    __syncthreads();
    const Neighbours nb = neighbours_of(s.nx, s.ny, ci, cj);
    const ConstF cb = (ConstF)(uintptr_t)(cand + 2LL * s.K * b);
    const PixelMap pm = pixel_map(s.dper, cw, ch);
    const long long base = 9LL * s.N * b;
    uint2* __restrict__ list = pairs + base + ((long long)y0 * W + (long long)x0 * ch + t0);
    for (int t = t0; t < t1; t += kUpdateWG) {                  // uniform
        const bool mine = t + tid < t1;
        int x = 0, y = 0;
        if (mine) {
            pixel_at(pm, t + tid, x, y);
            x += x0;
            y += y0;
        }
        const int p = y * W + x;
        const long long i = (long long)b * s.N + p;
        // a slot with Q_pj = 0 adds nothing to the softmax dot product, to
        // dL/df or to dL/dD (Q_pj < 2^-24): its Q, its dL/dQ and its
        // candidate's terms are not read
        const unsigned nz = mine ? pmask[i] : 0u;
        float Q[9], G[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            Q[j] = G[j] = 0.0f;
            if ((nz >> j) & 1u) {
                Q[j] = q[base + (long long)j * s.N + p];
                if (first) G[j] = gq_in[base + (long long)j * s.N + p];
            }
        }
        const float4 f = mine ? packed[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const float fx = (float)x, fy = (float)y;
        float gfl = 0.0f, gfa = 0.0f, gfb = 0.0f, dot = 0.0f;
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            if (__ballot((nz >> j) & 1u) == 0ULL) continue;     // uniform over the wave
            const ConstF u = cb + 8LL * __builtin_amdgcn_readfirstlane(nb.row[j / 3] + nb.col[j % 3]);
            const float u0 = u[0], u1 = u[1], u2 = u[2], u3 = u[3], u4 = u[4], v = u[5];
            if ((nz >> j) & 1u) {
                G[j] += (((u0 * f.x + u1 * f.y) + (u2 * f.z + u3 * fx)) + u4 * fy) - v;
                gfl += u0 * Q[j];
                gfa += u1 * Q[j];
                gfb += u2 * Q[j];
                dot += Q[j] * G[j];
            }
        }
        // A slot's whole path contribution is proportional to Q_pj; below
        // FP32's unit roundoff (2^-24) it is dropped, and the path pass skips
        // the slot (at low T most pixels have one slot above it).
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            const float g = Q[j] < kQMin ? 0.0f : -s.inv_t * Q[j] * (G[j] - dot);
            const unsigned long long m = __ballot(g != 0.0f);
            if (m == 0ULL) continue;                            // uniform over the wave
            const int at = wave_claim(&cnt[j], m);
            if (g != 0.0f)
                list[(long long)j * s.N + at] = make_uint2((unsigned)p, __float_as_uint(g));
        }
        if (mine) {
            float4 o = first ? make_float4(0.0f, 0.0f, 0.0f, 0.0f) : gf[i];
            o.x += gfl;
            o.y += gfa;
            o.z += gfb;
            gf[i] = o;
        }
    }
    __syncthreads();
    if (tid < 9) count[9LL * item + tid] = cnt[tid];
}

// Workgroup of the path pass: 256 lanes, or 512 where there are at most 2 kCUs
// superpixels in all (2 x 97x61, T = 5: 16.9 instead of 20.1 us per iteration; 2 x 256x256, k =
// 128, T = 5: 78 instead of 90; 512x512, k = 400, T = 5: 122 instead of 135, and no
// difference at T = 0.5).
constexpr int kPathWG = 256, kPathWideWG = 512;
// Most lists (9 cells x slices) of a superpixel.
constexpr int kBwdLists = 252;
// Texels per thread and trip of the fold, their loads in flight together.
constexpr int kFold = 4;
// Fewest pairs of a run of lists that pay for a tile of their own.
constexpr int kTilePairs = 128;

// One workgroup per (image, superpixel k): every pixel whose dL/dD of the slot
// that points at k is not zero (listed by k_soft_bwd_update under the 9 cells
// around k) re-walks its path.  Along a path to k every sample q receives the
// same two weights,
//   dL/df_q += cf (f_q - f_k)   with cf = dL/dD * B (1 - lambda) 2 / |P|
//   dL/dw_q += cw               with cw = dL/dD * A gamma / |P|
// (and p itself dL/dD * B lambda 2 (f_p - f_k)), so the walk only adds cf into
// an FP64 tile S(q) (p's lambda term included) and cw into an FP32 tile of
// dL/dw, over a box that holds the pixels and k's endpoint: two LDS atomics per
// sample and no texel read.  A fold over the box then forms, per texel,
// dL/df_q = S(q) (f_q - f_k) from one texel load, and k's centre gradient,
// -sum_q S(q) (f_q - f_k), in FP64.  The spatial part of the centre gradient
// and the endpoint's weights (every path ends there) are summed per lane.
//
// Pairs whose box exceeds the tile are taken by fewer lists at a time, and a list by
// halves (it is in the order of the cell's chunks) down to 64.  LARGE, for cells so
// large that those seldom fit: runs of lists take a tile each, folded once however
// many pairs it takes, as long as the box of their slices of cells fits and they have
// pairs enough to pay for it; the lists left share one.  What does not fit either way
// takes a tile around the endpoint, where the paths meet, and the samples before a path
// enters it are added to global memory one by one (paths only approach the endpoint,
// so they do not leave it again), as are all of a path too long for the
// carry-counting steps.  Every centre gradient is summed here, in FP64 (no FP32 partial
// sum longer than one path), and stored, with the terms that the update of the
// iteration before needs.
//
// What bounds it: the latency of a superpixel's chain of phases, with the tiles
// limiting a CU to 3 workgroups; the walks, the fold and its atomics take about
// a quarter of the time each.  16 x 512x512, k = 400, T = 0.5 (300 K to 400 K
// walked pairs, 47 to 64 per superpixel): 144 us per iteration, where a
// workgroup per cell with a tile for each of its 9 candidates and a fold over
// all of them took 298.  Atomics of one value of 64 texels instead of rows of
// 16 texels' four values: 235.  Workgroups of 128 or 512 threads: 175 and 221.
// Cells of 128x128 pixels (512x512, k = 16), 5 iterations at T = 0.5 and 5: 0.90 and
// 1.84 ms, 4.23 and 21.1 by halves alone.
template <int WG, bool LARGE>
__global__ __launch_bounds__(WG) void k_soft_bwd_path(
    SoftImg s, const float4* __restrict__ packed, const float* __restrict__ theta_prev,
    const float* __restrict__ fa, const float* __restrict__ fb, const uint2* __restrict__ pairs,
    const int* __restrict__ count, const double* __restrict__ z, const double* __restrict__ gth,
    const double* __restrict__ z_prev, double* __restrict__ gth_prev, float4* __restrict__ cand,
    float4* __restrict__ gf, int cap_bytes) {
    extern __shared__ double bwd_dyn[];
    constexpr int kWaves = WG / 64;
    __shared__ long long lbase[kBwdLists + 4];    // first entry of each list
    __shared__ int lpre[kBwdLists + 4];           // pairs in the lists before
    __shared__ unsigned char left[kBwdLists + 4]; // the list is one of those left
    __shared__ int wtot[kWaves];
    __shared__ int wbox[4][kWaves];
    __shared__ float4 turn[kWaves][64];
    __shared__ double red[5][kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = s.W, H = s.H;
    const int bk = xcd_remap(blockIdx.x, gridDim.x);
    const int b = bk / s.K, k = bk - b * s.K;
    const int ci = k / s.nx, cj = k - ci * s.nx;
    const float4* __restrict__ img = packed + (long long)b * s.N;
    float4* __restrict__ gimg = gf + (long long)b * s.N;
    const ConstF ck = (ConstF)(uintptr_t)(theta_prev + 5LL * bk);
    const float cl = ck[0], ca = ck[1], cb = ck[2], cxf = ck[3], cyf = ck[4];
    const int cx = round_coord(cxf, W - 1), cy = round_coord(cyf, H - 1);
    const long long base = 9LL * s.N * b;
    const int entries = cap_bytes / 12;
    // the lists of k: cell (ci + di, cj + dj), read under its slot (-di, -dj)
    const int lists = 9 * s.bspl;
    int n = 0;
    if (tid < lists) {
        const int nbr = tid / s.bspl, slice = tid - nbr * s.bspl;
        const int ii = ci + nbr / 3 - 1, jj = cj + nbr % 3 - 1;
        if (ii >= 0 && ii < s.ny && jj >= 0 && jj < s.nx) {
            const int x0 = cell_lo(jj, W, s.nx), cw = cell_lo(jj + 1, W, s.nx) - x0;
            const int y0 = cell_lo(ii, H, s.ny), ch = cell_lo(ii + 1, H, s.ny) - y0;
            int t0, t1;
            bwd_slice(s, cw * ch, slice, t0, t1);
            const long long item = ((long long)b * s.K + ii * s.nx + jj) * s.bspl + slice;
            n = count[9 * item + 8 - nbr];
            lbase[tid] = base + (long long)(8 - nbr) * s.N +
                         ((long long)y0 * W + (long long)x0 * ch + t0);
        }
    }
    // lpre from the lists' lengths: the number of pairs (all lanes call)
    auto scan = [&](int len) -> int {
        const int incl = wave_scan_incl(len);
        if (lane == 63) wtot[wave] = incl;
        __syncthreads();
        int total = 0;
        for (int v = 0; v < kWaves; ++v) {
            if (v == wave && tid <= lists) lpre[tid] = total + incl - len;
            total += wtot[v];
        }
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(total);
    };
    const int total = scan(n);
    // pair a: its pixel, dL/dD and the factors of its path
    struct Pair {
        int x, y;
        float g, A, B;
    };
    auto pair_at = [&](int a) {
        Pair q;
        int l = 0, h = lists - 1;                 // the last list that starts at or before it
        while (l < h) {
            const int m = (l + h + 1) >> 1;
            if (lpre[m] <= a) l = m; else h = m - 1;
        }
        const uint2 e = pairs[lbase[l] + (a - lpre[l])];
        const int p = (int)e.x;
        const long long o = base + (long long)(8 - l / s.bspl) * s.N + p;
        q.g = __uint_as_float(e.y);
        q.A = fa[o];
        q.B = fb[o];
        q.y = (int)((double)p * s.inv_w);
        q.x = p - q.y * W;
        if (q.x < 0) { --q.y; q.x += W; }
        if (q.x >= W) { ++q.y; q.x -= W; }
        return q;
    };
    // the box of list l's part of its cell (uniform)
    auto list_box = [&](int l) {
        const int nbr = l / s.bspl, slice = l - nbr * s.bspl;
        const int jj = cj + nbr % 3 - 1, ii = ci + nbr / 3 - 1;
        Box r;
        r.x0 = cell_lo(jj, W, s.nx);
        r.x1 = cell_lo(jj + 1, W, s.nx) - 1;
        r.y0 = cell_lo(ii, H, s.ny);
        r.y1 = cell_lo(ii + 1, H, s.ny) - 1;
        if (s.bspl > 1) {                         // its 8-column strips
            const int ch = r.y1 - r.y0 + 1;
            int t0, t1;
            bwd_slice(s, (r.x1 - r.x0 + 1) * ch, slice, t0, t1);
            r.x1 = min(r.x1, r.x0 + 8 * ((t1 - 1) / (8 * ch)) + 7);
            r.x0 += 8 * (t0 / (8 * ch));
        }
        return r;
    };
    auto fits = [&](const Box& r) {
        return (long long)(r.x1 - r.x0 + 1) * (r.y1 - r.y0 + 1) <= entries;
    };
    double gc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};     // this lane's share of dL/dTheta_k
    const float lambda = s.lambda, oml = 1.0f - lambda;
    // the most square box of a tile within `box` around the endpoint
    auto clip = [&](Box& box) {
        const int bw = box.x1 - box.x0 + 1, bh = box.y1 - box.y0 + 1;
        int w = min(bw, (int)sqrtf((float)entries));
        const int h = min(bh, entries / w);
        w = min(bw, entries / h);
        box.x0 = min(max(cx - w / 2, box.x0), box.x1 - w + 1);
        box.y0 = min(max(cy - h / 2, box.y0), box.y1 - h + 1);
        box.x1 = box.x0 + w - 1;
        box.y1 = box.y0 + h - 1;
    };
    const int own = lane * kWaves + wave;         // one pair per lane, spread over the waves
    int a0 = 0, a1 = min(total, WG);              // the pairs of a tile
    int next = 0, rest = 0;                       // LARGE: next list; pairs of the lists left
    bool last = false;
    while (LARGE ? !last : a0 < total) {          // uniform
        Box box = {cx, cy, cx, cy};
        Pair q = {cx, cy, 0.0f, 0.0f, 0.0f};
        if constexpr (!LARGE) {
            if (a0 + own < a1) q = pair_at(a0 + own);
            box.add(q.x, q.y);
            box = {wave_min_i32(box.x0), wave_min_i32(box.y0), wave_max_i32(box.x1),
                   wave_max_i32(box.y1)};
            if (lane == 0) {
                wbox[0][wave] = box.x0;
                wbox[1][wave] = box.y0;
                wbox[2][wave] = box.x1;
                wbox[3][wave] = box.y1;
            }
            __syncthreads();
            for (int v = 0; v < kWaves; ++v) {
                box.add(wbox[0][v], wbox[1][v]);
                box.add(wbox[2][v], wbox[3][v]);
            }
            box = {__builtin_amdgcn_readfirstlane(box.x0), __builtin_amdgcn_readfirstlane(box.y0),
                   __builtin_amdgcn_readfirstlane(box.x1), __builtin_amdgcn_readfirstlane(box.y1)};
            if (!fits(box)) {
                // fewer: the lists that end in the first half, or else the first
                // list, or else half of it
                const int len = a1 - a0;
                int first = a1, half = a0;
                for (int l = 0; l < lists; ++l) {
                    const int v = lpre[l];
                    if (v > a0) first = min(first, v);
                    if (v <= a0 + (len >> 1)) half = max(half, v);
                }
                const int fewer = __builtin_amdgcn_readfirstlane(
                    half > a0 ? half - a0 : first < a1 ? first - a0 : max(64, (len >> 1) & ~63));
                if (fewer < len) {                // uniform
                    a1 = a0 + fewer;
                    __syncthreads();              // wbox is written again
                    continue;
                }
                clip(box);
            }
        } else if (next < lists) {
            int l1 = next;
            a0 = a1 = __builtin_amdgcn_readfirstlane(lpre[next]);
            for (; l1 < lists; ++l1) {
                const int end = __builtin_amdgcn_readfirstlane(lpre[l1 + 1]);
                if (end == a1) continue;          // an empty list
                Box r = list_box(l1);
                r.add(box.x0, box.y0);
                r.add(box.x1, box.y1);
                if (!fits(r)) {
                    if (a1 > a0) break;
                    ++l1;                         // not even alone: left
                    a1 = end;
                    box.x1 = -1;
                    break;
                }
                box = r;
                a1 = end;
            }
            const bool taken = box.x1 >= 0 && a1 - a0 >= kTilePairs;
            if (tid >= next && tid < l1) left[tid] = taken ? 0 : 1;
            next = l1;
            if (!taken) {
                rest += a1 - a0;
                continue;
            }
        } else {
            if (rest == 0) break;
            __syncthreads();
            const bool mine = tid < lists && n > 0 && left[tid];
            a0 = 0;
            a1 = scan(mine ? n : 0);
            for (int l = 0; l < lists; ++l) {
                if (__builtin_amdgcn_readfirstlane(lpre[l + 1]) == __builtin_amdgcn_readfirstlane(lpre[l]))
                    continue;
                const Box r = list_box(l);
                box.add(r.x0, r.y0);
                box.add(r.x1, r.y1);
            }
            if (!fits(box)) clip(box);
            last = true;
        }
        const int mnx = box.x0, mny = box.y0;
        const int bw = box.x1 - mnx + 1, area = bw * (box.y1 - mny + 1);
        double* __restrict__ st = bwd_dyn;
        float* __restrict__ wt = reinterpret_cast<float*>(bwd_dyn + area);
        for (int e = tid; e < area; e += WG) {
            st[e] = 0.0;
            wt[e] = 0.0f;
        }
        __syncthreads();
        double vc = 0.0, vw = 0.0;                // the endpoint's weights
        // samples i = 0 .. n-1 of a pair's path (p itself first); the endpoint i = n is
        // added once
        auto walk = [&](const Pair& q) {
            int x = q.x, y = q.y;
            const int dx = cx - x, dy = cy - y;
            const int adx = dx < 0 ? -dx : dx, ady = dy < 0 ? -dy : dy;
            const int np = max(adx, ady);
            const float inv_np = 1.0f / (float)(np + 1);
            const float cf = 2.0f * q.g * q.B * oml * inv_np;  // per sample, times (f_q - f_k)
            const float cw_ = q.g * q.A * s.gamma * inv_np;    // per sample: dL/dw_q
            const float lf = 2.0f * q.g * q.B * lambda;        // lambda term of p
            gc[3] += (double)(-2.0f * q.g * s.spw * ((float)x - cxf));
            gc[4] += (double)(-2.0f * q.g * s.spw * ((float)y - cyf));
            const bool xmaj = adx >= ady;
            const int am = xmaj ? ady : adx;
            const double cfd = (double)cf;
            double first = cfd + (double)lf;
            int m = 0;
            int rem = np;
            while (m < np && (x < box.x0 || x > box.x1 || y < box.y0 || y > box.y1 || np >= 46340)) {
                const int g = y * W + x;
                const float4 fq = img[g];
                const double el = first * (double)(fq.x - cl), ea = first * (double)(fq.y - ca),
                             eb = first * (double)(fq.z - cb);
                unsafeAtomicAdd(&gimg[g].x, (float)el);
                unsafeAtomicAdd(&gimg[g].y, (float)ea);
                unsafeAtomicAdd(&gimg[g].z, (float)eb);
                unsafeAtomicAdd(&gimg[g].w, cw_);
                gc[0] -= el;
                gc[1] -= ea;
                gc[2] -= eb;
                first = cfd;
                ++m;
                rem += 2 * am;
                const bool step = rem >= 2 * np;
                rem -= step ? 2 * np : 0;
                x += xmaj || step ? (dx < 0 ? -1 : 1) : 0;
                y += !xmaj || step ? (dy < 0 ? -1 : 1) : 0;
            }
            const int stx = dx < 0 ? -1 : 1, sty = dy < 0 ? -bw : bw;
            const int smaj = xmaj ? stx : sty, sdiag = stx + sty;
            int ls = (y - mny) * bw + (x - mnx);
            if (m < np) {
                atomicAdd(&st[ls], first);
                atomicAdd(&wt[ls], cw_);
                const unsigned F = step_increment(am, np);
                // (after m steps; modulo 2^32, as the steps before would have left it)
                unsigned acc = 0x80000000u + (unsigned)m * F;
                for (++m; m < np; ++m) {
                    const bool cr = __builtin_add_overflow(acc, F, &acc);
                    ls += cr ? sdiag : smaj;
                    atomicAdd(&st[ls], cfd);
                    atomicAdd(&wt[ls], cw_);
                }
            } else if (np == 0) {
                atomicAdd(&st[ls], (double)lf);
            }
            vc += cfd;
            vw += (double)cw_;
        };
        if constexpr (LARGE) {
            for (int a = a0 + own; a < a1; a += WG) walk(pair_at(a));
        } else if (a0 + own < a1) {
            walk(q);
        }
        if (a0 + wave < a1) {                                // uniform: this wave walked
            vc = wave_sum_f64(vc);
            vw = wave_sum_f64(vw);
            const int e = (cy - mny) * bw + (cx - mnx);
            if (lane == 0) {
                atomicAdd(&st[e], vc);
                atomicAdd(&wt[e], (float)vw);
            }
        }
        __syncthreads();
        // the fold
        const int dr = WG / bw, dc = WG - dr * bw;
        int r = tid / bw, c = tid - r * bw;
        for (int e0 = 0; e0 < area; e0 += kFold * WG) {      // uniform: every lane stays
            double sv[kFold];
            float wv[kFold];
            float4 f[kFold];
            int p[kFold];
#pragma unroll
            for (int u = 0; u < kFold; ++u) {
                const int e = e0 + tid + u * WG;
                sv[u] = e < area ? st[e] : 0.0;
                wv[u] = e < area ? wt[e] : 0.0f;
                p[u] = (mny + r) * W + mnx + c;
                c += dc;
                const bool wrap = c >= bw;
                c -= wrap ? bw : 0;
                r += dr + (wrap ? 1 : 0);
            }
#pragma unroll
            for (int u = 0; u < kFold; ++u)
                if (sv[u] != 0.0 || wv[u] != 0.0f) f[u] = img[p[u]];
#pragma unroll
            for (int u = 0; u < kFold; ++u) {
                if (__ballot(sv[u] != 0.0 || wv[u] != 0.0f) == 0ULL) continue;   // uniform
                float4 d = make_float4(0.0f, 0.0f, 0.0f, wv[u]);
                if (sv[u] != 0.0) {
                    const double el = sv[u] * (double)(f[u].x - cl);
                    const double ea = sv[u] * (double)(f[u].y - ca);
                    const double eb = sv[u] * (double)(f[u].z - cb);
                    gc[0] -= el;
                    gc[1] -= ea;
                    gc[2] -= eb;
                    d.x = (float)el;
                    d.y = (float)ea;
                    d.z = (float)eb;
                }
                // through LDS, so that an atomic instruction adds the four
                // values of 16 neighbouring texels, 256 bytes in a row,
                // and not one value of 64 texels
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                turn[wave][lane] = d;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int from = 16 * v + (lane >> 2);
                    const float val = reinterpret_cast<const float*>(&turn[wave][from])[lane & 3];
                    const int q = __shfl(p[u], from, 64);
                    if (val != 0.0f)
                        unsafeAtomicAdd(reinterpret_cast<float*>(gimg + q) + (lane & 3), val);
                }
            }
        }
        if constexpr (!LARGE) {
            a0 = a1;
            a1 = min(total, a0 + WG);
        }
        __syncthreads();                          // wbox and the tiles are written again
    }
    // dL/dTheta_{t-1}: the pass-through of a superpixel whose soft mass was
    // zero (it kept its previous centre) and the path terms
    if (total > 0) {                              // uniform
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            gc[v] = wave_sum_f64(gc[v]);
            if (lane == 0) red[v][wave] = gc[v];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const bool kept = !(z[bk] >= kZMin);
        double g[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            g[v] = kept ? gth[5LL * bk + v] : 0.0;
            if (total > 0)
                for (int w = 0; w < kWaves; ++w) g[v] += red[v][w];
            gth_prev[5LL * bk + v] = g[v];
        }
        if (z_prev) store_cand(z_prev[bk], g, theta_prev + 5LL * bk, cand + 2LL * bk);
    }
}

// Theta_0 = cell means: dL/df_p += dL/dTheta_0 / |cell|; then the outputs:
// dL/dlab = dL/df and dL/dC = dL/dw * 2C/sigma^2 exp(-C^2/sigma^2).
__global__ __launch_bounds__(256) void k_soft_bwd_finish(SoftImg s, const float4* __restrict__ gf,
                                                         const double* __restrict__ gth0,
                                                         const float* __restrict__ contour,
                                                         float sigma, float* __restrict__ glab,
                                                         float* __restrict__ gcon) {
    const double s2 = (double)sigma * (double)sigma;
    SOFT_FOR_PIXELS(s) {
        const long long p = (long long)y * s.W + x;
        const long long i = (long long)b * s.N + p;
        const int ci = cell_of(y, s.ny, s.H), cj = cell_of(x, s.nx, s.W);
        const int cnt = (cell_lo(cj + 1, s.W, s.nx) - cell_lo(cj, s.W, s.nx)) *
                        (cell_lo(ci + 1, s.H, s.ny) - cell_lo(ci, s.H, s.ny));
        const double* g0 = gth0 + 5LL * s.K * b + 5LL * (ci * s.nx + cj);
        const float4 v = gf[i];
        glab[3 * i] = v.x + (float)(g0[0] / cnt);
        glab[3 * i + 1] = v.y + (float)(g0[1] / cnt);
        glab[3 * i + 2] = v.z + (float)(g0[2] / cnt);
        const double c = contour[i];
        gcon[i] = (float)((double)v.w * (2.0 * c / s2) * exp(-(c * c) / s2));
    }
}

constexpr int kSoftWG = 256;
// Tile budget of the backward path pass in bytes (an FP64 weight and an FP32
// dL/dw per texel): what the paths of one cell's pixels to a superpixel of the
// 3x3 block around it mostly span, 1.8 cells by 1.8 cells, at least
// kBwdLdsLeast and at most kBwdLdsBytes.  44 KiB and 9 KiB of static LDS fit three
// times in a CU's 160 KiB; with less the pairs of small cells come apart into more
// batches, with more a CU holds fewer workgroups.  Path pass at 28, 44 and 60 KiB,
// 512x512, k = 400, T = 0.5: 16 images 152, 144, 184 us, 4 images 67, 50, 56; 2 x
// 256x256, k = 128: 27, 17, 17; 16 images at T = 5: 674, 718, 831.
constexpr int kBwdLdsLeast = 44 * 1024;
constexpr int kBwdLdsBytes = 60 * 1024;

static int path_lds_bytes(const SoftGeom& g, int cap_bytes) {
    const double cw = (double)g.W / g.nx, ch = (double)g.H / g.ny;
    const double want = std::min(12.0 * 1.8 * 1.8 * cw * ch, (double)kBwdLdsBytes);
    return std::min(cap_bytes, std::max((int)want, kBwdLdsLeast)) & ~15;
}

unsigned grid_for(long long n) {
    return (unsigned)std::max<long long>(1, std::min<long long>((n + 255) / 256, 65536));
}

}  // namespace

SoftGeom soft_geom(int W, int H, int nx, int ny, int B, float spw, float gamma, float lambda,
                   float temperature, int wg, int prune) {
    SoftGeom g;
    g.W = W; g.H = H; g.nx = nx; g.ny = ny; g.B = B; g.wg = wg;
    g.spw = spw; g.gamma = gamma; g.lambda = lambda; g.temperature = temperature;
    g.prune = prune;
    return g;
}

// Grid of the per-pixel soft kernels: about 4096 blocks over all images.
static dim3 pixel_grid(const SoftImg& s) {
    const int bx = (s.W + 255) / 256;
    const int by = std::max(1, std::min(s.H, 4096 / std::max(1, bx * s.B)));
    return dim3((unsigned)bx, (unsigned)std::min(by, 65535), (unsigned)s.B);
}

int soft_bwd_slices(int W, int H, int nx, int ny) {
    return std::min(assign_slices(W, H, nx, ny, 1024, 1), kBwdLists / 9);
}

static SoftImg to_img(const SoftGeom& g) {
    SoftImg s;
    s.W = g.W; s.H = g.H; s.nx = g.nx; s.ny = g.ny; s.K = g.nx * g.ny; s.B = g.B;
    s.N = (long long)g.W * g.H;
    s.spl = 0;
    s.near = s.N < (1LL << 28) && g.W + g.H < 46340;
    s.bspl = soft_bwd_slices(g.W, g.H, g.nx, g.ny);
    s.inv_w = 1.0 / (double)g.W;
    for (int i = 0; i < 2; ++i) {
        const long long ch = g.H / g.ny + i, cw = g.W / g.nx + 1;
        s.dper[i] = fast_div(8 * ch, cw * ch);
    }
    s.spw = g.spw; s.gamma = g.gamma; s.lambda = g.lambda; s.inv_t = 1.0f / g.temperature;
    s.temp = (double)g.temperature;
    s.prune = g.prune;
    return s;
}

void lift_soft_lds_limits() {
    for (const auto kernel : {k_soft_bwd_path<kPathWG, false>, k_soft_bwd_path<kPathWideWG, false>,
                              k_soft_bwd_path<kPathWG, true>, k_soft_bwd_path<kPathWideWG, true>})
        static_cast<void>(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize,
                                              kBwdLdsBytes));
    static_cast<void>(hipGetLastError());
}

int launch_soft_init(const SoftGeom& g, const float4* packed, float* theta0, hipStream_t st) {
    const SoftImg s = to_img(g);
    hipLaunchKernelGGL(k_soft_init<kSoftWG>, dim3(s.B * s.K), dim3(kSoftWG), 0, st, s, packed,
                       theta0);
    return hipGetLastError();
}

template <int WG>
static int soft_assign_t(const SoftGeom& g, const float4* packed, const float* theta_prev, float* q,
                         float* fa, float* fb, unsigned short* pmask, hipStream_t st) {
    SoftImg s = to_img(g);
    s.spl = assign_slices(g.W, g.H, g.nx, g.ny, WG, fill_slices((long long)g.B * s.K));
    const auto kernel = s.near ? k_soft_assign<WG, true> : k_soft_assign<WG, false>;
    hipLaunchKernelGGL(kernel, dim3(s.B * s.K * s.spl), dim3(WG), 0, st, s, packed,
                       theta_prev, q, fa, fb, pmask);
    return hipGetLastError();
}

// Whether k_soft_tables takes the assignment: without exact pruning, or where the
// softmax reaches so far that the bound's spatial term rules few neighbours out: 111 T
// against the m^2 that one cell side adds to D, four times that for two (colours still
// may).  Not in launches of few cells, nor where a table has more entries than the
// pixels' paths samples (see walk_of).  Forward of 8 x 512x512, k = 400, at T = 0.5, 2,
// 3.6, 5 and 50: 955, 1063, 1112, 1136 and 1392 us, 735, 1040, 1205, 1276 and 1979 by pairs;
// 1 x 512x512, k = 1200, at 2 and 3.6: 240 and 246, 269 and 308.
static bool soft_tables(const SoftGeom& g) {
    const double N = (double)g.B * g.W * g.H, K = (double)g.B * g.nx * g.ny;
    return (!g.prune || 111.0 * g.temperature >= 3.0 * g.spw * N / K) &&
           N >= std::max(128, g.wg / 4) * K && std::max(K, N / kTablePixels) > 96;
}

// Workgroup size of the assignment.  By pairs, 512 lanes where there are no more cells
// than compute units (2 x 97x61, T = 5: 14.4 us per assignment at 256, 13.3 at 512,
// 13.9 at 1024; 2 x 256x256, k = 128: 34, 31, 40).  Over tables, 1024 where there are at
// most two workgroups of that size per compute unit (forward of 512x512, k = 400, T = 50:
// 350, 347 and 327 us; eight of them 1392, 1535 and 1512).
static int assign_wg(const SoftGeom& g, bool tables) {
    if (g.wg != 0) return g.wg;
    const long long cells = (long long)g.B * g.nx * g.ny;
    return tables ? cells <= 2 * kCUs ? 1024 : 256 : cells <= kCUs ? 512 : 256;
}

template <int WG>
static int soft_tables_t(const SoftGeom& g, const float4* packed, const float* theta_prev, float* q,
                         float* fa, float* fb, unsigned short* pmask, hipStream_t st) {
    SoftImg s = to_img(g);
    s.spl = assign_slices(g.W, g.H, g.nx, g.ny, WG, 1);
    const auto kernel = s.near ? k_soft_tables<WG, true> : k_soft_tables<WG, false>;
    hipLaunchKernelGGL(kernel, dim3(s.B * s.K * s.spl), dim3(WG), 0, st, s, packed,
                       theta_prev, q, fa, fb, pmask);
    return hipGetLastError();
}

int launch_soft_assign(const SoftGeom& g, const float4* packed, const float* theta_prev, float* q,
                       float* fa, float* fb, unsigned short* pmask, hipStream_t st) {
    const bool tables = soft_tables(g);
    const int wg = assign_wg(g, tables);
    const auto launch = wg == 1024  ? tables ? soft_tables_t<1024> : soft_assign_t<1024>
                        : wg == 512 ? tables ? soft_tables_t<512> : soft_assign_t<512>
                                    : tables ? soft_tables_t<256> : soft_assign_t<256>;
    return launch(g, packed, theta_prev, q, fa, fb, pmask, st);
}

int launch_soft_update(const SoftGeom& g, const float* q, const unsigned short* pmask,
                       const float4* packed, const float* theta_prev, float* theta_next, double* z,
                       hipStream_t st) {
    const SoftImg s = to_img(g);
    hipLaunchKernelGGL(k_soft_update<kSoftWG>, dim3(s.B * s.K), dim3(kSoftWG), 0, st, s, q, pmask,
                       packed, theta_prev, theta_next, z);
    return hipGetLastError();
}

int launch_soft_bwd_start(const SoftGeom& g, const float* grad_theta, const double* z,
                          const float* theta, double* gth, float4* cand, hipStream_t st) {
    const SoftImg s = to_img(g);
    hipLaunchKernelGGL(k_soft_bwd_start, dim3(grid_for((long long)s.B * s.K)), dim3(256), 0, st, s,
                       grad_theta, z, theta, gth, cand);
    return hipGetLastError();
}

int launch_soft_bwd_update(const SoftGeom& g, int first, const float* q,
                           const unsigned short* pmask, const float4* packed, const float* gq_in,
                           const float4* cand, uint2* pairs, int* count, float4* gf,
                           hipStream_t st) {
    const SoftImg s = to_img(g);
    hipLaunchKernelGGL(k_soft_bwd_update, dim3(s.B * s.K * s.bspl), dim3(kUpdateWG), 0, st, s,
                       first, q, pmask, cand, packed, gq_in, pairs, count, gf);
    return hipGetLastError();
}

int launch_soft_bwd_path(const SoftGeom& g, const float4* packed, const float* theta_prev,
                         const float* fa, const float* fb, const uint2* pairs, const int* count,
                         const double* z, const double* gth, const double* z_prev,
                         double* gth_prev, float4* cand, float4* gf, int cap_bytes,
                         hipStream_t st) {
    const SoftImg s = to_img(g);
    const int cap = path_lds_bytes(g, cap_bytes);
    const bool wide = (long long)s.B * s.K <= 2 * kCUs;
    // (512x512 pixels in cells of 51x51, 5 iterations at T = 0.5 and 5: 0.35 and 1.22 ms
    // LARGE, 0.36 and 1.29 else; four 256x256 in cells of 57x57 0.45 and 0.87, 0.70 and
    // 1.46; 512x512 in cells of 26x26 0.23 and 0.67, 0.20 and 0.66)
    const bool large = 1.75 * g.W / g.nx * g.H / g.ny > cap / 12;
    const auto kernel = large ? wide ? k_soft_bwd_path<kPathWideWG, true> : k_soft_bwd_path<kPathWG, true>
                        : wide ? k_soft_bwd_path<kPathWideWG, false> : k_soft_bwd_path<kPathWG, false>;
    hipLaunchKernelGGL(kernel, dim3(s.B * s.K), dim3(wide ? kPathWideWG : kPathWG), (size_t)cap, st, s,
                       packed, theta_prev, fa, fb, pairs, count, z, gth, z_prev, gth_prev, cand,
                       gf, cap);
    return hipGetLastError();
}

int launch_soft_bwd_finish(const SoftGeom& g, const float4* gf, const double* gth0,
                           const float* contour, float sigma, float* glab, float* gcon,
                           hipStream_t st) {
    const SoftImg s = to_img(g);
    hipLaunchKernelGGL(k_soft_bwd_finish, pixel_grid(s), dim3(256), 0, st, s, gf, gth0,
                       contour, sigma, glab, gcon);
    return hipGetLastError();
}

}  // namespace scalp
