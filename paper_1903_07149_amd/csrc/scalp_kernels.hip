// scalp_kernels.hip -- HIP kernels (gfx950) of the SCALP clustering path.
//
//   k_prepare         packs (l, a, b, w) with w = 1 - exp(-C^2/sigma^2), the
//                     summand of Eq. (2), evaluated in FP64 and rounded once.
//   k_init_cells      Algorithm 1 initialisation: labels = grid cell, per-cell
//                     integer sums (Sec. II-A regular grid).
//   k_assign*         Algorithm 1 assignment: one workgroup per (cell, slice)
//                     work item, one pixel per lane.  Each pixel orders its
//                     <= 9 candidates by an exact lower bound of their D
//                     (colour at the pixel and spatial term only), walks the
//                     discrete line (Sec. II-B) to the endpoint of the first,
//                     accumulating Eq. (1)'s colour term and Eq. (2)'s contour
//                     term in a fixed FP32 order, and forms D of Eq. (3); the
//                     candidates whose bound does not exceed that D are listed
//                     and walked by full waves.  The first strict minimum
//                     wins, as if every candidate had been walked.  With ACCUM
//                     the update's sums are fused in: each pixel can only
//                     choose among the cell's 9 candidates, so they reduce
//                     into 9 LDS bins and leave the workgroup as at most 54
//                     integer atomics.
//   k_finalize*       Algorithm 1 update: means from the integer sums, the
//                     rounded barycenter, and the membership test of the
//                     Sec. II-D Remark; clusters that fail it are queued.
//   k_project*        Eq. (4): nearest member pixel of each queued cluster.
//
// All FP32 arithmetic of the distance is written operation by operation and
// compiled with -ffp-contract=off, so it matches the plain CPU definition
// bit for bit.
#include <algorithm>
#include <climits>

#include "scalp_device.h"

namespace scalp {
namespace {

using namespace dev;

// Copies of the update bins: the lanes of a wave mostly pick the same
// candidate, and 64-bit LDS atomics on one word serialise, so lane t adds to
// copy (t ^ (t >> 3)) mod kBinCopies: every row and every column of the
// wave's 8x8 pixel block spreads over all copies, and at most 8 lanes of a
// wave share one word.
constexpr int kBinCopies = 8;

// Per work item, by pixel (lane of the first pass): its coordinates and its
// smallest (FP32 bits of D) << 32 | slot so far; the (pixel, slot) pairs of
// the second pass, and their number; and the update bins, [slot * 6 + sum][copy].
template <int WG>
struct ItemShared {
    unsigned long long bins[9 * 6][kBinCopies];
    unsigned long long win[WG];
    int2 xy[WG];
    unsigned short list[8 * WG];
    int pairs;
};

// Per work item of walk_tables: a candidate's table, or two of half the size; then the
// update bins.  72 bytes a lane: the LDS of as many workgroups as the registers let a
// CU hold.
template <int WG>
struct TableShared {
    static constexpr int kEntries = 9 * WG - 8;
    union {
        unsigned long long bins[9 * 6][kBinCopies];
        float2 table[kEntries];
    };
    int box[4];            // of the pixels
};

// An item of more pairs per pixel in its second pass than this goes over tables instead
// (walk_tables): images of noise, or whose contours are nowhere low, leave most of the
// candidates to be walked.  10 iterations of 1920x1080, k = 2000, at 4, 6 and 8 (none):
// the benchmark's image 732, 725 and 727 us; noise 2.52, 2.58 and 4.56 ms; contours of up
// to 0.2 everywhere added to the benchmark's 1.68, 1.86 and 1.96.  (By rounds of the
// lanes instead, which an item of 192 pixels never has six of: noise at k = 4000 3.57
// ms instead of 2.52, one colour at m = 0 4.15 instead of 1.79.)  Not items of at most
// half the lanes, whose pairs take few rounds: 12 scales of 481x321 2.29 ms instead of
// 2.20, 97x61 0.143 instead of 0.131.
constexpr int kManyPairs = 6;

// A descriptor read through the scalar cache, word by word (p uniform).
__device__ __forceinline__ Img load_const(const Img* p) {
    static_assert(sizeof(Img) % 4 == 0, "words");
    union {
        Img im;
        int w[sizeof(Img) / 4];
    } u;
    const ConstI c = (ConstI)(uintptr_t)p;
#pragma unroll
    for (unsigned i = 0; i < sizeof(Img) / 4; ++i) u.w[i] = __builtin_amdgcn_readfirstlane(c[i]);
    return u.im;
}

// First 64-pixel chunk of slice i of a cell of `chunks` chunks.
__device__ __forceinline__ int slice_chunk(int chunks, int i, const Img& im) {
    const long long v = (long long)chunks * i;
    return v < (1LL << 31) ? fdiv((int)v, im.dspl) : (int)(v / im.spl);
}

// The update's bins, [slot * 6 + sum][copy].
typedef unsigned long long Bins[9 * 6][kBinCopies];

template <int WG>
__device__ __forceinline__ void clear_bins(Bins& bins) {
    for (int t = threadIdx.x; t < 54 * kBinCopies; t += WG) (&bins[0][0])[t] = 0ULL;
}

// The label of pixel (px, py) and its share of the update's sums: superpixel k, slot j.
template <bool ACCUM>
__device__ __forceinline__ void settle(const Img& im, const float4* __restrict__ img, int px, int py,
                                       int j, int k, int* __restrict__ labels, Bins& bins) {
    const long long p = (long long)py * im.W + px;
    labels[im.pix + p] = k;
    if (ACCUM) {
        const float4 f = img[p];
        const int tid = threadIdx.x, cp = (tid ^ (tid >> 3)) & (kBinCopies - 1);
        unsigned long long(*bin)[kBinCopies] = bins + 6 * j;
        atomicAdd(&bin[0][cp], 1ULL);
        atomicAdd(&bin[1][cp], (unsigned long long)px);
        atomicAdd(&bin[2][cp], (unsigned long long)py);
        atomicAdd(&bin[3][cp], (unsigned long long)to_fixed(f.x));
        atomicAdd(&bin[4][cp], (unsigned long long)to_fixed(f.y));
        atomicAdd(&bin[5][cp], (unsigned long long)to_fixed(f.z));
    }
}

// The bins to the sums of superpixels k0, k0 + 1, ... (first of the cell's 3 rows).
__device__ __forceinline__ void flush_bins(const Img& im, int k0, Bins& bins,
                                           long long* __restrict__ acc) {
    const int tid = threadIdx.x;
    if (tid < 54) {
        const int j = tid / 6, di = j / 3;
        unsigned long long n = 0, v = 0;
        for (int c = 0; c < kBinCopies; ++c) {
            n += bins[6 * j][c];
            v += bins[tid][c];
        }
        if (n != 0ULL)
            atomicAdd((unsigned long long*)(acc + kAccStride * (long long)(im.sp + k0 + di * im.nx +
                                                                           (j - 3 * di)) +
                                            (tid - 6 * j)),
                      v);
    }
}

// A work item: pixels [t0, t1) in cell_pixel order of the cell of row ci and column cj.
struct Item {
    int ci, cj, x0, y0, cw, ch, t0, t1;
};

__device__ __forceinline__ Item item_of(const Img& im, int ci, int cj, int slice) {
    Item it;
    it.ci = ci;
    it.cj = cj;
    it.x0 = cell_lo(cj, im.W, im.nx, im.dnx);
    it.y0 = cell_lo(ci, im.H, im.ny, im.dny);
    it.cw = cell_lo(cj + 1, im.W, im.nx, im.dnx) - it.x0;
    it.ch = cell_lo(ci + 1, im.H, im.ny, im.dny) - it.y0;
    const int P = it.cw * it.ch;
    it.t0 = 0;
    it.t1 = P;
    if (im.spl > 1) {                              // uniform
        const int chunks = (P + 63) >> 6;
        it.t0 = 64 * slice_chunk(chunks, slice, im);
        it.t1 = min(P, 64 * slice_chunk(chunks, slice + 1, im));
    }
    return it;
}

template <bool NEAR>
__device__ __forceinline__ Eqs item_eqs(const Img& im, const Item& it, const Neighbours& nb,
                                        const float4* __restrict__ img, const int* __restrict__ end,
                                        float lambda) {
    Eqs eqs;
    eqs.img = img;
    eqs.W = im.W;
    near_all(eqs);
    if (!NEAR) {
        // (of the whole cell; endpoints outside the image are clamped into it)
        Box box = {it.x0, it.y0, it.x0 + it.cw - 1, it.y0 + it.ch - 1};
        const ConstI ce = (ConstI)(uintptr_t)end;
        for (int j = 0; j < 9; ++j) {
            const int k = nb.row[j / 3] + nb.col[j % 3];
            box.add(min(max(ce[2 * k], 0), im.W - 1), min(max(ce[2 * k + 1], 0), im.H - 1));
        }
        near_box(eqs, box);
    }
    eqs.lambda = lambda;
    eqs.oml = 1.0f - lambda;
    eqs.gamma = im.gamma;
    eqs.spw = im.spw;
    return eqs;
}

// A work item whose pixels walk many candidates: candidate by candidate the workgroup
// writes (d_c, w) over the box of the pixels and the candidate's endpoint, which holds
// every path to it, into an LDS table, and the paths are walked there; over global
// memory where the box exceeds the LDS.  The winner is the smallest (D, slot).  A lane
// has up to ROUNDS pixels, one at a time in best[0] and at[0] (x and y within the box,
// slot), which rotate.  Where two tables fit, they alternate: one barrier a candidate.
// PRUNE: the own cell's candidate first, then the edges', then the corners', and a
// pixel leaves those out whose bound (that of bound_keys, unfused: never above D) its
// smallest D so far rules out.
//
// What bounds it: VALU issue; a sample costs 5 instructions and an 8-byte LDS read.  10
// iterations of 1920x1080, k = 2000, without pruning: 1.63 ms; 4.68 by the pairs of
// process_cell, whose samples cost 13 instructions and 16 bytes through L1.
template <int WG, bool ACCUM, int ROUNDS, bool PRUNE>
__device__ __forceinline__ void walk_tables(const Eqs& eqs, const Img& im, const Item& it,
                                            const Neighbours& nb, int k0,
                                            const float* __restrict__ cen,
                                            const int* __restrict__ end, int* __restrict__ labels,
                                            TableShared<WG>& sh) {
    constexpr int kRounds = ROUNDS;
    const int tid = threadIdx.x, W = im.W, H = im.H;
    const float4* __restrict__ img = eqs.img;
    const bool cut = im.gamma <= 0x1p40f;
    float best[kRounds];
    unsigned at[kRounds];
    Box own;
    {
        const PixelMap map = pixel_map(im.dper, it.cw, it.ch);
        int x[kRounds], y[kRounds];
        int lx = INT_MAX, ly = INT_MAX, hx = 0, hy = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            x[r] = y[r] = -1;
            const int t = it.t0 + r * WG + tid;
            if (t < it.t1) {
                pixel_at(map, t, x[r], y[r]);
                x[r] += it.x0;
                y[r] += it.y0;
                lx = min(lx, x[r]);
                ly = min(ly, y[r]);
                hx = max(hx, x[r]);
                hy = max(hy, y[r]);
            }
        }
        lx = wave_min_i32(lx);
        ly = wave_min_i32(ly);
        hx = wave_max_i32(hx);
        hy = wave_max_i32(hy);
        if ((tid & 63) == 0) {
            atomicMin(&sh.box[0], lx);
            atomicMin(&sh.box[1], ly);
            atomicMax(&sh.box[2], hx);
            atomicMax(&sh.box[3], hy);
        }
        __syncthreads();
        own.x0 = __builtin_amdgcn_readfirstlane(sh.box[0]);
        own.y0 = __builtin_amdgcn_readfirstlane(sh.box[1]);
        own.x1 = __builtin_amdgcn_readfirstlane(sh.box[2]);
        own.y1 = __builtin_amdgcn_readfirstlane(sh.box[3]);
        // (kTablePixels pixels of 8-wide strips span fewer than 4096 rows and columns)
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            best[r] = INFINITY;
            at[r] = y[r] < 0 ? ~0u
                             : (unsigned)(x[r] - own.x0) | ((unsigned)(y[r] - own.y0) << 12) | (15u << 24);
        }
    }
    bool half = false, was_full = false;           // uniform
#pragma unroll 1
    for (int i = 0; i < 9; ++i) {
        // ascending, or 4, 1, 3, 5, 7, 0, 2, 6, 8
        const int j = PRUNE ? (int)((0x862075314ULL >> (4 * i)) & 15ULL) : i;
        if (!((nb.inside >> j) & 1u)) continue;    // uniform
        const int di = (j * 11) >> 5, kk = k0 + di * im.nx + (j - 3 * di);
        const ConstF cp = (ConstF)(uintptr_t)cen + 5 * kk;
        const ConstI ep = (ConstI)(uintptr_t)end + 2 * kk;
        const float ck[5] = {cp[0], cp[1], cp[2], cp[3], cp[4]};
        const int cx = min(max(ep[0], 0), W - 1), cy = min(max(ep[1], 0), H - 1);
        Box box = own;
        box.add(cx, cy);
        const Table t = table_of(box, TableShared<WG>::kEntries, WG);
        const bool full = t.pitch * t.rows > TableShared<WG>::kEntries / 2;
        if (t.fits) {
            if (full || was_full) __syncthreads(); // the table before was read
            half = !half && !full;
            was_full = full;
        }
        float2* table = sh.table + (half ? TableShared<WG>::kEntries / 2 : 0);
        if (t.fits) {
            fill_table<WG>(table, t, img, W, ck[0], ck[1], ck[2]);
            __syncthreads();
        }
#pragma unroll 1
        for (int r = 0; r < kRounds; ++r) {
            if (at[0] != ~0u) {
                const int px = own.x0 + (int)(at[0] & 4095u), py = own.y0 + (int)((at[0] >> 12) & 4095u);
                const int slot = (int)(at[0] >> 24);
                float A, B, D, lb = 0.0f;
                if (PRUNE) {
                    float dcp;
                    if (t.fits) {                  // uniform
                        dcp = table[(py - t.y0) * t.pitch + (px - t.x0)].x;
                    } else {
                        dcp = colour_dist(img[py * W + px], ck[0], ck[1], ck[2]);
                    }
                    const float ax = (float)px - ck[3], ay = (float)py - ck[4];
                    lb = eqs.lambda * dcp + (ax * ax + ay * ay) * eqs.spw;
                }
                if (!(PRUNE && (lb > best[0] || (lb == best[0] && j > slot)))) {
                    if (t.fits)                    // uniform
                        D = table_distance(eqs, ck, t, table, cx, cy, px, py, A, B);
                    else
                        D = path_distance(eqs, ck, img[py * W + px], cx, cy, px, py, PRUNE && cut,
                                          threshold(best[0]), A, B);
                    if (D < best[0] || (PRUNE && D == best[0] && j < slot)) {
                        best[0] = D;
                        at[0] = (at[0] & 0xffffffu) | ((unsigned)j << 24);
                    }
                }
            }
            const float b0 = best[0];
            const unsigned a0 = at[0];
#pragma unroll
            for (int q = 0; q + 1 < kRounds; ++q) {
                best[q] = best[q + 1];
                at[q] = at[q + 1];
            }
            best[kRounds - 1] = b0;
            at[kRounds - 1] = a0;
        }
    }
    __syncthreads();
    if (ACCUM) {
        clear_bins<WG>(sh.bins);
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (at[r] == ~0u) continue;
        const int slot = (int)(at[r] >> 24);
        const int j = slot == 15 ? 4 : slot;       // no slot only with non-finite input
        const int di = (j * 11) >> 5;
        settle<ACCUM>(im, img, own.x0 + (int)(at[r] & 4095u), own.y0 + (int)((at[r] >> 12) & 4095u),
                      j, k0 + di * im.nx + (j - 3 * di), labels, sh.bins);
    }
}

// Without exact pruning every pixel of a work item walks every candidate, up to
// kTablePixels of them.
template <int WG, bool ACCUM, bool NEAR>
__device__ __forceinline__ void assign_all(const Img& im, int ci, int cj, int slice,
                                           const float4* __restrict__ packed,
                                           const float* __restrict__ centres,
                                           const int* __restrict__ endpoints,
                                           int* __restrict__ labels, long long* __restrict__ acc,
                                           float lambda, TableShared<WG>& sh) {
    const Item it = item_of(im, ci, cj, slice);
    if (it.t1 <= it.t0) return;                    // an empty slice
    const float4* __restrict__ img = packed + im.pix;
    const float* __restrict__ cen = centres + 5LL * im.sp;
    const int* __restrict__ end = endpoints + 2LL * im.sp;
    const Neighbours nb = neighbours_of(im.nx, im.ny, ci, cj);
    const Eqs eqs = item_eqs<NEAR>(im, it, nb, img, end, lambda);
    const int k0 = (ci - 1) * im.nx + cj - 1;
    if (threadIdx.x == 0) {
        sh.box[0] = sh.box[1] = INT_MAX;
        sh.box[2] = sh.box[3] = 0;
    }
    __syncthreads();
    walk_tables<WG, ACCUM, kTablePixels / WG, false>(eqs, im, it, nb, k0, cen, end, labels, sh);
    if (ACCUM) {
        __syncthreads();
        flush_bins(im, k0, sh.bins, acc);
    }
}

// Work item (cell, slice): pixels [t0, t1) of the cell in cell_pixel order,
// one per lane.  The cell's ceil(P / 64) 64-pixel chunks are split evenly
// over its spl slices (spl is chosen on the host so that no slice has more
// than WG pixels), and every wave keeps an 8x8 block.
//
// Every pixel walks the candidate with the smallest lower bound of D first
// (bound_keys), and then only those whose bound does not exceed its D: the
// others could not have been chosen.  The winner is the smallest (D, slot)
// pair, which is the first strict minimum in ascending slot (hence ascending
// k) whatever the visiting order: the labels are those of evaluating every
// candidate.  An infinite or NaN D never wins.
//
// The first candidate decides 80 % of the pixels; the others whose bound does
// not exceed its D, 0.2 per pixel and most of them losers, are listed and
// walked by full waves of (pixel, slot) pairs, whose results meet in a 64-bit
// minimum per pixel.  They are listed slot by slot, so that the lanes of a wave walk
// to one endpoint: taken in the order of each pixel's bounds, an image of noise took 5.93
// ms instead of 4.56 (10 iterations of 1920x1080), 481x321 191 us instead of 186.  A wave
// takes its places in the list at once for all nine slots: a place per slot, nine LDS
// atomics in a row, 481x321 189 us instead of 179 and 97x61 139 instead of 130.  A walk of
// that second pass stops as soon as its partial sums prove that D exceeds the pixel's
// first one (Cut).
//
// NEAR (near_image): the walks by 32-bit indexes alone.  The other kernels choose per
// item (near_box); both walks in one kernel need 10 registers more and took 1 to 2 %
// longer.
//
// What bounds it: VALU issue.  32.3 M wave instructions per launch at
// 1920x1080, k = 2000 (the bounds 180 of a wave's 990, the first walk 300,
// its evaluation 150, the second pass 200), 0.69 per CU-clock of the whole launch, its
// start and end included, with 43 of 64 lanes active: the others wait for the longest
// path of their wave.  0.068 ms per launch.  (The settling is one piece of code for all pixels: settled
// in the first pass where nothing was listed, it ran twice in most waves, 1.6 % of
// this launch and 3 % of the 64-image batch.)  Tables of (d_c, w) per candidate in
// LDS, all nine taken in turn by the whole workgroup behind a barrier each, made a
// sample cost 5 instructions instead of 13 but walked 85 samples per pixel in
// 64-lane slots instead of 33, filled 20 table entries per pixel and waited at the
// barriers: 51.5 M instructions, 0.72 per CU-clock of the launch, 0.117 ms.  The
// texels are read through L1 and L2: a box of them staged in LDS per item left two
// items per CU and was slower (0.132 ms against 0.105 with the rest equal), as was a
// counting sort of the first walks by length (18 instead of 23 slots per pixel, but
// 100 more instructions and two more barriers).
template <int WG, bool ACCUM, bool NEAR>
__device__ __forceinline__ void process_cell(const Img& im, int ci, int cj, int slice,
                                             const float4* __restrict__ packed,
                                             const float* __restrict__ centres,
                                             const int* __restrict__ endpoints,
                                             int* __restrict__ labels,
                                             long long* __restrict__ acc, float lambda,
                                             ItemShared<WG>& sh, TableShared<WG>* tables) {
    const int tid = threadIdx.x;
    const int W = im.W, H = im.H;
    const Item it = item_of(im, ci, cj, slice);
    if (it.t1 <= it.t0) return;                    // an empty slice
    const float4* __restrict__ img = packed + im.pix;
    const int sp = __builtin_amdgcn_readfirstlane(im.sp);
    const float* __restrict__ cen = centres + 5LL * sp;
    const int* __restrict__ end = endpoints + 2LL * sp;
    const Neighbours nb = neighbours_of(im.nx, im.ny, ci, cj);
    const Eqs eqs = item_eqs<NEAR>(im, it, nb, img, end, lambda);
    // candidate slot j -> superpixel
    const int k0 = (ci - 1) * im.nx + cj - 1;
    auto superpixel = [&](int j) -> int {
        const int di = (j * 11) >> 5;              // j / 3 for j <= 8
        return k0 + di * im.nx + (j - 3 * di);
    };
    // D of pixel (px, py) with texel fp to candidate slot j (endpoints outside
    // the image are clamped into it); its loads do not wait for one another
    auto distance = [&](int j, float4 fp, int px, int py, bool cut, float thr) -> float {
        const int kk = superpixel(j);
        const int2 ep = *reinterpret_cast<const int2*>(end + 2 * kk);
        const float* cp = cen + 5 * kk;
        const float ck[5] = {cp[0], cp[1], cp[2], cp[3], cp[4]};
        float A, B;
        return path_distance(eqs, ck, fp, min(max(ep.x, 0), W - 1), min(max(ep.y, 0), H - 1), px,
                             py, cut, thr, A, B);
    };

    if (tid == 0) {
        sh.pairs = 0;
        if (tables) {
            tables->box[0] = tables->box[1] = INT_MAX;
            tables->box[2] = tables->box[3] = 0;
        }
    }
    if (ACCUM) clear_bins<WG>(sh.bins);
    __syncthreads();

    // first pass: the candidate with the smallest bound; then every other one
    // whose bound does not exceed that D is listed
    const bool prune = im.prune != 0;
    const bool mine = tid < it.t1 - it.t0;
    bool again = false;
    int px = 0, py = 0, bestj = -1;
    if (mine) {
        pixel_at(pixel_map(im.dper, it.cw, it.ch), it.t0 + tid, px, py);
        px += it.x0;
        py += it.y0;
        unsigned key[9];
        const float4 fp = img[py * W + px];
        bound_keys(nb, (ConstF)(uintptr_t)cen, im.spw, fp, px, py, lambda, key);
        const unsigned nk = next_key(key, kNoKey);
        float best = INFINITY;
        {
            const int j = (int)(nk & 15u);
            const float D = distance(j, fp, px, py, false, 0.0f);
            if (D < best) {
                best = D;
                bestj = j;
            }
        }
        // (keys as integers: a NaN bound is above every limit, and its D is NaN, too)
        const unsigned limit = prune ? __float_as_uint(threshold(best)) | 15u : 0x7fffffffu;
        unsigned long long listed[9];
        int total = 0;
#pragma unroll
        for (int j = 0; j < 9; ++j) {
            listed[j] = __ballot(key[j] <= limit && key[j] != nk);
            total += __popcll(listed[j]);
        }
        if (total != 0) {                          // uniform
            int at = 0;
            if ((tid & 63) == 0) at = atomicAdd(&sh.pairs, total);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const unsigned long long m = listed[j];
                if (key[j] <= limit && key[j] != nk) {
                    sh.list[at + lanes_below(m)] = (unsigned short)(tid | (j << 10));
                    again = true;
                }
                at += __popcll(m);
            }
        }
        if (again) {
            sh.xy[tid] = make_int2(px, py);
            sh.win[tid] = ((unsigned long long)__float_as_uint(best) << 32) | (unsigned)bestj;
        }
    }
    __syncthreads();
    const int pairs = __builtin_amdgcn_readfirstlane(sh.pairs);
    const int pixels = it.t1 - it.t0;
    if (tables && prune && 2 * pixels > WG && pairs > kManyPairs * pixels) {   // uniform
        walk_tables<WG, ACCUM, 1, true>(eqs, im, it, nb, k0, cen, end, labels, *tables);
        if (ACCUM) {
            __syncthreads();
            flush_bins(im, k0, tables->bins, acc);
        }
        return;
    }
    // second pass: the listed pairs, by full waves
    const bool cut = prune && im.gamma <= 0x1p40f;
    for (int i = tid; i < pairs; i += WG) {
        const unsigned e = sh.list[i];
        const int id = (int)(e & 1023u), j = (int)(e >> 10);
        const int2 q = sh.xy[id];
        const float best = __uint_as_float((unsigned)(sh.win[id] >> 32));
        const float D = distance(j, img[q.y * W + q.x], q.x, q.y, cut, threshold(best));
        if (D < INFINITY)
            atomicMin(&sh.win[id], ((unsigned long long)__float_as_uint(D) << 32) | (unsigned)j);
    }
    __syncthreads();
    if (mine) {
        if (again) bestj = (int)(unsigned)sh.win[tid];
        const int j = bestj < 0 ? 4 : bestj;       // no slot only with non-finite input
        settle<ACCUM>(im, img, px, py, j, superpixel(j), labels, sh.bins);
    }
    if (ACCUM) {
        __syncthreads();
        flush_bins(im, k0, sh.bins, acc);
    }
}

template <int WG, bool ACCUM, bool NEAR, Walk WALK>
__device__ __forceinline__ void assign_item(const Img& im, int item, const float4* __restrict__ packed,
                                            const float* __restrict__ centres,
                                            const int* __restrict__ endpoints,
                                            int* __restrict__ labels, long long* __restrict__ acc,
                                            float lambda) {
    const int pos = fdiv(item, im.dspl);
    int ci, cj;
    cell_in_strips(pos, im, ci, cj);
    const int slice = item - pos * im.spl;
    if constexpr (WALK == Walk::kAll) {
        __shared__ TableShared<WG> sh;
        assign_all<WG, ACCUM, NEAR>(im, ci, cj, slice, packed, centres, endpoints, labels, acc, lambda,
                                    sh);
    } else if constexpr (WALK == Walk::kMany) {
        __shared__ union {
            ItemShared<WG> item;
            TableShared<WG> tables;               // (its box behind the item's)
        } sh;
        static_assert(sizeof(ItemShared<WG>) <= offsetof(TableShared<WG>, box), "the box is apart");
        process_cell<WG, ACCUM, NEAR>(im, ci, cj, slice, packed, centres, endpoints, labels, acc,
                                      lambda, sh.item, &sh.tables);
    } else {
        __shared__ ItemShared<WG> sh;
        process_cell<WG, ACCUM, NEAR>(im, ci, cj, slice, packed, centres, endpoints, labels, acc,
                                      lambda, sh, nullptr);
    }
}

template <int WG, bool ACCUM, bool NEAR, Walk WALK>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(8))) void k_assign(
    Img im, const float4* __restrict__ packed, const float* __restrict__ centres,
    const int* __restrict__ endpoints, int* __restrict__ labels, long long* __restrict__ acc, int* ctrl,
    float lambda) {
    if (ACCUM && blockIdx.x == 0 && threadIdx.x == 0) ctrl[kCtrlProjCount] = 0;
    assign_item<WG, ACCUM, NEAR, WALK>(im, xcd_remap(blockIdx.x, gridDim.x), packed, centres, endpoints,
                                       labels, acc, lambda);
}

// The assignment over a ragged batch, a workgroup per (image, cell, slice) item,
// dispatched by the hardware as workgroups end.
//
// XCD x (workgroup b runs on XCD b mod 8) has its own run of items: the x-th
// eighth of every image's items, in the cell order of cell_in_strips, so its
// cells form a block and share its L2, and every XCD starts on every image
// (images of few, large cells walk long paths).  run x = item_start + (n_img +
// 1) (1 + x) holds where each image's share starts in the run.
//
// Workgroups that stayed and took items from eight queues spent their time at
// the queues: an atomic and two barriers per item, and eight failed atomics of
// every workgroup on eight words at the end: 40 us per iteration instead of 26 for 7
// scales of 189x117, 36 instead of 22 for 3 small images; 64 images of up to 2160
// pixels a side 2.95 ms instead of 2.93, and 12 scales of 481x321, where taking over
// another XCD's items helped, 202 instead of 207.
template <int WG, bool NEAR, Walk WALK>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(8))) void k_assign_batched(
    const Img* __restrict__ imgs, const int* __restrict__ item_start, int n_img,
    const float4* __restrict__ packed, const float* __restrict__ centres,
    const int* __restrict__ endpoints, int* __restrict__ labels, long long* __restrict__ acc, int* ctrl,
    float lambda, int h0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl[kCtrlProjCount] = 0;
    // (the tables are constant during the launch: scalar loads)
    const ConstI starts = (ConstI)(uintptr_t)item_start;
    const int x = (int)(blockIdx.x & 7u), h = h0 + (int)(blockIdx.x >> 3);
    const ConstI run = starts + (n_img + 1) * (1 + x);
    if (h >= run[n_img]) return;                   // the shorter runs
    const int i = find_image(run, n_img, h);
    const Img im = load_const(imgs + i);
    const int ni = starts[i + 1] - starts[i];
    const int local = __builtin_amdgcn_readfirstlane((int)((long long)ni * x >> 3) + (h - run[i]));
    assign_item<WG, true, NEAR, WALK>(im, local, packed, centres, endpoints, labels, acc, lambda);
}

// ---------------------------------------------------------------- window form

// Window candidate rule of Algorithm 1: a pixel's candidates are the
// clusters whose window (half-width R around the rounded barycenter)
// contains it, and it takes the smallest D of Eq. (3), the smallest k among
// equal distances: the smallest (FP32 bits of D, k) as a 64-bit number (D >= 0;
// an infinite or NaN D loses to every finite one).  A pixel that no window
// contains keeps its label.  Single images only (im.pix and im.sp are 0).

constexpr int kWinTile = 16;     // a workgroup's tile is kWinTile x kWinTile pixels, or 8 x 8
constexpr int kWinWG = kWinTile * kWinTile;
constexpr int kWinBatch = 15;    // candidates that a tile evaluates at a time (4-bit slots)
constexpr int kWinIds = 512;     // longest list of a tile
constexpr int kWinSmall = 4 * kCUs;   // most tiles of 8 pixels a side

// The tiles' candidates: count[tile] (cleared before the first pass; every tile
// clears its own again) and the first `cap` of them in list[tile * cap ...], in
// any order.
struct WinLists {
    int* count;
    int* list;
    int cap, tile, tx, tiles;   // pixels a side of a tile, tiles of a row, in all
};

// Adds cluster k with barycenter (x, y) to the tiles that its window meets.  The
// lanes of one wave call.
__device__ __forceinline__ void add_to_tiles(const Img& im, int k, float x, float y, int R,
                                             const WinLists& wl) {
    const int wx = round_coord(x, im.W - 1), wy = round_coord(y, im.H - 1);
    const int sh = wl.tile == 8 ? 3 : 4;           // uniform
    const int tx0 = max(wx - R, 0) >> sh, tx1 = min(wx + R, im.W - 1) >> sh;
    const int ty0 = max(wy - R, 0) >> sh, ty1 = min(wy + R, im.H - 1) >> sh;
    const int nx = tx1 - tx0 + 1, n = nx * (ty1 - ty0 + 1);
    for (int i = threadIdx.x & 63; i < n; i += 64) {
        const int r = i / nx;
        const int tile = (ty0 + r) * wl.tx + tx0 + (i - r * nx);
        const int at = atomicAdd(&wl.count[tile], 1);
        if (at < wl.cap) wl.list[(long long)tile * wl.cap + at] = k;
    }
}

// The lists of all clusters, a wave per cluster (before the first pass of a run;
// k_finalize_project makes those of the next one).
__global__ __launch_bounds__(256) void k_window_lists(Img im, const float* __restrict__ centres, int R,
                                                      WinLists wl) {
    const int k = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (k >= im.nx * im.ny) return;
    add_to_tiles(im, k, centres[5LL * k + 3], centres[5LL * k + 4], R, wl);
}

// Candidates are numbered by their place in ids, which is in ascending k; win is,
// by pixel, the smallest (FP32 bits of D) << 32 | number + 1, with 0 as the number
// of a cluster of an earlier list (its k is smaller; its label is stored).
struct WinShared {
    unsigned long long bins[kWinBatch * 6][kBinCopies];   // the update's sums, [slot * 6 + sum]
    unsigned long long win[kWinWG];
    float4 cand[kWinBatch][2];                            // (l, a, b, x), (y, endpoint)
    int2 box[kWinBatch];                                  // the window's corner
    int ids[kWinIds], unsorted[kWinIds];
    unsigned short list[(kWinBatch - 1) * kWinWG];        // pixel | slot << 8
    int pairs, count[kWinWG / 64];
};

__device__ __forceinline__ unsigned med3(unsigned a, unsigned b, unsigned c) {
    return max(min(a, b), min(max(a, b), c));
}

// What a bound must exceed for its candidate to lose to `win`; nothing does
// while that is no finite D.
__device__ __forceinline__ float win_threshold(unsigned long long win) {
    const float best = __uint_as_float((unsigned)(win >> 32));
    return best < INFINITY ? threshold(best) : INFINITY;
}

// A workgroup takes a tile of kWinTile x kWinTile pixels, one pixel per lane, a
// wave an 8x8 block.  It evaluates the tile's candidates as the grid form does its
// 9: the candidate with the smallest lower bound of D first, then by full waves the
// (pixel, candidate) pairs whose bound does not exceed that D.  More than kWinBatch
// candidates are taken in batches against the smallest D so far; a tile whose list
// overflowed, and every tile without lists, tests all clusters, kWinWG at a time.
// TILE is kWinTile, or 8 for small images (win_tile), where a tile of 16 would leave
// most of the chip without work (the lanes without a pixel test clusters and walk
// pairs): 10 iterations of 97x61, k = 30, 159 us with tiles of 16, 145 with 8; of 189x117,
// k = 300, with lists, 239 and 195.
// With ACCUM the update's sums go through bins per candidate of the tile (to global
// memory directly for pixels that no window contains, and for winners of an earlier
// turn of an overflowed list).
//
// What bounds it: VALU issue, as in the grid form (31 M wave instructions per
// launch at 1920x1080, k = 2000, R = 32).  69 us with the sums.  A workgroup per
// cluster that walked its whole window over a table in LDS (4.1 walks per pixel,
// each result through a 64-bit minimum in global memory) took 78, and the sums
// another 17.  One kernel for NEAR and not took 77 (the walks by 64-bit indexes made
// it spill), all keys of a batch in registers instead of the four smallest 95, and
// 72 at 7 waves per SIMD.
template <bool ACCUM, bool NEAR, int TILE>
__global__ __launch_bounds__(kWinWG) __attribute__((amdgpu_waves_per_eu(8))) void k_assign_window(
    Img im, const float4* __restrict__ packed, const float* __restrict__ centres,
    const int* __restrict__ endpoints, int* __restrict__ labels, long long* __restrict__ acc,
    int* __restrict__ ctrl, WinLists wl, int R, float lambda, int tile0) {
    __shared__ WinShared sh;
    const int tid = threadIdx.x;
    if (ACCUM && tile0 == 0 && blockIdx.x == 0 && tid == 0) ctrl[kCtrlProjCount] = 0;
    const int W = im.W, H = im.H, K = im.nx * im.ny;
    Eqs eqs;
    eqs.img = packed;
    eqs.W = W;
    near_all(eqs);
    eqs.lambda = lambda;
    eqs.oml = 1.0f - lambda;
    eqs.gamma = im.gamma;
    eqs.spw = im.spw;
    const bool prune = im.prune != 0;
    const bool cut = prune && im.gamma <= 0x1p40f;
    const unsigned span = 2u * (unsigned)R;
    // a cluster's centre, endpoint and the corner of its window
    struct Cluster {
        float l, a, b, x, y;
        int ex, ey, wx, wy;
    };
    auto cluster = [&](int k) {
        const float* c = centres + 5LL * k;
        const int* e = endpoints + 2LL * k;
        Cluster v = {c[0], c[1], c[2], c[3], c[4], e[0], e[1], 0, 0};
        v.ex = min(max(v.ex, 0), W - 1);
        v.ey = min(max(v.ey, 0), H - 1);
        v.wx = round_coord(v.x, W - 1) - R;
        v.wy = round_coord(v.y, H - 1) - R;
        return v;
    };
    auto stage = [&](int j, const Cluster& v) {
        sh.cand[j][0] = make_float4(v.l, v.a, v.b, v.x);
        sh.cand[j][1] = make_float4(v.y, __int_as_float(v.ex), __int_as_float(v.ey), 0.0f);
        sh.box[j] = make_int2(v.wx, v.wy);
    };
    // pixel `id` of the tile, relative to its corner
    auto pixel_x = [](int id) { return (id & 7) + ((id >> 3) & 8); };
    auto pixel_y = [](int id) { return ((id >> 3) & 7) + ((id >> 4) & 8); };

    const int tile = tile0 + xcd_remap(blockIdx.x, gridDim.x);
    const int ty = tile / wl.tx;
    const int x0 = (tile - ty * wl.tx) * TILE, y0 = ty * TILE;
    const int x1 = min(x0 + TILE, W) - 1, y1 = min(y0 + TILE, H) - 1;
    const int px = x0 + pixel_x(tid), py = y0 + pixel_y(tid);
    const bool mine = tid < TILE * TILE && px < W && py < H;

    auto distance = [&](int j, float4 f, int qx, int qy, bool on, float thr) -> float {
        const float4 c0 = sh.cand[j][0], c1 = sh.cand[j][1];
        const float ck[5] = {c0.x, c0.y, c0.z, c0.w, c1.x};
        float A, B;
        return path_distance(eqs, ck, f, __float_as_int(c1.y), __float_as_int(c1.z), qx, qy, on,
                             thr, A, B);
    };
    // key of slot j: the upper 28 bits of the bound of D (see bound_keys) with the slot
    // below, kNoKey where the window does not contain the lane's pixel
    auto key_of = [&](int j, float4 fp) -> unsigned {
        const float4 c0 = sh.cand[j][0], c1 = sh.cand[j][1];
        const float dl = fp.x - c0.x, da = fp.y - c0.y, db = fp.z - c0.z;
        const float ex = (float)px - c0.w, ey = (float)py - c1.x;
        const float dcp = __builtin_fmaf(db, db, __builtin_fmaf(da, da, dl * dl));
        const float lb = __builtin_fmaf(ex * ex + ey * ey, im.spw, lambda * dcp);
        const int2 box = sh.box[j];
        const bool in = (unsigned)(px - box.x) <= span && (unsigned)(py - box.y) <= span;
        // (without the sign that a NaN may have)
        return in ? (__float_as_uint(lb) & 0x7ffffff0u) | (unsigned)j : kNoKey;
    };
    sh.win[tid] = ~0ULL;
    const int all = wl.count
        ? __builtin_amdgcn_readfirstlane(*const_cast<volatile int*>(&wl.count[tile])) : 0;
    const bool scan = !wl.count || all > wl.cap;
    if (ACCUM)
        for (int t = tid; t < kWinBatch * 6 * kBinCopies; t += kWinWG) (&sh.bins[0][0])[t] = 0ULL;
    int listed = all;
    // one turn, or one per kWinWG clusters (the same control in all waves)
    for (int k0 = 0;; k0 += kWinWG) {
        const bool last = !scan || k0 + kWinWG >= K;
        int k = k0 + tid, rank = 0;
        if (scan) {
            // the candidates among the lanes' clusters, in the order of the lanes
            const bool own = k < K;
            const Cluster v = cluster(own ? k : K - 1);
            const bool in = own && v.wx <= x1 && v.wx + 2 * R >= x0 && v.wy <= y1 && v.wy + 2 * R >= y0;
            const unsigned long long m = __ballot(in);
            if ((tid & 63) == 0) sh.count[tid >> 6] = __popcll(m);
            __syncthreads();
            rank = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            listed = 0;
            for (int w = 0; w < kWinWG / 64; ++w) {
                if (w == tid >> 6) rank += listed;
                listed += __builtin_amdgcn_readfirstlane(sh.count[w]);
            }
            if (in) {
                sh.ids[rank] = k;
                if (rank < kWinBatch) stage(rank, v);
            }
        } else {
            const int* list = wl.list + (long long)tile * wl.cap;
            for (int t = tid; t < listed; t += kWinWG) sh.unsorted[t] = list[t];
            __syncthreads();
            if (tid == 0) wl.count[tile] = 0;              // all waves have read it
            for (int t = tid; t < listed; t += kWinWG) {
                k = sh.unsorted[t];
                rank = 0;
                for (int u = 0; u < listed; ++u) rank += sh.unsorted[u] < k ? 1 : 0;
                sh.ids[rank] = k;
                if (rank < kWinBatch) stage(rank, cluster(k));
            }
        }
        __syncthreads();
        for (int b0 = 0; b0 < listed; b0 += kWinBatch) {
            const int n = min(listed - b0, kWinBatch);
            if (b0 > 0 && tid < n) stage(tid, cluster(sh.ids[b0 + tid]));
            if (tid == 0) sh.pairs = 0;
            __syncthreads();
            if (!NEAR) {
                Box box = {x0, y0, x1, y1};
                for (int j = 0; j < n; ++j)
                    box.add(__builtin_amdgcn_readfirstlane(__float_as_int(sh.cand[j][1].y)),
                            __builtin_amdgcn_readfirstlane(__float_as_int(sh.cand[j][1].z)));
                near_box(eqs, box);
            }
            if (mine) {
                const float4 fp = packed[py * W + px];
                unsigned long long win = sh.win[tid];
                // the four smallest keys, k1 < k2 < k3 < k4
                unsigned k1 = kNoKey, k2 = kNoKey, k3 = kNoKey, k4 = kNoKey;
                for (int j = 0; j < n; ++j) {
                    const unsigned key = key_of(j, fp);
                    k4 = med3(k3, k4, key);
                    k3 = med3(k2, k3, key);
                    k2 = med3(k1, k2, key);
                    k1 = min(k1, key);
                }
                if (k1 != kNoKey && !(prune && key_bound(k1) > win_threshold(win))) {
                    const int j = (int)(k1 & 15u);
                    const float D = distance(j, fp, px, py, false, 0.0f);
                    const unsigned long long found =
                        ((unsigned long long)__float_as_uint(D) << 32) | (unsigned)(b0 + j + 1);
                    if (found < win) sh.win[tid] = win = found;
                }
                const float thr = win_threshold(win);
                auto list = [&](unsigned key) {            // whether any lane's is
                    const bool more = key != kNoKey && !(prune && key_bound(key) > thr);
                    const unsigned long long m = __ballot(more);
                    if (m == 0ULL) return false;
                    const int at = wave_claim(&sh.pairs, m);
                    if (more) sh.list[at] = (unsigned short)(tid | ((key & 15u) << 8));
                    return true;
                };
                if (list(k2) && list(k3) && list(k4)) {
                    for (int j = 0; j < n; ++j) {
                        const unsigned key = key_of(j, fp);
                        list(key > k4 ? key : kNoKey);
                    }
                }
            }
            __syncthreads();
            const int pairs = __builtin_amdgcn_readfirstlane(sh.pairs);
            for (int i = tid; i < pairs; i += kWinWG) {
                const unsigned e = sh.list[i];
                const int id = (int)(e & 255u), j = (int)(e >> 8);
                const int qx = x0 + pixel_x(id), qy = y0 + pixel_y(id);
                const float D = distance(j, packed[qy * W + qx], qx, qy, cut, win_threshold(sh.win[id]));
                atomicMin(&sh.win[id], ((unsigned long long)__float_as_uint(D) << 32) |
                                           (unsigned)(b0 + j + 1));
            }
            __syncthreads();
        }
        if (last) break;
        const unsigned long long win = sh.win[tid];
        if (mine && win != ~0ULL && (unsigned)win != 0u) {
            labels[py * W + px] = sh.ids[(unsigned)win - 1u];
            sh.win[tid] = win & ~0xffffffffULL;
        }
        __syncthreads();
    }
    if (scan && wl.count && tid == 0) wl.count[tile] = 0;

    const unsigned long long win = sh.win[tid];
    const int slot = mine && win != ~0ULL ? (int)(unsigned)win - 1 : -1;
    const int p = py * W + px;
    if (slot >= 0) labels[p] = sh.ids[slot];
    if (!ACCUM) return;
    unsigned long long v[6] = {1ULL, (unsigned long long)px, (unsigned long long)py, 0ULL, 0ULL, 0ULL};
    if (mine) {
        const float4 f = packed[py * W + px];
        v[3] = (unsigned long long)to_fixed(f.x);
        v[4] = (unsigned long long)to_fixed(f.y);
        v[5] = (unsigned long long)to_fixed(f.z);
        if (slot < 0) {
            const int k = labels[p];
            if (k >= 0 && k < K)
                for (int c = 0; c < 6; ++c)
                    atomicAdd((unsigned long long*)(acc + kAccStride * (long long)k + c),
                              v[c]);
        }
    }
    // the bins hold kWinBatch candidates at a time
    const int cp = (tid ^ (tid >> 3)) & (kBinCopies - 1);
    for (int s0 = 0; s0 < listed; s0 += kWinBatch) {
        if (slot >= s0 && slot < s0 + kWinBatch) {
#pragma unroll
            for (int c = 0; c < 6; ++c) atomicAdd(&sh.bins[6 * (slot - s0) + c][cp], v[c]);
        }
        __syncthreads();
        const int j = tid / 6;
        if (j < min(listed - s0, kWinBatch)) {
            unsigned long long n = 0, sum = 0;
            for (int c = 0; c < kBinCopies; ++c) {
                n += sh.bins[6 * j][c];
                sum += sh.bins[tid][c];
            }
            if (n != 0ULL)
                atomicAdd((unsigned long long*)(acc + kAccStride * (long long)sh.ids[s0 + j] +
                                                (tid - 6 * j)),
                          sum);
        }
        if (s0 + kWinBatch >= listed) break;
        __syncthreads();
        for (int t = tid; t < kWinBatch * 6 * kBinCopies; t += kWinWG) (&sh.bins[0][0])[t] = 0ULL;
        __syncthreads();
    }
}

// ---------------------------------------------------------------- prepare

__global__ void k_prepare(long long n, const float* __restrict__ lab,
                          const float* __restrict__ contour, float sigma,
                          float4* __restrict__ packed) {
    const double s2 = (double)sigma * (double)sigma;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const double c = (double)contour[i];
        const float w = (float)(1.0 - exp(-(c * c) / s2));
        packed[i] = make_float4(lab[3 * i], lab[3 * i + 1], lab[3 * i + 2], w);
    }
}

__global__ void k_clear(long long* __restrict__ p, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = 0;
}

// ---------------------------------------------------------------- init

template <int WG>
__device__ __forceinline__ void init_cell(const Img& im, int cell, const float4* __restrict__ packed,
                                          int* __restrict__ labels, long long* __restrict__ acc) {
    __shared__ long long red[6][WG];
    const int tid = threadIdx.x;
    const int ci = cell / im.nx, cj = cell - ci * im.nx;
    const int x0 = cell_lo(cj, im.W, im.nx), x1 = cell_lo(cj + 1, im.W, im.nx);
    const int y0 = cell_lo(ci, im.H, im.ny), y1 = cell_lo(ci + 1, im.H, im.ny);
    const int cw = x1 - x0, P = cw * (y1 - y0);
    long long s[6] = {0, 0, 0, 0, 0, 0};
    for (int t = tid; t < P; t += WG) {
        const int r = t / cw;
        const int x = x0 + (t - r * cw), y = y0 + r;
        const long long p = (long long)y * im.W + x;
        const float4 f = packed[im.pix + p];
        labels[im.pix + p] = cell;
        s[0] += 1; s[1] += x; s[2] += y;
        s[3] += to_fixed(f.x); s[4] += to_fixed(f.y); s[5] += to_fixed(f.z);
    }
    for (int v = 0; v < 6; ++v) red[v][tid] = s[v];
    __syncthreads();
    for (int h = WG / 2; h > 0; h >>= 1) {
        if (tid < h)
            for (int v = 0; v < 6; ++v) red[v][tid] += red[v][tid + h];
        __syncthreads();
    }
    if (tid < 6) acc[kAccStride * (long long)(im.sp + cell) + tid] = red[tid][0];
    __syncthreads();
}

template <int WG>
__global__ __launch_bounds__(WG) void k_init_cells(Img im, const float4* __restrict__ packed,
                                                   int* __restrict__ labels,
                                                   long long* __restrict__ acc) {
    init_cell<WG>(im, blockIdx.x, packed, labels, acc);
}

template <int WG>
__global__ __launch_bounds__(WG) void k_init_cells_batched(const Img* __restrict__ imgs,
                                                           const int* __restrict__ cell_start,
                                                           int n_img, const float4* packed,
                                                           int* labels, long long* acc) {
    const int i = find_image(cell_start, n_img, blockIdx.x);
    init_cell<WG>(imgs[i], blockIdx.x - cell_start[i], packed, labels, acc);
}

// ---------------------------------------------------------------- update from labels

// Integer sums of the update for caller-supplied labels, which need not be grid
// neighbours.  One workgroup per grid cell
// accumulates into a small LDS table keyed by label (open addressing, key
// claimed with a compare-and-swap); a label that finds no free slot goes
// straight to the global sums.  The sums are integers, so the result does
// not depend on the order of the atomics.
constexpr int kAccSlots = 32;

template <int WG>
__global__ __launch_bounds__(WG) void k_accumulate(Img im, const float* __restrict__ lab,
                                                   const int* __restrict__ labels,
                                                   long long* __restrict__ acc) {
    __shared__ int keys[kAccSlots];
    // [slot * 6 + sum][copy]: the lanes of a wave mostly carry one label, so
    // each adds to copy (t ^ t >> 3) mod kBinCopies (see ItemShared)
    __shared__ unsigned long long bins[kAccSlots * 6][kBinCopies];
    const int tid = threadIdx.x;
    const int cell = blockIdx.x;
    const int ci = cell / im.nx, cj = cell - ci * im.nx;
    const int x0 = cell_lo(cj, im.W, im.nx), x1 = cell_lo(cj + 1, im.W, im.nx);
    const int y0 = cell_lo(ci, im.H, im.ny), y1 = cell_lo(ci + 1, im.H, im.ny);
    const int K = im.nx * im.ny;
    for (int t = tid; t < kAccSlots * 6 * kBinCopies; t += WG) (&bins[0][0])[t] = 0ULL;
    for (int t = tid; t < kAccSlots; t += WG) keys[t] = -1;
    const int cp = (tid ^ (tid >> 3)) & (kBinCopies - 1);
    __syncthreads();
    const int cw = x1 - x0, P = cw * (y1 - y0);
    for (int t = tid; t < P; t += WG) {
        const int r = t / cw;
        const int x = x0 + (t - r * cw), y = y0 + r;
        const long long p = (long long)y * im.W + x;
        const int k = labels[p];
        if (k < 0 || k >= K) continue;
        const float3 f = make_float3(lab[3 * p], lab[3 * p + 1], lab[3 * p + 2]);
        const unsigned long long v[6] = {1ULL, (unsigned long long)x, (unsigned long long)y,
                                         (unsigned long long)to_fixed(f.x),
                                         (unsigned long long)to_fixed(f.y),
                                         (unsigned long long)to_fixed(f.z)};
        int slot = -1;
        for (int probe = 0, h = k & (kAccSlots - 1); probe < kAccSlots;
             ++probe, h = (h + 1) & (kAccSlots - 1)) {
            const int cur = keys[h];
            if (cur == k) { slot = h; break; }
            if (cur == -1) {
                const int old = atomicCAS(&keys[h], -1, k);
                if (old == -1 || old == k) { slot = h; break; }
            }
        }
        if (slot >= 0) {
            for (int q = 0; q < 6; ++q) atomicAdd(&bins[slot * 6 + q][cp], v[q]);
        } else {
            for (int q = 0; q < 6; ++q)
                atomicAdd((unsigned long long*)(acc + kAccStride * (long long)(im.sp + k) + q), v[q]);
        }
    }
    __syncthreads();
    for (int t = tid; t < kAccSlots * 6; t += WG) {
        const int slot = t / 6, q = t - 6 * (t / 6);
        const int k = keys[slot];
        unsigned long long n = 0, v = 0;
        for (int c = 0; c < kBinCopies; ++c) {
            n += bins[slot * 6][c];
            v += bins[t][c];
        }
        if (k >= 0 && n != 0ULL)
            atomicAdd((unsigned long long*)(acc + kAccStride * (long long)(im.sp + k) + q), v);
    }
}

// ---------------------------------------------------------------- finalize

// Superpixel k's centre, barycenter and count from its sums (which it
// clears); the endpoint is the rounded barycenter when that pixel is one of
// k's own or projection is off.  Returns true when the projection has to
// move the endpoint instead (then xk, yk, cnt are what it needs).
__device__ __forceinline__ bool finalize_core(const Img& im, int k, float* __restrict__ centres,
                                              int* __restrict__ endpoints,
                                              int* __restrict__ counts,
                                              long long* __restrict__ acc,
                                              const int* __restrict__ labels, bool project,
                                              float& xk, float& yk, int& cnt_out) {
    long long* a = acc + kAccStride * (long long)(im.sp + k);
    const long long cnt = a[0];
    bool move = false;
    if (cnt > 0) {
        const double n = (double)cnt;
        float* c = centres + 5LL * (im.sp + k);
        c[0] = (float)(((double)a[3] / n) * kFixInv);
        c[1] = (float)(((double)a[4] / n) * kFixInv);
        c[2] = (float)(((double)a[5] / n) * kFixInv);
        xk = (float)((double)a[1] / n);
        yk = (float)((double)a[2] / n);
        c[3] = xk;
        c[4] = yk;
        const int ex = round_coord(xk, im.W - 1), ey = round_coord(yk, im.H - 1);
        if (!project || labels[im.pix + (long long)ey * im.W + ex] == k) {
            endpoints[2LL * (im.sp + k)] = ex;
            endpoints[2LL * (im.sp + k) + 1] = ey;
        } else {
            move = true;
        }
    }
    counts[im.sp + k] = (int)cnt;
    cnt_out = (int)cnt;
    for (int v = 0; v < 6; ++v) a[v] = 0;
    return move;
}

__device__ __forceinline__ void finalize_one(const Img& im, int k, float* __restrict__ centres,
                                             int* __restrict__ endpoints,
                                             int* __restrict__ counts,
                                             long long* __restrict__ acc,
                                             const int* __restrict__ labels, int* ctrl,
                                             int* plist, bool project) {
    float xk, yk;
    int cnt;
    if (finalize_core(im, k, centres, endpoints, counts, acc, labels, project, xk, yk, cnt)) {
        const int slot = atomicAdd(&ctrl[kCtrlProjCount], 1);
        plist[slot] = im.sp + k;
    }
}

__global__ void k_finalize(Img im, float* centres, int* endpoints, int* counts, long long* acc,
                           const int* labels, int* ctrl, int* plist, int project) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < im.nx * im.ny)
        finalize_one(im, k, centres, endpoints, counts, acc, labels, ctrl, plist, project != 0);
}

__global__ void k_finalize_batched(const Img* __restrict__ imgs, const int* __restrict__ sp_start,
                                   int n_img, int total, float* centres, int* endpoints,
                                   int* counts, long long* acc, const int* labels, int* ctrl,
                                   int* plist, int project) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const int i = find_image(sp_start, n_img, g);
    const Img im = imgs[i];
    finalize_one(im, g - im.sp, centres, endpoints, counts, acc, labels, ctrl, plist,
                 project != 0);
}

// ---------------------------------------------------------------- projection

// Minimum key and member count over the workgroup: shuffles within each
// wave, then one LDS slot per wave (two barriers in all).
template <int WG>
__device__ __forceinline__ void block_min_sum(unsigned long long& key, int& cnt) {
    __shared__ unsigned long long rk[WG / 64];
    __shared__ int rc[WG / 64];
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long k2 = __shfl_xor(key, o, 64);
        key = k2 < key ? k2 : key;
        cnt += __shfl_xor(cnt, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        rk[threadIdx.x >> 6] = key;
        rc[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    key = rk[0];
    cnt = rc[0];
    for (int q = 1; q < WG / 64; ++q) {
        key = rk[q] < key ? rk[q] : key;
        cnt += rc[q];
    }
    __syncthreads();   // the slots are reused by the next reduction
}

// Squared FP32 distance to (xk, yk) in the high word, raster index in the
// low word: the minimum key is the nearest pixel, ties to the lowest index.
__device__ __forceinline__ unsigned long long proj_key(int x, int y, int W, float xk, float yk) {
    const float dx = (float)x - xk;
    const float dy = (float)y - yk;
    const float d = dx * dx + dy * dy;
    return ((unsigned long long)__float_as_uint(d) << 32) | (unsigned)(y * W + x);
}

// Nearest member of cluster k (key of proj_key) and the number of members
// inside [X0, X1) x [Y0, Y1), reduced over the workgroup; four independent
// label loads in flight per thread per round.
template <int WG>
__device__ void scan_region(const int* __restrict__ lb, int W, int k, int X0, int X1, int Y0,
                            int Y1, float xk, float yk, unsigned long long& best, int& found) {
    const int tid = threadIdx.x;
    const int bw = X1 - X0, area = bw * (Y1 - Y0);
    best = ~0ULL;
    found = 0;
    // element e = r * bw + c; lanes step by WG elements = (dr rows, dc
    // columns), eight loads in flight per trip (the minimum over packed keys
    // does not depend on the order)
    constexpr int kU = 8;
    const int dr = WG / bw, dc = WG - dr * bw;
    int r = tid / bw, c = tid - r * bw;
    for (int e0 = tid; e0 < area; e0 += kU * WG) {
        int lbl[kU], xs[kU], ys[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            xs[u] = X0 + c;
            ys[u] = Y0 + r;
            lbl[u] = e0 + u * WG < area ? lb[(long long)ys[u] * W + xs[u]] : -1;
            c += dc;
            const bool wrap = c >= bw;
            c -= wrap ? bw : 0;
            r += dr + (wrap ? 1 : 0);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (lbl[u] == k) {
                ++found;
                const unsigned long long key = proj_key(xs[u], ys[u], W, xk, yk);
                best = key < best ? key : best;
            }
        }
    }
    block_min_sum<WG>(best, found);
}

// Eq. (4) for one queued cluster: the argmin over all its members.  First the
// square of half-width kNearHalf around the rounded barycenter: a member there
// whose squared distance is below kNearHalf^2 is the nearest, as every pixel
// outside is at least kNearHalf + 1/2 - ulp away (coordinates up to 2^22, ulp
// 1/4).  Else regions of growing size until every member (counts) was seen:
// the 3x3 cell block around its grid cell (where the grid form's labels
// lie), then the square of half-width 2R + 2 around the rounded barycenter
// (the window form: members lie within R of the previous barycenter, which
// lies within R of the new one), then the whole image (any labels).
//
// What bounds it: the latency of the label loads.  1920x1080, k = 2000, per
// launch of k_finalize_project: 9.1 us with the 9400-pixel block always scanned
// and 15.5 in the window form, whose members leave it; 6.1 and 6.2 now (the latter
// with the next pass's lists); the 64-image batch: 135 to 95 us.  With a half-width
// of 16 some clusters of nearly every launch still scan the block: 7.5.
constexpr int kNearHalf = 22;   // 45 x 45 pixels: one trip of 256 lanes' 8 loads

template <int WG>
__device__ void project_at(const Img& im, int k, float xk, float yk, int count,
                           const int* __restrict__ labels, int* __restrict__ endpoints) {
    const int W = im.W, H = im.H;
    const int* lb = labels + im.pix;
    const int cx = round_coord(xk, W - 1), cy = round_coord(yk, H - 1);
    unsigned long long best = ~0ULL;
    int found = 0;
    bool done = false;
    if (max(W, H) <= 1 << 22) {
        scan_region<WG>(lb, W, k, max(cx - kNearHalf, 0), min(cx + kNearHalf + 1, W),
                        max(cy - kNearHalf, 0), min(cy + kNearHalf + 1, H), xk, yk, best, found);
        done = found == count ||
               (found > 0 && __uint_as_float((unsigned)(best >> 32)) < (float)(kNearHalf * kNearHalf));
    }
    if (!done) {                                   // uniform: reduced over the workgroup
        const int ci = k / im.nx, cj = k - ci * im.nx;
        scan_region<WG>(lb, W, k, cell_lo(max(cj - 1, 0), W, im.nx),
                        cell_lo(min(cj + 2, im.nx), W, im.nx), cell_lo(max(ci - 1, 0), H, im.ny),
                        cell_lo(min(ci + 2, im.ny), H, im.ny), xk, yk, best, found);
        if (found < count) {
            const int h = 2 * im.rad + 2;
            scan_region<WG>(lb, W, k, max(cx - h, 0), min(cx + h + 1, W), max(cy - h, 0),
                            min(cy + h + 1, H), xk, yk, best, found);
            if (found < count) scan_region<WG>(lb, W, k, 0, W, 0, H, xk, yk, best, found);
        }
    }
    if (threadIdx.x == 0 && best != ~0ULL) {
        const unsigned idx = (unsigned)(best & 0xffffffffULL);
        endpoints[2LL * (im.sp + k)] = (int)(idx % (unsigned)W);
        endpoints[2LL * (im.sp + k) + 1] = (int)(idx / (unsigned)W);
    }
}

template <int WG>
__device__ void project_one(const Img& im, int k, const float* __restrict__ centres,
                            const int* __restrict__ counts, const int* __restrict__ labels,
                            int* __restrict__ endpoints) {
    project_at<WG>(im, k, centres[5LL * (im.sp + k) + 3], centres[5LL * (im.sp + k) + 4],
                   counts[im.sp + k], labels, endpoints);
}

// Finalize and projection in one pass, a workgroup per superpixel: thread 0
// takes the superpixel's sums, and when its rounded barycenter is not one of
// its pixels the workgroup moves the endpoint to the nearest member at once
// (no queue, no second launch; projecting k reads only k's own centre and
// count and the labels).
template <int WG>
__global__ __launch_bounds__(WG) void k_finalize_project(Img im, float* centres, int* endpoints,
                                                         int* counts, long long* acc,
                                                         const int* labels, int R, WinLists wl) {
    __shared__ float sx, sy;
    __shared__ int scnt, smove;
    const int k = blockIdx.x;
    if (threadIdx.x == 0) {
        float xk = 0.0f, yk = 0.0f;
        int cnt = 0;
        smove = finalize_core(im, k, centres, endpoints, counts, acc, labels, true, xk, yk, cnt)
                    ? 1 : 0;
        if (wl.count && cnt == 0) {                // an empty cluster stays where it was
            xk = centres[5LL * (im.sp + k) + 3];
            yk = centres[5LL * (im.sp + k) + 4];
        }
        sx = xk;
        sy = yk;
        scnt = cnt;
    }
    __syncthreads();
    if (wl.count && threadIdx.x < 64) add_to_tiles(im, k, sx, sy, R, wl);
    if (smove) project_at<WG>(im, k, sx, sy, scnt, labels, endpoints);   // uniform
}

// The same over a ragged batch, a workgroup per superpixel of the batch.
template <int WG>
__global__ __launch_bounds__(WG) void k_finalize_project_batched(const Img* __restrict__ imgs,
                                                                 const int* __restrict__ sp_start,
                                                                 int n_img, float* centres,
                                                                 int* endpoints, int* counts,
                                                                 long long* acc,
                                                                 const int* labels) {
    __shared__ float sx, sy;
    __shared__ int scnt, smove, simg;
    const int g = blockIdx.x;
    if (threadIdx.x == 0) {
        const int i = find_image(sp_start, n_img, g);
        float xk = 0.0f, yk = 0.0f;
        int cnt = 0;
        smove = finalize_core(imgs[i], g - imgs[i].sp, centres, endpoints, counts, acc, labels,
                              true, xk, yk, cnt) ? 1 : 0;
        sx = xk;
        sy = yk;
        scnt = cnt;
        simg = i;
    }
    __syncthreads();
    if (smove) {                                   // uniform
        const Img im = imgs[simg];
        project_at<WG>(im, g - im.sp, sx, sy, scnt, labels, endpoints);
    }
}

template <int WG>
__global__ __launch_bounds__(WG) void k_project(Img im, const float* centres, const int* counts,
                                                const int* labels, int* endpoints,
                                                const int* ctrl, const int* plist) {
    const int n = ctrl[kCtrlProjCount];
    for (int i = blockIdx.x; i < n; i += gridDim.x)
        project_one<WG>(im, plist[i] - im.sp, centres, counts, labels, endpoints);
}

// Small host tables (image descriptors) reach the device as kernel
// arguments, so no host buffer has to outlive the call and the copy can be
// captured into a graph.
struct ByteChunk {
    unsigned nbytes;
    unsigned char data[3072];
};

__global__ void k_write_bytes(unsigned char* __restrict__ dst, ByteChunk c) {
    for (unsigned i = threadIdx.x; i < c.nbytes; i += blockDim.x) dst[i] = c.data[i];
}

constexpr int kSmallWG = 256;
constexpr int kProjectWG = 1024;
constexpr int kProjectBlocks = 256;
// Workgroup of the finalize + projection pass: 256 lanes, or 1024 where a
// superpixel's 3x3 cell block holds more than kWideProjectPixels pixels (the
// coarse scales of the multi-scale batch: one projection then scans most of
// the image, and its workgroup alone bounds the pass).
constexpr int kFinProjectWG = 256;
constexpr int kWideProjectWG = 1024;
constexpr long long kWideProjectPixels = 32768;

}  // namespace

bool near_image(const Img& im) { return !im.far && im.W + im.H < 46340; }

void finish_img(Img& im) {
    const long long W = im.W, H = im.H, nx = im.nx, ny = im.ny, K = nx * ny;
    im.far = W * H >= (1LL << 28);
    im.dnx = fast_div(nx, nx * (W + 1));
    im.dny = fast_div(ny, ny * (H + 1));
    im.dspl = fast_div(im.spl, std::max(K, (W / nx + 1) * (H / ny + 1) / 64 + 2) * im.spl);
    const long long tw = (nx + im.strips - 1) / im.strips;
    im.dcol = fast_div(tw, tw * ny);
    im.dstrip = fast_div(tw * ny, K);
    im.dlast = fast_div(nx % tw ? nx % tw : tw, tw * ny);
    for (int i = 0; i < 2; ++i) {
        const long long ch = H / ny + i, cw = W / nx + 1;
        im.dper[i] = fast_div(8 * ch, cw * ch);
    }
}

int launch_write_bytes(void* dst, const void* src, size_t n, hipStream_t s) {
    const unsigned char* in = static_cast<const unsigned char*>(src);
    unsigned char* out = static_cast<unsigned char*>(dst);
    for (size_t off = 0; off < n; off += sizeof(ByteChunk::data)) {
        ByteChunk c;
        c.nbytes = (unsigned)std::min(n - off, sizeof(c.data));
        std::copy(in + off, in + off + c.nbytes, c.data);
        hipLaunchKernelGGL(k_write_bytes, dim3(1), dim3(256), 0, s, out + off, c);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int launch_prepare(long long n, const float* lab, const float* contour, float sigma,
                   float4* packed, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const long long blocks = std::min<long long>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_prepare, dim3((unsigned)blocks), dim3(256), 0, s, n, lab, contour, sigma,
                       packed);
    return hipGetLastError();
}

int launch_clear(long long* p, long long n_words, hipStream_t s) {
    if (n_words <= 0) return hipSuccess;
    const long long blocks = std::min<long long>((n_words + 255) / 256, 4096);
    hipLaunchKernelGGL(k_clear, dim3((unsigned)blocks), dim3(256), 0, s, p, n_words);
    return hipGetLastError();
}

int launch_init_cells(const Img& im, const float4* packed, int* labels, long long* acc,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_init_cells<kSmallWG>, dim3(im.nx * im.ny), dim3(kSmallWG), 0, s, im,
                       packed, labels, acc);
    return hipGetLastError();
}

int launch_init_cells_batched(const Img* imgs, const int* cell_start, int n_img, int total_cells,
                              const float4* packed, int* labels, long long* acc, hipStream_t s) {
    hipLaunchKernelGGL(k_init_cells_batched<kSmallWG>, dim3(total_cells), dim3(kSmallWG), 0, s,
                       imgs, cell_start, n_img, packed, labels, acc);
    return hipGetLastError();
}

template <int WG, bool ACCUM, Walk WALK>
static int launch_assign_t(const Img& im, const float4* packed, const float* centres,
                           const int* endpoints, int* labels, long long* acc, int* ctrl,
                           float lambda, hipStream_t s) {
    const auto kernel = near_image(im) ? k_assign<WG, ACCUM, true, WALK> : k_assign<WG, ACCUM, false, WALK>;
    hipLaunchKernelGGL(kernel, dim3(im.nx * im.ny * im.spl), dim3(WG), 0, s, im, packed, centres,
                       endpoints, labels, acc, ctrl, lambda);
    return hipGetLastError();
}

template <int WG, bool ACCUM>
static int launch_assign_wg(const Img& im, const float4* packed, const float* centres,
                            const int* endpoints, int* labels, long long* acc, int* ctrl,
                            float lambda, hipStream_t s) {
    const Walk walk = walk_of(im.prune, (long long)im.W * im.H, im.nx * im.ny);
    const auto launch = walk == Walk::kAll    ? launch_assign_t<WG, ACCUM, Walk::kAll>
                        : walk == Walk::kMany ? launch_assign_t<WG, ACCUM, Walk::kMany>
                                              : launch_assign_t<WG, ACCUM, Walk::kPairs>;
    return launch(im, packed, centres, endpoints, labels, acc, ctrl, lambda, s);
}

int launch_assign(const Img& im, const float4* packed, const float* centres,
                  const int* endpoints, int* labels, long long* acc, int* ctrl, float lambda,
                  bool accumulate, const Tuning& t, hipStream_t s) {
    const auto launch =
        t.wg == 1024  ? accumulate ? launch_assign_wg<1024, true> : launch_assign_wg<1024, false>
        : t.wg == 512 ? accumulate ? launch_assign_wg<512, true> : launch_assign_wg<512, false>
                      : accumulate ? launch_assign_wg<256, true> : launch_assign_wg<256, false>;
    return launch(im, packed, centres, endpoints, labels, acc, ctrl, lambda, s);
}

template <int WG, Walk WALK>
static int launch_assign_batched_t(const Img* imgs, const int* item_start, int n_img, int longest_run,
                                   const float4* packed, const float* centres, const int* endpoints,
                                   int* labels, long long* acc, int* ctrl, float lambda, bool near,
                                   hipStream_t s) {
    const auto kernel = near ? k_assign_batched<WG, true, WALK> : k_assign_batched<WG, false, WALK>;
    // (a launch holds below 2^32 lanes)
    for (int h0 = 0; h0 < longest_run; h0 += 1 << 18) {
        const unsigned n = (unsigned)std::min(longest_run - h0, 1 << 18);
        hipLaunchKernelGGL(kernel, dim3(8u * n), dim3(WG), 0, s, imgs, item_start, n_img, packed,
                           centres, endpoints, labels, acc, ctrl, lambda, h0);
    }
    return hipGetLastError();
}

template <int WG>
static int launch_assign_batched_wg(const Img* imgs, const int* item_start, int n_img, int longest_run,
                                    const float4* packed, const float* centres, const int* endpoints,
                                    int* labels, long long* acc, int* ctrl, float lambda, bool near,
                                    Walk walk, hipStream_t s) {
    const auto launch = walk == Walk::kAll    ? launch_assign_batched_t<WG, Walk::kAll>
                        : walk == Walk::kMany ? launch_assign_batched_t<WG, Walk::kMany>
                                              : launch_assign_batched_t<WG, Walk::kPairs>;
    return launch(imgs, item_start, n_img, longest_run, packed, centres, endpoints, labels, acc, ctrl,
                  lambda, near, s);
}

int launch_assign_batched(const Img* imgs, const int* item_start, int n_img, int longest_run,
                          const float4* packed, const float* centres, const int* endpoints,
                          int* labels, long long* acc, int* ctrl, float lambda, const Tuning& t,
                          bool near, Walk walk, hipStream_t s) {
    const auto launch = t.wg == 1024 ? launch_assign_batched_wg<1024>
                        : t.wg == 512 ? launch_assign_batched_wg<512> : launch_assign_batched_wg<256>;
    return launch(imgs, item_start, n_img, longest_run, packed, centres, endpoints, labels, acc, ctrl,
                  lambda, near, walk, s);
}

// Side of the window form's tiles: 8 where that gives no more than kWinSmall of them, 4
// per compute unit (300x200, k = 300, 925 tiles: 186 us in 10 iterations, 198 with tiles of
// 16; 189x117, k = 1000, 231 and 355; 481x321, 2500 tiles, no difference).
static int win_tile(int W, int H) {
    const long long tiles = (long long)((W + kWinTile - 1) / kWinTile) * ((H + kWinTile - 1) / kWinTile);
    return 4 * tiles <= kWinSmall ? 8 : kWinTile;
}

static long long win_tiles(int W, int H) {
    const int t = win_tile(W, H);
    return (long long)((W + t - 1) / t) * ((H + t - 1) / t);
}

// 8 W H bytes, but at least 256, hold the counts and a list of at least 12 ids per tile
// (W = 33, H = 1, tiles of 8; a row of tiles of 16, one pixel high, has 31).
//
// No lists (count null) for up to kWinWG clusters: every tile tests them all in one
// turn, which takes no longer than reading a list does, and nothing has to make them
// (97x61, 30 clusters, 10 iterations: 172 us with lists, 165 without).
static WinLists win_lists(const Img& im, void* mem) {
    WinLists wl = {};
    wl.tile = win_tile(im.W, im.H);
    wl.tx = (im.W + wl.tile - 1) / wl.tile;
    wl.tiles = (int)win_tiles(im.W, im.H);
    const long long words = std::max(2LL * im.W * im.H, 64LL);
    if (!mem || im.nx * im.ny <= kWinWG) return wl;
    wl.cap = (int)std::min<long long>(words / wl.tiles - 1, kWinIds);
    wl.count = static_cast<int*>(mem);
    wl.list = wl.count + wl.tiles;
    return wl;
}

long long window_count_words(int W, int H) { return (win_tiles(W, H) + 1) / 2; }

int launch_assign_window(const Img& im, const float4* packed, const float* centres,
                         const int* endpoints, int* labels, long long* acc, int* ctrl, void* lists,
                         int R, float lambda, bool accumulate, bool listed, hipStream_t s) {
    const WinLists wl = win_lists(im, lists);
    const int K = im.nx * im.ny;
    const bool near = near_image(im), small = wl.tile == 8;
    if (wl.count && !listed)
        hipLaunchKernelGGL(k_window_lists, dim3((K + 3) / 4), dim3(256), 0, s, im, centres, R, wl);
    const int tiles = wl.tiles;
    // at most 2^22 workgroups a launch (an image one pixel high may have 2^27 tiles)
    for (int t0 = 0; t0 < tiles; t0 += 1 << 22) {
        const dim3 grid((unsigned)std::min(tiles - t0, 1 << 22));
        const auto kernel =
            small        ? accumulate ? near ? k_assign_window<true, true, 8> : k_assign_window<true, false, 8>
                           : near ? k_assign_window<false, true, 8> : k_assign_window<false, false, 8>
            : accumulate ? near ? k_assign_window<true, true, kWinTile> : k_assign_window<true, false, kWinTile>
                         : near ? k_assign_window<false, true, kWinTile>
                                : k_assign_window<false, false, kWinTile>;
        hipLaunchKernelGGL(kernel, grid, dim3(kWinWG), 0, s, im, packed, centres, endpoints, labels,
                           acc, ctrl, wl, R, lambda, t0);
    }
    return hipGetLastError();
}

int launch_accumulate(const Img& im, const float* lab, const int* labels, long long* acc,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_accumulate<kSmallWG>, dim3(im.nx * im.ny), dim3(kSmallWG), 0, s, im, lab,
                       labels, acc);
    return hipGetLastError();
}

int launch_finalize(const Img& im, float* centres, int* endpoints, int* counts, long long* acc,
                    const int* labels, int* ctrl, int* plist, bool project, hipStream_t s) {
    const int K = im.nx * im.ny;
    hipLaunchKernelGGL(k_finalize, dim3((K + 255) / 256), dim3(256), 0, s, im, centres,
                       endpoints, counts, acc, labels, ctrl, plist, project ? 1 : 0);
    return hipGetLastError();
}

int launch_finalize_batched(const Img* imgs, const int* sp_start, int n_img, int total_sp,
                            float* centres, int* endpoints, int* counts, long long* acc,
                            const int* labels, int* ctrl, int* plist, bool project,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_finalize_batched, dim3((total_sp + 255) / 256), dim3(256), 0, s, imgs,
                       sp_start, n_img, total_sp, centres, endpoints, counts, acc, labels, ctrl,
                       plist, project ? 1 : 0);
    return hipGetLastError();
}

long long block_pixels(int W, int H, int nx, int ny) {
    return 9LL * ((W + nx - 1) / nx) * ((H + ny - 1) / ny);
}

int launch_finalize_project(const Img& im, float* centres, int* endpoints, int* counts,
                            long long* acc, const int* labels, void* lists, int R, hipStream_t s) {
    const WinLists wl = win_lists(im, lists);
    if (block_pixels(im.W, im.H, im.nx, im.ny) > kWideProjectPixels)
        hipLaunchKernelGGL(k_finalize_project<kWideProjectWG>, dim3(im.nx * im.ny),
                           dim3(kWideProjectWG), 0, s, im, centres, endpoints, counts, acc, labels, R,
                           wl);
    else
        hipLaunchKernelGGL(k_finalize_project<kFinProjectWG>, dim3(im.nx * im.ny),
                           dim3(kFinProjectWG), 0, s, im, centres, endpoints, counts, acc, labels, R,
                           wl);
    return hipGetLastError();
}

int launch_finalize_project_batched(const Img* imgs, const int* sp_start, int n_img,
                                    int total_sp, long long max_block_px, float* centres,
                                    int* endpoints, int* counts, long long* acc, const int* labels,
                                    hipStream_t s) {
    if (max_block_px > kWideProjectPixels)
        hipLaunchKernelGGL(k_finalize_project_batched<kWideProjectWG>, dim3(total_sp),
                           dim3(kWideProjectWG), 0, s, imgs, sp_start, n_img, centres, endpoints,
                           counts, acc, labels);
    else
        hipLaunchKernelGGL(k_finalize_project_batched<kFinProjectWG>, dim3(total_sp),
                           dim3(kFinProjectWG), 0, s, imgs, sp_start, n_img, centres, endpoints,
                           counts, acc, labels);
    return hipGetLastError();
}

int launch_project(const Img& im, const float* centres, const int* counts, const int* labels,
                   int* endpoints, const int* ctrl, const int* plist, hipStream_t s) {
    hipLaunchKernelGGL(k_project<kProjectWG>, dim3(kProjectBlocks), dim3(kProjectWG), 0, s, im,
                       centres, counts, labels, endpoints, ctrl, plist);
    return hipGetLastError();
}

}  // namespace scalp
