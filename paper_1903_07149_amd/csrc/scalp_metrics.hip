// scalp_metrics.hip -- superpixel quality metrics of Sec. III-A.2 on the GPU:
// boundary recall (Eq. (5)), achievable segmentation accuracy (Eq. (6)),
// undersegmentation error (Eq. (7)) and compactness (Eq. (8)) of a label map
// against a ground-truth partition.
//
//   k_metric_pixels  one pass over the pixels, a wave per 64 columns by 4 rows
//                    (every row loaded once, all in flight together; left and
//                    right neighbours from the lanes beside): the overlap
//                    table |S_k n G_i| and the perimeter of every superpixel
//                    in pixel edges (4-connectivity, image border included),
//                    gathered per run of equal (k, i) in a row into a hash
//                    table in LDS and added to global memory once per pair
//                    and block; and two boundary bitmaps, one 64-bit word per
//                    wave and row (bit b = pixel 64 w + b).
//   k_metric_rest    thread per bitmap word: boundary-recall counts
//                    (ground-truth boundary pixels, those with a superpixel
//                    boundary pixel at distance < epsilon, superpixel
//                    boundary pixels) from the superpixel bitmap dilated
//                    over the epsilon disc with word shifts; one partial sum
//                    per workgroup;
//                    and, in the launch's other blocks, wave per superpixel:
//                    area, largest overlap, UE row sum (integers) and the CO
//                    term 4 pi A^2 / P^2 (FP64).
//   k_metric_final   one workgroup: fixed-order sums of the rows and of the
//                    recall partials, so the result does not depend on the
//                    order of the atomics.
#include <algorithm>

#include "scalp_device.h"

namespace scalp {
namespace {

using namespace dev;

constexpr int kMetricWG = 256;

struct MetricGeom {
    int W, H, K, R;
    int Wq;         // bitmap words per row, ceil(W / 64)
    int nrb;        // recall blocks (partial sums)
    int keep;       // 1: the pair table holds all pairs there are
    int r;          // neighbourhood half-width for boundary recall
    float eps2;     // epsilon^2
};

// Pair table of one workgroup: open addressing over kPairSlots entries in
// LDS, key k * R + i (< 2^30, so kEmpty never collides with a key).
constexpr int kPairBits = 9, kPairSlots = 1 << kPairBits;
constexpr unsigned kEmpty = 0xffffffffu;

struct PairTable {
    unsigned key[kPairSlots], cnt[kPairSlots], edge[kPairSlots];
};

// One row of a wave: lane `head` begins a run of equal (k, i) (or of lanes with
// !ok) that ends before the next head.  Every head with ok adds its run's pixels
// and edge counts to the workgroup's table, all heads at once.  e0..e2 are the
// bit planes of the lanes' edge counts (0..4), so a run's edge sum is three
// masked popcounts.  A full table sends the pair straight to global memory.
__device__ __forceinline__ void row_count(PairTable& pt, unsigned* __restrict__ table,
                                          unsigned* __restrict__ perim, int R, bool ok, bool head,
                                          int k, int i, unsigned e) {
    const int lane = threadIdx.x & 63;
    const unsigned long long heads = __ballot(head);
    const unsigned long long e0 = __ballot(e & 1u), e1 = __ballot(e & 2u), e2 = __ballot(e & 4u);
    if (!head || !ok) return;
    // bits lane .. the next head (exclusive); without one, to the end
    const unsigned long long above = heads & ~((2ULL << lane) - 1ULL);
    const unsigned long long m = ((above & (0ULL - above)) - 1ULL) & ~((1ULL << lane) - 1ULL);
    const unsigned n = (unsigned)__popcll(m);
    const unsigned edges = (unsigned)(__popcll(e0 & m) + 2 * __popcll(e1 & m) + 4 * __popcll(e2 & m));
    const unsigned key = (unsigned)k * (unsigned)R + (unsigned)i;
    unsigned h = (key * 2654435761u) >> (32 - kPairBits);
    for (int probe = 0; probe < kPairSlots; ++probe) {
        unsigned old = *const_cast<volatile unsigned*>(&pt.key[h]);
        if (old == kEmpty) old = atomicCAS(&pt.key[h], kEmpty, key);
        if (old == kEmpty || old == key) {
            atomicAdd(&pt.cnt[h], n);
            if (edges) atomicAdd(&pt.edge[h], edges);
            return;
        }
        h = (h + 1) & (kPairSlots - 1);
    }
    atomicAdd(&table[key], n);
    if (edges) atomicAdd(&perim[k], edges);
}

// The lane below's (DPP wave_shr:1) or above's (wave_shl:1) value; the wave's
// first or last lane gets `edge`.
template <int CTRL>
__device__ __forceinline__ int beside(int v, int edge) {
    return __builtin_amdgcn_update_dpp(edge, v, CTRL, 0xf, 0xf, false);
}

constexpr int kTileRows = 4;                                    // of a wave
constexpr int kBlockRows = kTileRows * (kMetricWG / 64);

// A workgroup takes a run of tiles of 64 columns by kBlockRows rows, `tiles` in all, and
// adds its pairs to global memory after each, or with `keep` at the end.  A pixel is a
// boundary pixel when a 4-neighbour inside the image has another label; the clamped
// neighbour of a border pixel is the pixel itself, which never differs.
//
// What bounds it: the latency of a wave's chain (loads, 4 rows of table updates,
// the block's flush).  8 rows a wave: 12.3 us, 16: 32.  1920x1080, 2000 superpixels, 400
// regions: 34.4 us with a turn of the table update per distinct pair of a row
// (24 us of it those turns), 11.3 now.
__global__ __launch_bounds__(kMetricWG) void k_metric_pixels(MetricGeom g, int tiles,
                                                             const int* __restrict__ S,
                                                             const int* __restrict__ G,
                                                             unsigned* __restrict__ table,
                                                             unsigned* __restrict__ perim,
                                                             unsigned long long* __restrict__ smap,
                                                             unsigned long long* __restrict__ gmap) {
    __shared__ PairTable pt;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int per = (tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int begin = xcd_remap(blockIdx.x, gridDim.x) * per, end = min(tiles, begin + per);
    for (int tile = begin; tile < end; ++tile) {      // uniform
        const int by = tile / g.Wq, word = tile - by * g.Wq;
        const int x = word * 64 + lane, y0 = by * kBlockRows + wave * kTileRows;
        const bool in = x < g.W;
        const int xc = min(x, g.W - 1);
        // column beside the wave, for its first and last lanes
        const int xe = lane == 0 ? max(x - 1, 0) : min(x + 1, g.W - 1);
        int s[kTileRows + 2], r[kTileRows + 2], se[kTileRows], re[kTileRows];
        for (int i = 0; i < kTileRows + 2; ++i) {
            const long long row = (long long)min(max(y0 + i - 1, 0), g.H - 1) * g.W;
            s[i] = S[row + xc];
            r[i] = G[row + xc];
        }
        for (int i = 0; i < kTileRows; ++i) {
            se[i] = re[i] = 0;
            const long long row = (long long)min(y0 + i, g.H - 1) * g.W;
            if (lane == 0 || lane == 63) {
                se[i] = S[row + xe];
                re[i] = G[row + xe];
            }
        }
        if (!g.keep || tile == begin) {
            for (int t = threadIdx.x; t < kPairSlots; t += kMetricWG) {   // while they come
                pt.key[t] = kEmpty;
                pt.cnt[t] = 0u;
                pt.edge[t] = 0u;
            }
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < kTileRows; ++i) {
            const int y = y0 + i;
            if (y >= g.H) break;                      // uniform over the wave
            const int k = s[i + 1], reg = r[i + 1];
            const int kl = beside<0x138>(k, se[i]), kr = beside<0x130>(k, se[i]);
            const int gl = beside<0x138>(reg, re[i]), gr = beside<0x130>(reg, re[i]);
            const bool dl = kl != k, dr = in && kr != k, du = s[i] != k, dd = s[i + 2] != k;
            const bool sb = in && (dl || dr || du || dd);
            const bool gb = in && (gl != reg || gr != reg || r[i] != reg || r[i + 2] != reg);
            const unsigned long long sm = __ballot(sb), gm = __ballot(gb);
            if (lane == 0) {
                smap[(long long)y * g.Wq + word] = sm;
                gmap[(long long)y * g.Wq + word] = gm;
            }
            const bool ok = in && k >= 0 && k < g.K && reg >= 0 && reg < g.R;
            const unsigned e = (unsigned)(dl || x == 0) + (unsigned)(dr || x + 1 >= g.W) +
                               (unsigned)(du || y == 0) + (unsigned)(dd || y + 1 >= g.H);
            const bool head = lane == 0 || dl || gl != reg || x == g.W;
            row_count(pt, table, perim, g.R, ok, head, k, reg, ok ? e : 0u);
        }
        if (g.keep && tile + 1 < end) continue;
        __syncthreads();
        for (int t = threadIdx.x; t < kPairSlots; t += kMetricWG) {
            const unsigned key = pt.key[t];
            if (key == kEmpty) continue;
            atomicAdd(&table[key], pt.cnt[t]);
            if (pt.edge[t]) atomicAdd(&perim[key / (unsigned)g.R], pt.edge[t]);
        }
        __syncthreads();
    }
}

// 192-bit window {lo, mid, hi} (lo holds the lowest pixel indices), dilated by
// [-a, a] along the row: intervals grow by {-s, 0, s} steps with s <= 2m + 1,
// so the union stays gap-free; for a <= 63 every shifted-in bit of mid comes
// from inside the window.
__device__ __forceinline__ unsigned long long dilate_mid(unsigned long long lo,
                                                         unsigned long long mid,
                                                         unsigned long long hi, int a) {
    int m = 0;
    while (m < a) {
        const int s = min(2 * m + 1, a - m), t = 64 - s;
        const unsigned long long l2 = lo | (lo << s) | (lo >> s) | (mid << t);
        const unsigned long long m2 = mid | (mid << s) | (lo >> t) | (mid >> s) | (hi << t);
        const unsigned long long h2 = hi | (hi << s) | (mid >> t) | (hi >> s);
        lo = l2;
        mid = m2;
        hi = h2;
        m += s;
    }
    return mid;
}

// Thread per bitmap word (row y, word w): a ground-truth boundary pixel is
// recalled when a superpixel boundary pixel lies at (dx, dy) with
// dx^2 + dy^2 < epsilon^2 (Eq. (5)); out-of-image pixels are zero bits.
// The disc rows are taken three at a time, their words loaded before any is
// dilated.  part[3 b + {0, 1, 2}] = this block's ground-truth boundary
// pixels, recalled ones, superpixel boundary pixels.
__device__ __forceinline__ void metric_recall(const MetricGeom& g,
                                              const unsigned long long* __restrict__ smap,
                                              const unsigned long long* __restrict__ gmap,
                                              unsigned long long* __restrict__ part) {
    __shared__ unsigned long long red[kMetricWG / 64][3];
    const long long words = (long long)g.H * g.Wq;
    unsigned long long gb = 0, hit = 0, sb = 0;
    for (long long t = blockIdx.x * (long long)kMetricWG + threadIdx.x; t < words;
         t += (long long)g.nrb * kMetricWG) {
        const int y = (int)(t / g.Wq), w = (int)(t - (long long)y * g.Wq);
        const unsigned long long gw = gmap[t];
        sb += (unsigned long long)__popcll(smap[t]);
        if (gw == 0ULL) continue;
        gb += (unsigned long long)__popcll(gw);
        unsigned long long d = 0;
        for (int dy0 = -g.r; dy0 <= g.r && (gw & ~d) != 0ULL; dy0 += 3) {
            unsigned long long lo[3], mid[3], hi[3];
            int a[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int dy = dy0 + j, yy = y + dy;
                a[j] = -1;                            // largest |dx| inside the disc
                if (dy <= g.r && yy >= 0 && yy < g.H)
                    while (a[j] < g.r && (float)((a[j] + 1) * (a[j] + 1) + dy * dy) < g.eps2) ++a[j];
                lo[j] = mid[j] = hi[j] = 0ULL;
                if (a[j] >= 0) {
                    const unsigned long long* rw = smap + (long long)yy * g.Wq;
                    mid[j] = rw[w];
                    if (w > 0) lo[j] = rw[w - 1];
                    if (w + 1 < g.Wq) hi[j] = rw[w + 1];
                }
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (a[j] >= 0) d |= dilate_mid(lo[j], mid[j], hi[j], a[j]);
        }
        hit += (unsigned long long)__popcll(gw & d);
    }
    for (int o = 32; o > 0; o >>= 1) {
        gb += __shfl_xor(gb, o, 64);
        hit += __shfl_xor(hit, o, 64);
        sb += __shfl_xor(sb, o, 64);
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[wv][0] = gb;
        red[wv][1] = hit;
        red[wv][2] = sb;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long v = 0;
        for (int q = 0; q < kMetricWG / 64; ++q) v += red[q][threadIdx.x];
        part[3LL * blockIdx.x + threadIdx.x] = v;
    }
}

// Per superpixel (one wave each, lanes striding over the regions): area,
// largest overlap (ASA), sum over meeting regions of |S_k| - |S_k n G_i|
// (UE), and the CO term.  Integer sums and maxima: exact in any order.
__device__ __forceinline__ void metric_rows(const MetricGeom& g, int block,
                                            const unsigned* __restrict__ table,
                                            const unsigned* __restrict__ perim,
                                            unsigned long long* __restrict__ row_max,
                                            unsigned long long* __restrict__ row_ue,
                                            double* __restrict__ row_co) {
    const int k = block * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k >= g.K) return;                             // uniform over the wave
    const unsigned* t = table + (long long)k * g.R;
    unsigned long long area = 0, meet = 0;
    unsigned mx = 0;
    for (int i = lane; i < g.R; i += 64) {
        const unsigned c = t[i];
        area += c;
        mx = c > mx ? c : mx;
        meet += c ? 1ULL : 0ULL;
    }
    for (int o = 32; o > 0; o >>= 1) {
        area += __shfl_xor(area, o, 64);
        meet += __shfl_xor(meet, o, 64);
        const unsigned m2 = __shfl_xor(mx, o, 64);
        mx = m2 > mx ? m2 : mx;
    }
    if (lane == 0) {
        row_max[k] = mx;
        row_ue[k] = meet * area - area;   // sum over meeting i of (area - c_i)
        const double P = (double)perim[k];
        row_co[k] = area ? 4.0 * 3.14159265358979323846 * (double)area * (double)area / (P * P)
                         : 0.0;
    }
}

// Recall in blocks [0, g.nrb), rows in the others: neither reads what the other
// writes, and each alone lasts about as long as a launch (4.5 and 4.6 us apart,
// 4.7 together).
__global__ __launch_bounds__(kMetricWG) void k_metric_rest(MetricGeom g,
                                                           const unsigned long long* __restrict__ smap,
                                                           const unsigned long long* __restrict__ gmap,
                                                           unsigned long long* __restrict__ part,
                                                           const unsigned* __restrict__ table,
                                                           const unsigned* __restrict__ perim,
                                                           unsigned long long* __restrict__ row_max,
                                                           unsigned long long* __restrict__ row_ue,
                                                           double* __restrict__ row_co) {
    if ((int)blockIdx.x < g.nrb)
        metric_recall(g, smap, gmap, part);
    else
        metric_rows(g, (int)blockIdx.x - g.nrb, table, perim, row_max, row_ue, row_co);
}

__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sums of integers in any order; the FP64 terms are summed in 1024 strands (k mod
// 1024, four to a lane), paired t with t + 512, then t + 256, ...: in registers,
// then through LDS above a wave and by shuffles within.  One workgroup of four
// waves: with sixteen the reductions took longer than the loads they save.
__global__ __launch_bounds__(kMetricWG) void k_metric_final(MetricGeom g,
                                                            const unsigned long long* __restrict__ row_max,
                                                            const unsigned long long* __restrict__ row_ue,
                                                            const double* __restrict__ row_co,
                                                            const unsigned long long* __restrict__ part,
                                                            double* __restrict__ out) {
    __shared__ unsigned long long red[5][kMetricWG / 64];
    __shared__ double rc[kMetricWG];
    const int tid = threadIdx.x;
    unsigned long long v[5] = {0, 0, 0, 0, 0};
    double c[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < g.K; k0 += 1024) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // (loads of a lane past the end repeat the last row: all in flight)
            const int k = k0 + 256 * q + tid, kc = min(k, g.K - 1);
            const unsigned long long m = row_max[kc], u = row_ue[kc];
            const double t = row_co[kc];
            v[0] += k < g.K ? m : 0ULL;
            v[1] += k < g.K ? u : 0ULL;
            c[q] += k < g.K ? t : 0.0;
        }
    }
    for (int b = tid; b < g.nrb; b += kMetricWG) {
        v[2] += part[3LL * b];
        v[3] += part[3LL * b + 1];
        v[4] += part[3LL * b + 2];
    }
    rc[tid] = (c[0] + c[2]) + (c[1] + c[3]);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        v[j] = wave_total(v[j]);
        if ((tid & 63) == 0) red[j][tid >> 6] = v[j];
    }
    __syncthreads();
    if (tid >= 64) return;
    double co = (rc[tid] + rc[tid + 128]) + (rc[tid + 64] + rc[tid + 192]);
    for (int o = 32; o > 0; o >>= 1) co += __shfl_down(co, o, 64);   // lane 0: the tree's order
    if (tid == 0) {
#pragma unroll
        for (int j = 0; j < 5; ++j) v[j] = red[j][0] + red[j][1] + red[j][2] + red[j][3];
        const double N = (double)g.W * (double)g.H;
        out[0] = v[2] ? (double)v[3] / (double)v[2] : 1.0;      // BR
        out[1] = (double)v[0] / N;                                 // ASA
        out[2] = (double)v[1] / N;                                 // UE
        out[3] = co / N;                                         // CO
        out[4] = (double)v[2];                                     // |B(G)|
        out[5] = (double)v[4];                                     // |B(S)|
    }
}

__global__ void k_zero_u32(unsigned* __restrict__ p, long long n) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = 0u;
}

}  // namespace

constexpr int kRecallBlocks = 2048;   // most recall blocks (partial sums)

size_t metrics_workspace_bytes(int W, int H, int K, int R) {
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t table = (size_t)K * (size_t)R * 4, perim = (size_t)K * 4;
    const size_t rows = (size_t)K * 8 * 3, part = (size_t)kRecallBlocks * 3 * 8;
    const size_t map = (size_t)H * (size_t)((W + 63) / 64) * 8;
    return up(table) + up(perim) + up(rows) + up(part) + 2 * up(map);
}

int launch_metrics(int W, int H, const int* S, int K, const int* G, int R, float eps, double* out,
                   void* ws, hipStream_t st) {
    MetricGeom g;
    g.W = W; g.H = H; g.K = K; g.R = R;
    g.Wq = (W + 63) / 64;
    g.r = (int)ceilf(eps) - 1;
    g.eps2 = eps * eps;
    const int tiles = g.Wq * ((H + kBlockRows - 1) / kBlockRows);   // below 2^27
    // A block per tile; where the LDS table holds all pairs there are, as many blocks as
    // the chip holds at once, and two tiles each at least: one label everywhere,
    // 3840x2160, 45 us instead of 105, as every block adds to the same words.  (Runs of tiles for
    // all images took 84 us instead of 79 for 10000 superpixels.)
    g.keep = (long long)K * R <= kPairSlots / 2;
    const int blocks = g.keep ? std::min((tiles + 1) / 2, 2048) : std::min(tiles, 65536);
    const long long map = (long long)H * g.Wq;
    g.nrb = (int)std::min<long long>((map + kMetricWG - 1) / kMetricWG, kRecallBlocks);
    char* b = static_cast<char*>(ws);
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    unsigned* table = reinterpret_cast<unsigned*>(b);
    size_t off = up((size_t)K * R * 4);
    unsigned* perim = reinterpret_cast<unsigned*>(b + off);
    off += up((size_t)K * 4);
    unsigned long long* row_max = reinterpret_cast<unsigned long long*>(b + off);
    unsigned long long* row_ue = row_max + K;
    double* row_co = reinterpret_cast<double*>(row_ue + K);
    off += up((size_t)K * 8 * 3);
    unsigned long long* part = reinterpret_cast<unsigned long long*>(b + off);
    off += up((size_t)kRecallBlocks * 3 * 8);
    unsigned long long* smap = reinterpret_cast<unsigned long long*>(b + off);
    unsigned long long* gmap = smap + up((size_t)map * 8) / 8;
    // table and perim (contiguous up to row_max) start at zero; every bitmap
    // word and every partial sum is written before it is read
    const long long zero_words = (long long)(reinterpret_cast<char*>(row_max) - b) / 4;
    const unsigned zb = (unsigned)std::min<long long>((zero_words + 255) / 256, 65536);
    hipLaunchKernelGGL(k_zero_u32, dim3(zb), dim3(256), 0, st, table, zero_words);
    hipLaunchKernelGGL(k_metric_pixels, dim3((unsigned)blocks), dim3(kMetricWG), 0,
                       st, g, tiles, S, G, table, perim, smap, gmap);
    hipLaunchKernelGGL(k_metric_rest, dim3((unsigned)(g.nrb + (K + 3) / 4)), dim3(kMetricWG), 0, st,
                       g, smap, gmap, part, table, perim, row_max, row_ue, row_co);
    hipLaunchKernelGGL(k_metric_final, dim3(1), dim3(kMetricWG), 0, st, g, row_max, row_ue, row_co, part,
                       out);
    return hipGetLastError();
}

}  // namespace scalp
