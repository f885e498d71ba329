// scalp_internal.h -- shared declarations of the HIP kernels and the host ABI
// layer of libscalp.so (not part of the public interface).
#pragma once

#include <algorithm>

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scalp {

// Fixed point of the colour sums in the update: values are rounded to
// multiples of 2^-24 and summed as 64-bit integers, so the sum does not
// depend on the order in which pixels arrive (atomics, workgroups).
constexpr float kFixScaleF = 16777216.0f;
constexpr double kFixInv = 1.0 / 16777216.0;

// Per-superpixel accumulator stride (int64 words): count, sum x, sum y,
// sum l, sum a, sum b, 2 pad -> one 64-byte line per superpixel.
constexpr int kAccStride = 8;

// Control words in the workspace.
enum Ctrl : int {
    kCtrlProjCount = 0,   // entries in the projection list
    kCtrlGradMax = 64,    // words 64-1087: kGradSlots maxima of the squared gradient
                          // magnitude (FP64 bits)
    kCtrlWords = 1344     // (the rest is unused: callers' buffers are sized by it)
};

// Each block of the gradient's maximum pass has one of kGradSlots 64-bit slots.
constexpr int kGradSlots = 512;
constexpr int kGradBytes = kGradSlots * 8;

// Division of numbers below a known limit by an invariant d, as one high
// multiplication: floor(v / d) = floor(v m / 2^32) with m = ceil(2^32 / d)
// whenever v (m d - 2^32) < 2^32, hence for every v with v d < 2^32; m = 0
// (d = 1, or a limit beyond that): the division itself.
struct FastDiv {
    unsigned m, d;
};

inline FastDiv fast_div(long long d, long long limit) {
    FastDiv f;
    f.d = (unsigned)d;
    f.m = d > 1 && limit < (1LL << 32) / d ? (unsigned)((0x100000000LL + d - 1) / d) : 0u;
    return f;
}

// One image as the kernels see it.
struct Img {
    int W, H, nx, ny;
    long long pix;    // first pixel in the concatenated pixel arrays
    int sp;           // first superpixel in the concatenated superpixel arrays
    float spw;        // m^2 / r^2 of Eq. (3)
    float gamma;      // gamma of Eq. (2)
    int spl;          // assignment work items per grid cell (at most WG pixels each)
    int rad;          // R = r rounded to whole pixels (the window form's half-width)
    int prune;        // 1: skip the walks that the exact lower bound of D rules out
    int strips;       // column strips of the grid assignment's cell order (see cell_in_strips)
    int far;          // 1: byte offsets of texels need more than 32 bits
    FastDiv dnx, dny;               // cell boundaries: x ny / H and x nx / W
    FastDiv dspl;                   // work item -> cell
    FastDiv dstrip, dcol, dlast;    // cell order: strips, columns of a strip, of the last strip
    FastDiv dper[2];                // 8 x the two cell heights: 8-column strips of a cell
};
// Fills the derived fields above from W, H, nx, ny, spl and strips.
void finish_img(Img& im);
// Whether 32-bit indexes and step counters serve every path of the image.
bool near_image(const Img& im);

// An assignment work item has at most as many pixels as its workgroup has
// lanes (one pixel per lane): cells larger than that are split into several
// items, which also spreads images with few, large superpixels over the chip.
constexpr int kMinAssignWG = 256;

constexpr int kCUs = 256;

// Whether the work items of an image of N pixels and K cells take half a workgroup's
// pixels.  Where paths are long (cells above 48 x 48 pixels) a pixel has several pairs
// in the second pass: such items halve its rounds, which shortens launches of few items.
// 10 iterations, 256 lanes, half and whole: 300x200, 12 cells, 0.38 and 0.48 ms; 481x321,
// 40 cells, 0.43 and 0.62; 12 scales of 481x321 2.20 and 2.45.  From 2^20 pixels on the
// idle lanes cost more: 1920x1080, 700 cells, 1.27 and 1.20; 3840x2160, 3000, 3.85 and
// 3.12.  (A launch, 2 W H lanes with half items, also holds below 2^32.)
inline bool half_items(long long N, long long K) { return N > 2304 * K && N < 1 << 20; }

// Pixels of a work item of a hard assignment by workgroups of wg lanes.
inline int item_pixels(long long W, long long H, long long K, int wg) {
    return half_items(W * H, K) ? wg / 2 : wg;
}

// Without exact pruning every pixel walks every candidate: over LDS tables that a
// workgroup makes of each, up to kTablePixels pixels an item whatever the workgroup.
// In a launch of few cells the chain of nine tables takes longer than lists of pairs,
// whose items can be smaller, and in small cells a table has more entries than its
// paths samples.  10 iterations over tables and by pairs: 97x61, 30 cells, 228 and 170
// us; 160x120, 70, 248 and 225; 300x200, 130, 276 and 365; 1920x1080 with 41 pixels a
// cell 9.48 and 3.16 ms, with 207 2.39 and 2.91, with 20 cells 28.5 and 37.7.
constexpr int kTablePixels = 1024;

// How a hard assignment walks: every candidate (kAll); the listed pairs, or over tables
// in items that list many (kMany); or the pairs alone, also where cells are so small that
// tables would not pay, and where items of half the lanes never list many: without the
// tables' code and LDS 1920x1080 in 500000 cells took 13.0 instead of 13.6 ms.
enum class Walk { kPairs, kMany, kAll };

inline Walk walk_of(int prune, long long N, long long K) {
    const bool cells = N >= 128 * K;
    if (!prune) return cells && std::max(K, N / kTablePixels) > 96 ? Walk::kAll : Walk::kPairs;
    return cells && !half_items(N, K) ? Walk::kMany : Walk::kPairs;
}

// Items per cell: so many that no item has more than `pixels` pixels, and at least
// `fill` of them, down to one 64-pixel chunk each.
inline int assign_slices(int W, int H, int nx, int ny, int pixels, long long fill) {
    const long long cw = (W + nx - 1) / nx, ch = (H + ny - 1) / ny;
    const long long chunks = (cw * ch + 63) / 64, per = pixels / 64;
    return (int)std::max((chunks + per - 1) / per, std::min(chunks, fill));
}

// `fill` of a launch over `cells` cells: where a workgroup each would not reach all
// compute units, as many as do (the lanes without a pixel walk the second pass's
// pairs).  97x61, 30 cells, one item per cell: 11.2 us instead of 10.6; two such
// images soft at T = 5: 20.5 instead of 13.7.  More items than kCUs gain nothing
// (481x321, 250 cells in 3 items: 14.0 us, in 4: 14.6).
inline long long fill_slices(long long cells) { return kCUs / cells; }

// Pixels of a work item of a batch of N pixels, for its image of W x H pixels and K
// cells.  A batch of fewer pixels than half the lanes that the chip holds takes a
// quarter of a workgroup's pixels: 7 scales of 189x117 (0.15 M pixels) 32 us per
// iteration with 128 or 256 of 256 lanes, 26 with 64.  Batches of 250 pixels a
// superpixel, 10 iterations with whole and quarter items: 0.22 M pixels 0.34 and 0.28
// ms, 0.33 M 0.36 and 0.37, 0.53 M 0.36 and 0.45, 0.79 M 0.42 and 0.61, 1.05 M 0.47
// and 0.77.  Workgroups of 1024 lanes with 64 pixels each left 15 lanes of 16 idle: 3
// images of up to 480 pixels a side 52.3 us per iteration, 34.4 with 256 pixels.
constexpr long long kFewPixels = 1 << 18;

inline int batch_item_pixels(long long N, long long W, long long H, long long K, int wg) {
    return N < kFewPixels ? wg / 4 : item_pixels(W, H, K, wg);
}

struct Tuning {
    int wg;           // workgroup size of the assignment kernel (256, 512 or 1024)
};

// LDS budget of the soft backward's tiles in 16-byte units: the default, and the
// largest (152 KiB of the 160 KiB of a gfx950 CU).
constexpr int kDefaultLdsPixels = 4800;
constexpr int kMaxLdsPixels = 9728;

int launch_write_bytes(void* dst, const void* src, size_t n, hipStream_t s);

// Launchers (return hipError_t as int).  All enqueue on `s`.
int launch_prepare(long long n, const float* lab, const float* contour, float sigma,
                   float4* packed, hipStream_t s);
int launch_clear(long long* p, long long n_words, hipStream_t s);
int launch_init_cells(const Img& im, const float4* packed, int* labels, long long* acc,
                      hipStream_t s);
int launch_assign(const Img& im, const float4* packed, const float* centres,
                  const int* endpoints, int* labels, long long* acc, int* ctrl, float lambda,
                  bool accumulate, const Tuning& t, hipStream_t s);
int launch_accumulate(const Img& im, const float* lab, const int* labels, long long* acc,
                      hipStream_t s);
// Window form of the assignment (candidate rule of Algorithm 1; labels in/out).
// lists: max(8 W H, 256) bytes of scratch, the first window_count_words 64-bit
// words of them zero before the first pass (every pass leaves them zero).
// listed: the lists are made already (launch_finalize_project of the pass before).
// accumulate: add the update's sums to acc and empty the projection queue, as the
// grid form does.
long long window_count_words(int W, int H);
int launch_assign_window(const Img& im, const float4* packed, const float* centres,
                         const int* endpoints, int* labels, long long* acc, int* ctrl, void* lists,
                         int R, float lambda, bool accumulate, bool listed, hipStream_t s);
int launch_finalize(const Img& im, float* centres, int* endpoints, int* counts,
                    long long* acc, const int* labels, int* ctrl, int* plist, bool project,
                    hipStream_t s);
// finalize + projection in one launch (one workgroup per superpixel)
// (max_block_px: the most pixels of any superpixel's 3x3 cell block in the batch)
int launch_finalize_project_batched(const Img* imgs, const int* sp_start, int n_img,
                                    int total_sp, long long max_block_px, float* centres,
                                    int* endpoints, int* counts, long long* acc, const int* labels,
                                    hipStream_t s);
long long block_pixels(int W, int H, int nx, int ny);
// lists (or null) and R: make the tile lists of the window form's next pass, too
int launch_finalize_project(const Img& im, float* centres, int* endpoints, int* counts,
                            long long* acc, const int* labels, void* lists, int R, hipStream_t s);
int launch_project(const Img& im, const float* centres, const int* counts, const int* labels,
                   int* endpoints, const int* ctrl, const int* plist, hipStream_t s);

// Batched variants: imgs/cell_start/sp_start are device arrays in the workspace.
int launch_init_cells_batched(const Img* imgs, const int* cell_start, int n_img, int total_cells,
                              const float4* packed, int* labels, long long* acc, hipStream_t s);
// longest_run: items of the longest of the 8 XCDs' runs; near: near_image of every
// image
int launch_assign_batched(const Img* imgs, const int* item_start, int n_img, int longest_run,
                          const float4* packed, const float* centres, const int* endpoints,
                          int* labels, long long* acc, int* ctrl, float lambda, const Tuning& t,
                          bool near, Walk walk, hipStream_t s);
int launch_finalize_batched(const Img* imgs, const int* sp_start, int n_img, int total_sp,
                            float* centres, int* endpoints, int* counts, long long* acc,
                            const int* labels, int* ctrl, int* plist, bool project,
                            hipStream_t s);

// ---- soft SCALP (scalp_soft.hip)
struct SoftGeom {
    int W, H, nx, ny, B;
    int wg;   // workgroup size of the forward's assignment (0: chosen, 256, 512 or 1024)
    float spw, gamma, lambda, temperature;
    int prune;  // 1: skip the walks of slots whose softmax weight is provably 0
};
SoftGeom soft_geom(int W, int H, int nx, int ny, int B, float spw, float gamma, float lambda,
                   float temperature, int wg, int prune);
void lift_soft_lds_limits();
int launch_soft_init(const SoftGeom& g, const float4* packed, float* theta0, hipStream_t st);
// pmask [B][N]: bit j of a pixel: its Q of slot j is not 0
int launch_soft_assign(const SoftGeom& g, const float4* packed, const float* theta_prev, float* q,
                       float* fa, float* fb, unsigned short* pmask, hipStream_t st);
int launch_soft_update(const SoftGeom& g, const float* q, const unsigned short* pmask,
                       const float4* packed, const float* theta_prev, float* theta_next, double* z,
                       hipStream_t st);
// Backward.  cand: 2 * B * K float4, per superpixel the terms of the update
// backward; pairs: [B][9][N] (pixel, dL/dD) lists, count: their lengths, 9 per
// (image, cell, slice); gth, gth_prev (dL/dTheta) are FP64; z_prev: masses of
// the iteration before (null in the first); cap_bytes: LDS tile budget.
int soft_bwd_slices(int W, int H, int nx, int ny);
int launch_soft_bwd_start(const SoftGeom& g, const float* grad_theta, const double* z,
                          const float* theta, double* gth, float4* cand, hipStream_t st);
int launch_soft_bwd_update(const SoftGeom& g, int first, const float* q,
                           const unsigned short* pmask, const float4* packed, const float* gq_in,
                           const float4* cand, uint2* pairs, int* count, float4* gf,
                           hipStream_t st);
int launch_soft_bwd_path(const SoftGeom& g, const float4* packed, const float* theta_prev,
                         const float* fa, const float* fb, const uint2* pairs, const int* count,
                         const double* z, const double* gth, const double* z_prev,
                         double* gth_prev, float4* cand, float4* gf, int cap_bytes,
                         hipStream_t st);
int launch_soft_bwd_finish(const SoftGeom& g, const float4* gf, const double* gth0,
                           const float* contour, float sigma, float* glab, float* gcon,
                           hipStream_t st);

// ---- per-pixel maps (scalp_maps.hip)
int launch_boundary_frequency(int W, int H, int n, const int* labels, float* out, hipStream_t s);
int launch_contour_from_lab(int W, int H, const float* lab, float* out, void* ws, hipStream_t s);
// prepare with the contour prior computed from lab (same values as
// launch_contour_from_lab followed by launch_prepare); mx: kGradBytes of scratch
int launch_prepare_gradient(int W, int H, const float* lab, float sigma, float4* packed,
                            unsigned long long* mx, hipStream_t s);

// ---- quality metrics (scalp_metrics.hip)
size_t metrics_workspace_bytes(int W, int H, int K, int R);
int launch_metrics(int W, int H, const int* S, int K, const int* G, int R, float eps, double* out,
                   void* ws, hipStream_t st);

}  // namespace scalp
