// scalp_internal.h -- shared declarations of the HIP kernels and the host ABI
// layer of libscalp.so (not part of the public interface).
#pragma once

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
    kCtrlQueue = 1088,    // words 1088-1343: the persistent assignment's 8 queue heads
                          // (one per XCD's run of items), one per 128-byte line
    kCtrlWords = 1344
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

struct Tuning {
    int wg;           // workgroup size of the assignment kernel (256, 512 or 1024)
    int blocks_per_cu = 0;   // persistent launch: workgroups per CU (0: as many as fit)
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
                                    int* ctrl, hipStream_t s);
long long block_pixels(int W, int H, int nx, int ny);
// lists (or null) and R: make the tile lists of the window form's next pass, too
int launch_finalize_project(const Img& im, float* centres, int* endpoints, int* counts,
                            long long* acc, const int* labels, void* lists, int R, hipStream_t s);
int launch_project(const Img& im, const float* centres, const int* counts, const int* labels,
                   int* endpoints, const int* ctrl, const int* plist, hipStream_t s);

// Batched variants: imgs/cell_start/sp_start are device arrays in the workspace.
int launch_init_cells_batched(const Img* imgs, const int* cell_start, int n_img, int total_cells,
                              const float4* packed, int* labels, long long* acc, hipStream_t s);
// (near: near_image of every image)
int launch_assign_persistent(const Img* imgs, const int* item_start, int n_img, int total_items,
                             const float4* packed, const float* centres, const int* endpoints,
                             int* labels, long long* acc, int* ctrl, float lambda,
                             const Tuning& t, bool near, int grid, hipStream_t s);
int launch_finalize_batched(const Img* imgs, const int* sp_start, int n_img, int total_sp,
                            float* centres, int* endpoints, int* counts, long long* acc,
                            const int* labels, int* ctrl, int* plist, bool project,
                            hipStream_t s);
int persistent_grid(const Tuning& t);

// ---- soft SCALP (scalp_soft.hip)
struct SoftGeom {
    int W, H, nx, ny, B;
    int wg;   // workgroup size of the path kernels (256, 512 or 1024)
    float spw, gamma, lambda, temperature;
    int prune;  // 1: skip the walks of slots whose softmax weight is provably 0
};
SoftGeom soft_geom(int W, int H, int nx, int ny, int B, float spw, float gamma, float lambda,
                   float temperature, int wg, int prune);
void lift_soft_lds_limits();
// Work items per cell of the soft assignment at workgroup size wg: a cell
// is cut into slices of whole 64-pixel chunks, at most wg pixels each.
int soft_slices(int W, int H, int nx, int ny, int wg);
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
