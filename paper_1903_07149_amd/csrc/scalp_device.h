// scalp_device.h -- device helpers shared by the hard and soft kernels.
#pragma once

#include "scalp_internal.h"

namespace scalp {
namespace dev {

// First coordinate of grid cell `idx` of `n` along an axis of `len` pixels:
// pixel c is in cell floor(c * n / len), i.e. cell idx starts at
// ceil(idx * len / n).  With n <= len < 2^16 every product fits 32 bits and
// the division is a 32-bit one (len and n are uniform, so is the branch).
__device__ __forceinline__ int cell_lo(int idx, int len, int n) {
    if (len < 65536)
        return (int)(((unsigned)idx * (unsigned)len + (unsigned)(n - 1)) / (unsigned)n);
    return (int)(((long long)idx * len + n - 1) / n);
}

__device__ __forceinline__ int fdiv(int v, const FastDiv& f) {
    if (f.m) return (int)__umulhi((unsigned)v, f.m);      // uniform
    return f.d == 1u ? v : (int)((unsigned)v / f.d);
}

// cell_lo by f = the image's FastDiv for n cells over len pixels.
__device__ __forceinline__ int cell_lo(int idx, int len, int n, const FastDiv& f) {
    if (f.m)                                              // uniform
        return (int)__umulhi((unsigned)idx * (unsigned)len + (unsigned)(n - 1), f.m);
    return cell_lo(idx, len, n);
}

// Grid cell of coordinate c along an axis of `len` pixels cut into n cells:
// floor(c * n / len), in 32 bits when len < 2^16.
__device__ __forceinline__ int cell_of(int c, int n, int len) {
    if (len < 65536) return (int)(((unsigned)c * (unsigned)n) / (unsigned)len);
    return (int)(((long long)c * n) / len);
}

__device__ __forceinline__ float colour_dist(float4 f, float l, float a, float b) {
    float dl = f.x - l;
    float da = f.y - a;
    float db = f.z - b;
    return (dl * dl + da * da) + db * db;
}

__device__ __forceinline__ long long to_fixed(float v) {
    return (long long)rintf(v * kFixScaleF);
}

// Accumulates the samples i = 1 .. n-1 of the path from the pixel at linear
// index `idx` toward (dx, dy): on major-axis step i the minor offset is
// floor((2 i |d_minor| + n) / (2 n)).  stepx / stepy are the index strides
// of one pixel in x / y.  For paths of any length, by 64-bit indexes (walk_near
// takes the others); samples are accumulated in path order, with up to three
// texel loads in flight.  Paths of up to 46340 steps count the minor steps as the
// carries of a 32-bit accumulator (exact there, see step_increment); longer ones
// (cells over ~15000 pixels wide, or caller-supplied endpoints far across a wide
// image) keep the remainder exactly.
__device__ __forceinline__ unsigned step_increment(int am, int n);

__device__ __forceinline__ void walk_path(const float4* __restrict__ base, int idx, int stepx,
                                          int stepy, int dx, int dy, float l, float a, float b,
                                          float& sc, float& sw) {
    const int adx = dx < 0 ? -dx : dx;
    const int ady = dy < 0 ? -dy : dy;
    const bool xmaj = adx >= ady;
    const int n = xmaj ? adx : ady;
    if (n < 2) return;
    const int am = xmaj ? ady : adx;
    const int sx = dx < 0 ? -stepx : stepx;
    const int sy = dy < 0 ? -stepy : stepy;
    const int smaj = xmaj ? sx : sy;
    const int sdiag = smaj + (xmaj ? sy : sx);
#define SCALP_GACC(f)                                             \
    do {                                                          \
        const float dl_ = (f).x - l;                              \
        const float da_ = (f).y - a;                              \
        const float db_ = (f).z - b;                              \
        const float dc_ = (dl_ * dl_ + da_ * da_) + db_ * db_;    \
        sc = sc + dc_;                                            \
        sw = sw + (f).w;                                          \
    } while (0)
    if (n <= 46340) {
        const unsigned F = step_increment(am, n);
        unsigned acc = 0x80000000u;
#define SCALP_CSTEP()                                             \
    do {                                                          \
        const bool c_ = __builtin_add_overflow(acc, F, &acc);     \
        idx += c_ ? sdiag : smaj;                                 \
    } while (0)
        SCALP_CSTEP();
        float4 fa = base[idx];
        unsigned trips = (unsigned)(n - 2) >> 1;
        while (!__builtin_sub_overflow(trips, 1u, &trips)) {
            SCALP_CSTEP();
            const float4 fb = base[idx];
            SCALP_CSTEP();
            const float4 fc = base[idx];
            SCALP_GACC(fa);
            SCALP_GACC(fb);
            fa = fc;
            asm volatile("" : "+v"(acc));
        }
        if ((n - 2) & 1) {
            SCALP_CSTEP();
            const float4 fb = base[idx];
            SCALP_GACC(fa);
            fa = fb;
        }
        SCALP_GACC(fa);
#undef SCALP_CSTEP
        return;
    }
    const int two_n = 2 * n;
    const int inc = 2 * am;
    int rem = n;
#define SCALP_GSTEP()                                             \
    do {                                                          \
        rem += inc;                                               \
        const bool st_ = rem >= two_n;                            \
        rem -= st_ ? two_n : 0;                                   \
        idx += st_ ? sdiag : smaj;                                \
    } while (0)
    SCALP_GSTEP();
    float4 fa = base[idx];
    int left = n - 2;
    while (left >= 2) {
        SCALP_GSTEP();
        const float4 fb = base[idx];
        SCALP_GSTEP();
        const float4 fc = base[idx];
        SCALP_GACC(fa);
        SCALP_GACC(fb);
        fa = fc;
        left -= 2;
    }
    if (left == 1) {
        SCALP_GSTEP();
        const float4 fb = base[idx];
        SCALP_GACC(fa);
        fa = fb;
    }
    SCALP_GACC(fa);
#undef SCALP_GSTEP
#undef SCALP_GACC
}

// Stepping along a discrete line: the minor-axis offset after i major steps,
// floor(i s + 1/2) with s = |d_minor| / n, is the number of carries out of a
// 32-bit accumulator that starts at 2^31 and adds F = ceil(2^32 s) per step (2^32
// - 1 when s = 1).  The accumulated excess i (F - 2^32 s) < i stays below the gap
// 2^32 / (2n) between i s + 1/2 and the next integer whenever 2 n^2 < 2^32, i.e.
// n < 46340, and an exact tie is never undershot since F rounds up: one add with
// carry-out, one select and one address add per sample.
//
// Increment F for minor extent am and major extent n (0 <= am <= n).  Any F with
// 0 <= F - 2^32 am/n < 2^32/(2 n^2) steps exactly.  For n < 1023 a reciprocal good to one ulp
// gives 2^32 am/n within 769, and adding 1025 lands in (256, 1794]: inside
// the window for every n up to 1094.  (The largest float below 2^32 bounds it: a diagonal
// gives 2^32 or just above, and a path of no steps NaN; the sum then saturates to
// 2^32 - 1.)  Longer paths take the correctly rounded double quotient, rounded up.
__device__ __forceinline__ unsigned step_increment(int am, int n) {
    if (n < 1023) {
        const float sf = (float)am * __builtin_amdgcn_rcpf((float)n);
        return __builtin_elementwise_add_sat((unsigned)fminf(sf * 4294967296.0f, 0x1.fffffep31f), 1025u);
    }
    if (am == n) return 0xffffffffu;
    return (unsigned)ceil((double)am * 4294967296.0 / (double)n);
}

// The steps of a path from (dx, dy): major and diagonal index strides and the
// carry-counting increment (see step_increment), for strides sx, sy of one pixel.
struct PathStep {
    int n, smaj, sdiag;
    unsigned F;
};

__device__ __forceinline__ PathStep path_step(int dx, int dy, int sx, int sy) {
    const int adx = dx < 0 ? -dx : dx;
    const int ady = dy < 0 ? -dy : dy;
    PathStep s;
    s.n = max(adx, ady);
    const int stx = dx < 0 ? -sx : sx, sty = dy < 0 ? -sy : sy;
    s.smaj = adx >= ady ? stx : sty;
    s.sdiag = stx + sty;
    s.F = step_increment(min(adx, ady), s.n);
    return s;
}

#define SCALP_STEP(off)                                           \
    do {                                                          \
        const bool c_ = __builtin_add_overflow(acc, s.F, &acc);   \
        off += c_ ? s.sdiag : s.smaj;                             \
    } while (0)
#define SCALP_ACC(f)                                              \
    do {                                                          \
        sc = sc + colour_dist(f, l, a, b);                        \
        sw = sw + (f).w;                                          \
    } while (0)

// When a walk may stop: from the sums so far, lo = fl(fl(fl(a0 + f sc) fl(1 +
// g sw)) + dsp) with f = (1 - lambda) / |P|, g = gamma / |P| (approximate) and
// a0 = lambda dcp is Eq. (3)'s D of the path cut short.  Every summand of D is
// >= 0, so lo > thr, a threshold() or more, proves that D exceeds it.  Walks
// are never cut where gamma exceeds 2^40 (which could raise an underflow's
// error above 2^-70).
struct Cut {
    bool on;               // uniform
    float a0, f, g, dsp, thr;
};

__device__ __forceinline__ bool cut_now(const Cut& c, float sc, float sw) {
    return (c.a0 + c.f * sc) * (1.0f + c.g * sw) + c.dsp > c.thr;
}

// Samples i = 1 .. n (the endpoint) of the path s over the packed image, at
// 32-bit byte offsets from a uniform base (Eqs.near_img; paths of up to 46340
// steps), from the texel at `off`: 13 VALU instructions per
// sample, of which 8 are the colour distance.  Four samples per trip, their
// loads in flight together.  A walk that is cut returns an infinite sc.
__device__ __forceinline__ void walk_near(const float4* __restrict__ img, unsigned off,
                                          const PathStep& s, float l, float a, float b,
                                          const Cut& cut, float& sc, float& sw) {
    unsigned acc = 0x80000000u;
    const char* q = reinterpret_cast<const char*>(img);
#define SCALP_LOAD() (*reinterpret_cast<const float4*>(q + off))
    unsigned trips = (unsigned)s.n >> 2;
    while (!__builtin_sub_overflow(trips, 1u, &trips)) {
        SCALP_STEP(off);
        const float4 fa = SCALP_LOAD();
        SCALP_STEP(off);
        const float4 fb = SCALP_LOAD();
        SCALP_STEP(off);
        const float4 fc = SCALP_LOAD();
        SCALP_STEP(off);
        const float4 fd = SCALP_LOAD();
        SCALP_ACC(fa);
        SCALP_ACC(fb);
        SCALP_ACC(fc);
        SCALP_ACC(fd);
        asm volatile("" : "+v"(acc));
        if (cut.on && cut_now(cut, sc, sw)) {
            sc = INFINITY;
            return;
        }
    }
    if (s.n & 2) {
        SCALP_STEP(off);
        const float4 fa = SCALP_LOAD();
        SCALP_STEP(off);
        const float4 fb = SCALP_LOAD();
        SCALP_ACC(fa);
        SCALP_ACC(fb);
    }
    if (s.n & 1) {
        SCALP_STEP(off);
        const float4 fa = SCALP_LOAD();
        SCALP_ACC(fa);
    }
#undef SCALP_LOAD
}

// The same over an LDS table of (colour distance to the candidate, w) of the texels
// around the paths, from byte offset `off`: 5 VALU instructions and an 8-byte LDS
// read per sample.  The colour distances are those that walk_near forms, added in
// the same order: the same sums.
__device__ __forceinline__ void walk_table(const float2* table, unsigned off, const PathStep& s,
                                           float& sc, float& sw) {
    unsigned acc = 0x80000000u;
    const char* q = reinterpret_cast<const char*>(table);
#define SCALP_LOAD() (*reinterpret_cast<const float2*>(q + off))
    unsigned trips = (unsigned)s.n >> 2;
    while (!__builtin_sub_overflow(trips, 1u, &trips)) {
        SCALP_STEP(off);
        const float2 fa = SCALP_LOAD();
        SCALP_STEP(off);
        const float2 fb = SCALP_LOAD();
        SCALP_STEP(off);
        const float2 fc = SCALP_LOAD();
        SCALP_STEP(off);
        const float2 fd = SCALP_LOAD();
        sc = ((sc + fa.x) + fb.x) + fc.x + fd.x;
        sw = ((sw + fa.y) + fb.y) + fc.y + fd.y;
        asm volatile("" : "+v"(acc));
    }
    for (int i = s.n & 3; i > 0; --i) {
        SCALP_STEP(off);
        const float2 fa = SCALP_LOAD();
        sc = sc + fa.x;
        sw = sw + fa.y;
    }
#undef SCALP_LOAD
}
#undef SCALP_STEP
#undef SCALP_ACC

// Correctly rounded FP64 reciprocals 1/1 .. 1/1024, built at compile time.
struct RecipTable {
    double v[1025];
    constexpr RecipTable() : v() {
        for (int i = 1; i <= 1024; ++i) v[i] = 1.0 / (double)i;
    }
};
namespace {
__constant__ const RecipTable kRecip = RecipTable();
}

// RN(1 / (n + 1)) for a path of n steps (np = n + 1 samples), clamped to the
// table; callers fetch it before walking the path so that the load's latency
// hides behind the walk.
__device__ __forceinline__ double path_recip(int n) { return kRecip.v[(n < 1023 ? n : 1023) + 1]; }

// a / np and b / np in IEEE FP32 (np = n + 1) for the two averages of
// Eqs. (1)-(2); inv = path_recip(n).  For np <= 1024 and a, b zero or at
// least 2^-100, the FP32 rounding of the FP64 product a * RN(1/np) is the
// IEEE quotient: a float divided by an integer np is never a rounding
// midpoint of FP32 and stays at least 2^-35 (relative) away from one for
// np <= 1024, while the product's error is below 2^-52.  Other operands take
// the IEEE division itself.
__device__ __forceinline__ void div_path_len(float a, float b, int n, double inv, float& qa,
                                             float& qb) {
    // tiny operands: bits in [1, 2^-100), i.e. bits - 1 below those of 2^-100 - 1
    const unsigned ta = __float_as_uint(a) - 1u, tb = __float_as_uint(b) - 1u;
    const bool fast = n < 1024 && min(ta, tb) >= __float_as_uint(0x1p-100f) - 1u;
    if (fast) {
        qa = (float)((double)a * inv);
        qb = (float)((double)b * inv);
    } else {
        const float np = (float)(n + 1);
        qa = a / np;
        qb = b / np;
    }
}

// The parameters of Eqs. (1)-(3), and the image they are evaluated on.
struct Eqs {
    const float4* img;     // packed texels
    int W;
    bool near;             // 32-bit byte offsets from near_img reach every texel of a path,
                           // and every path is below 46340 steps
    const float4* near_img;   // the texel of pixel (near_x, near_y)
    int near_x, near_y;
    float lambda, oml, gamma, spw;
};

// The near walk's fields for an image that it serves as a whole.
__device__ __forceinline__ void near_all(Eqs& q) {
    q.near = true;
    q.near_img = q.img;
    q.near_x = q.near_y = 0;
}

// The box of a work item's pixels and path endpoints, which holds its paths, too.
struct Box {
    int x0, y0, x1, y1;    // inclusive
    __device__ __forceinline__ void add(int x, int y) {
        x0 = min(x0, x);
        y0 = min(y0, y);
        x1 = max(x1, x);
        y1 = max(y1, y);
    }
};

// Whether the near walk serves the paths of a box (uniform), from its corner: in an
// image of 2^28 pixels and more, or of W + H >= 46340, nearly every item's.  10
// iterations of 60000x400, k = 24000: 18.3 ms, 40.6 by walk_path alone; 18.0 of
// 40000x600, which is near as a whole.
__device__ __forceinline__ void near_box(Eqs& q, const Box& b) {
    const int w = b.x1 - b.x0, h = b.y1 - b.y0;
    q.near = w < 46340 && h < 46340 && (long long)h * q.W + w < 1LL << 28;
    q.near_img = q.img + ((long long)b.y0 * q.W + b.x0);
    q.near_x = b.x0;
    q.near_y = b.y0;
}

// A path from pixel (px, py) to the endpoint (cx, cy) of the cluster at ck = (l, a, b,
// x, y): its steps, 1 / (n + 1) and the spatial term of Eq. (3).
struct Path {
    int dx, dy, n;
    double inv;
    float dsp;
};

__device__ __forceinline__ Path path_of(const Eqs& q, const float (&ck)[5], int cx, int cy, int px,
                                        int py) {
    Path p;
    const float ax = (float)px - ck[3], ay = (float)py - ck[4];
    p.dx = cx - px;
    p.dy = cy - py;
    p.n = max(abs(p.dx), abs(p.dy));
    p.inv = path_recip(p.n);
    p.dsp = (ax * ax + ay * ay) * q.spw;
    return p;
}

// D of Eq. (3) from the colour distance of the path's first pixel and the sums over
// all its samples, and the factors A, B of Eqs. (1)-(2).
__device__ __forceinline__ float path_value(const Eqs& q, const Path& p, float dcp, float sc, float sw,
                                            float& A, float& B) {
    float qc, qw;                                  // sc / |P|, sw / |P|
    div_path_len(sc, sw, p.n, p.inv, qc, qw);
    A = q.lambda * dcp + q.oml * qc;               // Eq. (1)
    B = 1.0f + q.gamma * qw;                       // Eq. (2)
    return A * B + p.dsp;                          // Eq. (3)
}

// D of Eq. (3) of pixel (px, py), whose texel is fp, to the cluster at ck =
// (l, a, b, x, y) with endpoint (cx, cy), and its factors A, B of Eqs.
// (1)-(2); FP32, operation by operation.  cut: an infinite D may be returned
// once D is known to exceed thr's best (see Cut; A and B are then
// meaningless).
__device__ __forceinline__ float path_distance(const Eqs& q, const float (&ck)[5], float4 fp,
                                               int cx, int cy, int px, int py, bool cut_on,
                                               float thr, float& A, float& B) {
    const float l = ck[0], a = ck[1], b = ck[2];
    const Path p = path_of(q, ck, cx, cy, px, py);
    const float dcp = colour_dist(fp, l, a, b);
    float sc = dcp, sw = fp.w;                     // sample i = 0 is p itself
    if (q.near) {                                  // uniform
        Cut cut;
        cut.on = cut_on;
        if (cut_on) {
            const float rnp = __builtin_amdgcn_rcpf((float)(p.n + 1));
            cut.a0 = q.lambda * dcp;
            cut.f = q.oml * rnp;
            cut.g = q.gamma * rnp;
            cut.dsp = p.dsp;
            cut.thr = thr;
        }
        const unsigned row = 16u * (unsigned)q.W;
        walk_near(q.near_img, row * (unsigned)(py - q.near_y) + 16u * (unsigned)(px - q.near_x),
                  path_step(p.dx, p.dy, 16, (int)row), l, a, b, cut, sc, sw);
    } else {
        walk_path(q.img, py * q.W + px, 1, q.W, p.dx, p.dy, l, a, b, sc, sw);
        if (p.n > 0) {                             // sample i = n is the endpoint
            const float4 fc = q.img[(long long)cy * q.W + cx];
            sc = sc + colour_dist(fc, l, a, b);
            sw = sw + fc.w;
        }
    }
    return path_value(q, p, dcp, sc, sw, A, B);
}

// An LDS table over a box of texels, row-major.  The row pitch is 4 (mod 8) entries
// where that fits: the 8 rows of a wave's 8x8 block of pixels then lie evenly over the
// LDS banks.
struct Table {
    int x0, y0, pitch, rows;
    bool fits;             // in `cap` entries, and a row in the workgroup's lanes
};

__device__ __forceinline__ Table table_of(const Box& b, int cap, int lanes) {
    Table t;
    const int w = b.x1 - b.x0 + 1;
    t.x0 = b.x0;
    t.y0 = b.y0;
    t.rows = b.y1 - b.y0 + 1;
    t.pitch = w + ((12 - w % 8) % 8);
    if (t.pitch > lanes || (long long)t.pitch * t.rows > cap) t.pitch = w;
    t.fits = t.pitch <= lanes && (long long)t.pitch * t.rows <= cap;
    return t;
}

// Fills it with (d_c(q), w_q), column by column: lane tid keeps one column, c = tid
// mod pitch, of rows tid / pitch, tid / pitch + R, ... (R = WG / pitch, both as high
// multiplications by ceil(2^24 / pitch)), so that an entry costs one load, its colour
// distance and two index adds; four rows' loads in flight.  Entries past the box's
// width only pad the pitch.
template <int WG>
__device__ __forceinline__ void fill_table(float2* table, const Table& t,
                                           const float4* __restrict__ img, int W, float l, float a,
                                           float b) {
    const int tid = threadIdx.x;
    const unsigned m = (0x1000000u + (unsigned)t.pitch - 1u) / (unsigned)t.pitch;
    const int R = (int)__umulhi((unsigned)WG << 8, m);
    const int r0 = (int)__umulhi((unsigned)tid << 8, m);
    if (r0 >= R) return;                           // lanes past R pitch
    const int c = tid - r0 * t.pitch;
    const float4* p = img + ((long long)(t.y0 + r0) * W + min(t.x0 + c, W - 1));
    const long long dp = (long long)R * W;
    const int de = R * t.pitch;
    int e = tid, r = r0;
#define SCALP_ENTRY(f) make_float2(colour_dist(f, l, a, b), (f).w)
    for (; r + 3 * R < t.rows; r += 4 * R) {
        const float4 f0 = p[0], f1 = p[dp], f2 = p[2 * dp], f3 = p[3 * dp];
        table[e] = SCALP_ENTRY(f0);
        table[e + de] = SCALP_ENTRY(f1);
        table[e + 2 * de] = SCALP_ENTRY(f2);
        table[e + 3 * de] = SCALP_ENTRY(f3);
        p += 4 * dp;
        e += 4 * de;
    }
    if (r + R < t.rows) {
        const float4 f0 = p[0], f1 = p[dp];
        table[e] = SCALP_ENTRY(f0);
        table[e + de] = SCALP_ENTRY(f1);
        p += 2 * dp;
        e += 2 * de;
        r += 2 * R;
    }
    if (r < t.rows) {
        const float4 f = p[0];
        table[e] = SCALP_ENTRY(f);
    }
#undef SCALP_ENTRY
}

// path_distance over a table that holds the path.
__device__ __forceinline__ float table_distance(const Eqs& q, const float (&ck)[5], const Table& t,
                                                const float2* table, int cx, int cy, int px, int py,
                                                float& A, float& B) {
    const Path p = path_of(q, ck, cx, cy, px, py);
    const int at = (py - t.y0) * t.pitch + (px - t.x0);
    const float2 f = table[at];
    float sc = f.x, sw = f.y;                      // sample i = 0 is the pixel itself
    walk_table(table, 8u * (unsigned)at, path_step(p.dx, p.dy, 8, 8 * t.pitch), sc, sw);
    return path_value(q, p, f.x, sc, sw, A, B);
}

__device__ __forceinline__ int round_coord(float v, int hi) {
    int e = (int)floorf(v + 0.5f);
    e = e < 0 ? 0 : e;
    return e > hi ? hi : e;
}

// Workgroup index -> work item.  Workgroups are dispatched round-robin over
// the 8 XCDs; give each XCD a contiguous run of items so that neighbouring
// cells, whose paths overlap, share an L2.
__device__ __forceinline__ int xcd_remap(int b, int G) {
    const int q = G >> 3, rem = G & 7;
    const int x = b & 7, slot = b >> 3;
    return x < rem ? x * (q + 1) + slot : rem * (q + 1) + (x - rem) * q + slot;
}

// Cell (row ci, column cj) at position i of the cell order of the grid
// assignment: column strips ceil(nx / strips) cells wide (the last one
// narrower), row-major within a strip.  A bijection of [0, nx ny); strips = 1
// is row-major order.
__device__ __forceinline__ void cell_in_strips(int i, const Img& im, int& ci, int& cj) {
    const int tw = (int)im.dcol.d;
    const int s = fdiv(i, im.dstrip);
    const int x0 = s * tw;
    const int l = i - s * tw * im.ny;
    const bool last = im.nx - x0 < tw;
    const int w = last ? im.nx - x0 : tw;
    ci = last ? fdiv(l, im.dlast) : fdiv(l, im.dcol);
    cj = x0 + (l - ci * w);
}

template <typename Table>
__device__ __forceinline__ int find_image(Table start, int n, int v) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Pixel t of a cell of width cw and height ch, enumerated in 8-wide column
// strips walked serpentine (down, up, ...): 64 consecutive indices form a
// compact 8x8 block, so the lanes of a wave walk paths of similar length.
__device__ __forceinline__ void cell_pixel(int t, int cw, int ch, int& x, int& y) {
    const int nfull = cw >> 3, wr = cw & 7;
    const int fullpx = nfull * 8 * ch;
    int s, row, col;
    if (t < fullpx) {
        const int per = 8 * ch;
        s = t / per;
        const int r = t - s * per;
        row = r >> 3;
        col = 8 * s + (r & 7);
    } else {
        s = nfull;
        const int r = t - fullpx;
        row = r / wr;
        col = 8 * nfull + (r - row * wr);
    }
    y = (s & 1) ? (ch - 1 - row) : row;
    x = col;
}

// cell_pixel with its two divisions, by numbers uniform over the work item,
// as high multiplications (FastDiv; `fast` says that both are exact over the
// cell: t < cw ch against 8 ch, and against the last strip's 2 to 7 columns).
struct PixelMap {
    int cw, ch, per, fullpx;
    unsigned mper, mwr;
    bool fast;
};

// ceil(2^32 / d) for a last strip of d = 2 .. 7 columns.
__constant__ const unsigned kLastStrip[8] = {0u, 0u, 0x80000000u, 0x55555556u, 0x40000000u,
                                             0x33333334u, 0x2aaaaaabu, 0x24924925u};

__device__ __forceinline__ PixelMap pixel_map(const FastDiv (&dper)[2], int cw, int ch) {
    PixelMap p;
    p.cw = cw;
    p.ch = ch;
    p.per = 8 * ch;
    p.fullpx = (cw >> 3) * p.per;
    p.mper = ch == (int)(dper[0].d >> 3) ? dper[0].m : dper[1].m;
    p.mwr = kLastStrip[cw & 7];
    p.fast = p.mper != 0u;
    return p;
}

__device__ __forceinline__ void pixel_at(const PixelMap& p, int t, int& x, int& y) {
    if (!p.fast) {                                 // uniform
        cell_pixel(t, p.cw, p.ch, x, y);
        return;
    }
    int s, row;
    if (t < p.fullpx) {
        s = (int)__umulhi((unsigned)t, p.mper);
        const int r = t - s * p.per;
        row = r >> 3;
        x = 8 * s + (r & 7);
    } else {
        const int wr = p.cw & 7;
        const int r = t - p.fullpx;
        row = wr > 1 ? (int)__umulhi((unsigned)r, p.mwr) : r;
        s = p.cw >> 3;
        x = 8 * s + (r - row * wr);
    }
    y = (s & 1) ? (p.ch - 1 - row) : row;
}

// The candidates' centres as the bounds read them: the item's 9 superpixels
// are uniform over the workgroup, so their values come through the scalar
// cache into scalar registers (nothing writes centres or endpoints while an
// assignment pass runs).
typedef const __attribute__((address_space(4))) float* ConstF;
typedef const __attribute__((address_space(4))) int* ConstI;

// Rows and columns of the 3x3 candidates of a cell, clamped into the grid (a
// clamped one repeats another candidate of the cell), and which are inside
// (bit j: slot j).
struct Neighbours {
    int row[3], col[3];   // superpixel index of (row, column 0); column
    unsigned inside;
};

__device__ __forceinline__ Neighbours neighbours_of(int nx, int ny, int ci, int cj) {
    Neighbours g;
    g.row[0] = max(ci - 1, 0) * nx;
    g.row[1] = ci * nx;
    g.row[2] = min(ci + 1, ny - 1) * nx;
    g.col[0] = max(cj - 1, 0);
    g.col[1] = cj;
    g.col[2] = min(cj + 1, nx - 1);
    g.inside = 0x1ffu;
    if (ci == 0) g.inside &= ~0x007u;
    if (ci == ny - 1) g.inside &= ~0x1c0u;
    if (cj == 0) g.inside &= ~0x049u;
    if (cj == nx - 1) g.inside &= ~0x124u;
    return g;
}

constexpr unsigned kNoKey = 0xffffffffu;

// Keys of the 9 candidates of a pixel with texel f: the upper 28 bits of
// LB = lambda dcp + ds spw, with the slot in the low 4 bits; kNoKey for a slot
// outside the grid.  LB is what D of Eq. (3) cannot fall below: lambda is in
// [0, 1], gamma >= 0 and every colour distance and w is >= 0, so
// A >= lambda dcp and B >= 1, and FP32 rounding is monotone.  Here it is
// evaluated with fused operations (13 per candidate instead of 16), within
// 2^-21 of its exact value: a candidate is left out only when its key, cut to
// 28 bits, exceeds threshold(best).  The centres are read one row of
// candidates at a time (the barrier keeps the scheduler from holding all 45
// scalars at once, which spilled).
__device__ __forceinline__ void bound_keys(const Neighbours& g, ConstF cen, float spw, float4 f,
                                           int x, int y, float lambda, unsigned (&key)[9]) {
    const float fx = (float)x, fy = (float)y;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ConstF row = cen + 5LL * __builtin_amdgcn_readfirstlane(g.row[i]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < 3; ++jj) {
            const int j = 3 * i + jj;
            ConstF c = row + 5 * __builtin_amdgcn_readfirstlane(g.col[jj]);
            const float dl = f.x - c[0], da = f.y - c[1], db = f.z - c[2];
            const float ex = fx - c[3], ey = fy - c[4];
            const float dcp = __builtin_fmaf(db, db, __builtin_fmaf(da, da, dl * dl));
            const float lb = __builtin_fmaf(ex * ex + ey * ey, spw, lambda * dcp);
            const unsigned tag = (g.inside >> j) & 1u ? (unsigned)j : kNoKey;   // uniform
            key[j] = (__float_as_uint(lb) & ~15u) | tag;
        }
    }
}

// What a bound, or the value of a path cut short, must exceed to prove that D
// exceeds best: the margin of 2^-16 covers their rounding (a dozen operations
// and one reciprocal good to an ulp), and 2^-70 any absolute error that
// underflow can leave.
__device__ __forceinline__ float threshold(float best) {
    return fmaxf(best * (1.0f + 0x1p-16f), 0x1p-70f);
}

// The smallest key above `cur` (0xffffffff: the smallest of all), all ones
// when there is none.
__device__ __forceinline__ unsigned next_key(const unsigned (&key)[9], unsigned cur) {
    const unsigned c1 = cur + 1u;          // keys up to cur wrap to [2^32 - c1, 2^32)
    const unsigned a = min(min(key[0] - c1, key[1] - c1), key[2] - c1);
    const unsigned b = min(min(key[3] - c1, key[4] - c1), key[5] - c1);
    const unsigned c = min(min(key[6] - c1, key[7] - c1), key[8] - c1);
    unsigned next;
    return __builtin_add_overflow(min(min(a, b), c), c1, &next) ? 0xffffffffu : next;
}

// Lanes of m below this one.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Adds the number of lanes in m (a ballot of the lanes here, not 0) to *count
// and gives the n-th of them the old value + n.
__device__ __forceinline__ int wave_claim(int* count, unsigned long long m) {
    const int leader = __ffsll((long long)m) - 1;
    int at = 0;
    if ((int)(threadIdx.x & 63) == leader) at = atomicAdd(count, __popcll(m));
    return __builtin_amdgcn_readlane(at, leader) + lanes_below(m);
}

__device__ __forceinline__ float key_bound(unsigned key) { return __uint_as_float(key & ~15u); }

// Sum over the lanes up to and including this one, in six DPP steps (no LDS
// traffic): row prefix sums by shifts of 1, 2, 4 and 8 lanes, then the last lane
// of each row is added to the next row (row_bcast:15) and lane 31 to rows 2 and 3
// (row_bcast:31).  All lanes must be active.
__device__ __forceinline__ int wave_scan_incl(int v) {
#define SCALP_SCAN_STEP(ctrl, rows) \
    v += __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xf, false)
    SCALP_SCAN_STEP(0x111, 0xf);
    SCALP_SCAN_STEP(0x112, 0xf);
    SCALP_SCAN_STEP(0x114, 0xf);
    SCALP_SCAN_STEP(0x118, 0xf);
    SCALP_SCAN_STEP(0x142, 0xa);
    SCALP_SCAN_STEP(0x143, 0xc);
#undef SCALP_SCAN_STEP
    return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Minimum and maximum over the 64 lanes of a wave (all lanes active), the
// same value in every lane.
__device__ __forceinline__ int wave_min_i32(int v) {
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ int wave_max_i32(int v) {
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return __builtin_amdgcn_readfirstlane(v);
}

}  // namespace dev
}  // namespace scalp
