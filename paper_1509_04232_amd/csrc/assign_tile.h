// Device code shared by the association launches (one round each) and the
// rounds launch (all rounds of a frame): the distances, the choice of each
// pixel's centre among the nine staged candidates, and the accumulation of
// the pixels into the workgroup's bins.  See assign.hip for the method.
#pragma once

#include "slic_internal.h"

#pragma clang fp contract(off)

namespace slic {
namespace {

constexpr int kThreads = 256;
constexpr unsigned kCertify = 160;  // distance of two keys
// Infinite distance, the last slot: bounds the second key.  A given centre may
// lie so far out that its distances overflow, and with m = 0 its spatial term
// is then 0 * inf.  Under Eq. 1 an infinite or undefined distance is then never
// certified as the best (the cells outside the grid would win), and the pixel
// stays in its own cell.  Under the squared-sum distance an infinite one is not
// settled either; where all nine are undefined (no cell outside the grid among
// them) the first is taken.  The keys have no sign, so that an undefined
// distance comes after an infinite one.
constexpr unsigned kNoKey = 0x7F80000Fu, kKeyBits = 0x7FFFFFF0u;

// Reference Eq. 1 distance: the exact operation sequence of the definition.
__device__ __forceinline__ float eq1_reference(float cl, float ca, float cb, float cx, float cy,
                                               float l, float a, float b, float xf, float yf,
                                               float wgt) {
    const float dl = cl - l, da = ca - a, db = cb - b;
    float s = dl * dl;
    s = s + da * da;
    s = s + db * db;
    const float dlab = sqrtf(s);
    const float dx = cx - xf, dy = cy - yf;
    float t = dx * dx;
    t = t + dy * dy;
    const float dxy = sqrtf(t);
    const float sp = wgt * dxy;
    return dlab + sp;
}

// Smallest and middle of three keys (the forms that compile to one
// v_min3_u32 and one v_med3_u32).
__device__ __forceinline__ unsigned umin3(unsigned a, unsigned b, unsigned c) {
    return min(a, min(b, c));
}
__device__ __forceinline__ unsigned umed3(unsigned a, unsigned b, unsigned c) {
    return max(min(a, b), min(max(a, b), c));
}

// 16-byte global accesses (builtin vector types: HIP's float4 and int4 are
// classes whose members assume generic pointers).
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef int vi4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 load_f4(gmem<const float>* p) {
    const vf4 v = *reinterpret_cast<gmem<const vf4>*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ void store_f4(gmem<float>* p, float4 v) {
    *reinterpret_cast<gmem<vf4>*>(p) = vf4{v.x, v.y, v.z, v.w};
}

__device__ __forceinline__ void store_i4(gmem<int32_t>* p, int a, int b, int c, int d) {
    *reinterpret_cast<gmem<vi4>*>(p) = vi4{a, b, c, d};
}

typedef float vf2 __attribute__((ext_vector_type(2)));
typedef int vi2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ vf2 load_f2(gmem<const float>* p) {
    return *reinterpret_cast<gmem<const vf2>*>(p);
}

__device__ __forceinline__ void store_i2(gmem<int32_t>* p, int a, int b) {
    *reinterpret_cast<gmem<vi2>*>(p) = vi2{a, b};
}

// The squared-sum distance of the SLIC paper the method builds on (an
// option): d_lab^2 + w^2 d_xy^2 in FP32 in this order, no square roots, so
// the values compared are the exact ones.
__device__ __forceinline__ float dist_squared(float cl, float ca, float cb, float cx, float dy2,
                                              float l, float a, float b, float xf, float wgt) {
    const float dl = cl - l, da = ca - a, db = cb - b;
    float s = dl * dl;
    s = s + da * da;
    s = s + db * db;
    const float dx = cx - xf;
    float t = dx * dx;
    t = t + dy2;
    const float w2 = wgt * wgt;
    const float sp = w2 * t;
    return s + sp;
}

// Fast Eq. 1 distance (fused multiply-adds, hardware square root); dy2 is
// the squared vertical offset, shared by the pixels of a row.
__device__ __forceinline__ float eq1_fast(float cl, float ca, float cb, float cx, float dy2,
                                          float l, float a, float b, float xf, float wgt) {
    const float dl = cl - l, da = ca - a, db = cb - b;
    const float s = __builtin_fmaf(db, db, __builtin_fmaf(da, da, dl * dl));
    const float dx = cx - xf;
    const float t = __builtin_fmaf(dx, dx, dy2);
    return __builtin_fmaf(wgt, __builtin_amdgcn_sqrtf(t), __builtin_amdgcn_sqrtf(s));
}

// Reference argmin over the nine candidates of one pixel (near ties only).
// A cell outside the grid is staged with an infinite colour distance and
// every distance of a cell inside it is finite (the compactness bound), so
// the strict test below never selects an outside cell; the pixel's own cell
// (slot 4) is the starting choice.
__device__ __forceinline__ int reference_slot(const float4* cen4, const float* ceny, int base,
                                               int ncx, float l, float a, float b, float xf,
                                               float yf, float wgt) {
    float bref = __builtin_huge_valf();
    int sref = 4;
#pragma unroll 1
    for (int c = 0; c < 9; ++c) {
        const int li = base + (c / 3) * ncx + (c % 3);
        const float4 q = cen4[li];
        const float d = eq1_reference(q.x, q.y, q.z, q.w, ceny[li], l, a, b, xf, yf, wgt);
        if (d < bref) {
            bref = d;
            sref = c;
        }
    }
    return sref;
}

// The same under the squared-sum distance, where two keys agree: the lowest
// distance bits, the lowest slot on ties.
__device__ __forceinline__ int squared_slot(const float4* cen4, const float* ceny, int base, int ncx,
                                            float l, float a, float b, float xf, float yf, float wgt) {
    unsigned bref = ~0u;
    int sref = 0;
#pragma unroll 1
    for (int c = 0; c < 9; ++c) {
        const int li = base + (c / 3) * ncx + (c % 3);
        const float4 q = cen4[li];
        const float dy = ceny[li] - yf;
        const unsigned d =
            __float_as_uint(dist_squared(q.x, q.y, q.z, q.w, dy * dy, l, a, b, xf, wgt));
        if (d < bref) {
            bref = d;
            sref = c;
        }
    }
    return sref;
}

// Shared-memory layout (dynamic): for every cell of the staged window
// (the workgroup's cells plus a one-cell ring, out-of-grid cells included):
//   float4 cen4[n] (L, a, b, x), float ceny[n], int kidx[n] (-1: none), then
//   `copies` sets of u64 bins[4][n] (sum qL, sum qa, sum qb, packed x | y << 24
//   | count << 48, positions from the tile's corner; at most 2048 pixels per
//   workgroup), each one word longer than its bins.
// Lane l adds to copy l % copies: neighbouring lanes mostly hold the same
// cell, and atomics of a wavefront to one address are done one by one.  With
// one copy a 3631 x 3859 frame at S = 84 (a wavefront in one to four cells)
// took 1,435 us, with eight 1,163 us; 933 x 800 at S = 27 164 and 151 us.  At
// S = 8 and 16, where a wavefront spans many cells, it makes no difference.
__host__ __device__ inline int bin_stride(int ncells) { return 4 * ncells + 1; }
inline size_t assign_lds_bytes(int ncells, int copies) {
    return static_cast<size_t>(ncells) * 24 + static_cast<size_t>(copies) * bin_stride(ncells) * 8 + 16;
}
// Copies for a window of n cells: eight where they cost at most 8 KB.
inline int bin_copies(int ncells) {
    int c = 8;
    while (c > 1 && c * ncells > 256) c /= 2;
    return c;
}

// Launch shape of a variant: each thread owns VEC horizontally adjacent
// pixels in each of ROWS consecutive rows.  VEC = 2 or 4 uses 8- or 16-byte
// loads and evaluates each staged centre once for the VEC pixels, so it
// needs them in one cell (S % VEC == 0) and aligned rows (width % VEC == 0).
template <int VEC, int ROWS, int TX = (VEC == 4 ? 16 : 32)>
struct Shape {
    static constexpr int kTX = TX;  // threads per row
    static constexpr int kTY = kThreads / kTX;
    static constexpr int kTileW = kTX * VEC;
    static constexpr int kTileH = kTY * ROWS;
    static constexpr int kPx = VEC * ROWS;
};

__device__ __forceinline__ void add_bin(unsigned long long* bins, int ncells, int cell,
                                        long long rl, long long ra, long long rb,
                                        unsigned long long rxyc) {
    atomicAdd(bins + cell, static_cast<unsigned long long>(rl));
    atomicAdd(bins + ncells + cell, static_cast<unsigned long long>(ra));
    atomicAdd(bins + 2 * ncells + cell, static_cast<unsigned long long>(rb));
    atomicAdd(bins + 3 * ncells + cell, rxyc);
}

// Selection among the nine candidates of a row of VEC pixels that lie in one
// cell (base: its left upper candidate's window entry): the winners' window
// cells, and where the keys do not settle the choice.  Under Eq. 1 that is
// where two fast values are too near to certify it; the squared-sum distance
// is computed exactly, so only where the two smallest agree in all the bits
// that a key keeps (keys of 32 bits for 64 took 154 instructions per pixel for
// 189, and a 1080p frame of ten rounds 179 us for 193).  (All rows of a thread
// against one load of each candidate took 8 instructions per pixel less, and
// more time: 104 registers for 86.)
template <int VEC, int DIST>
__device__ __forceinline__ void find_row(const float4* cen4, const float* ceny, int ncx, int base,
                                         float wgt, int x, int y, const float (&pl)[VEC],
                                         const float (&pa)[VEC], const float (&pb)[VEC],
                                         bool (&near)[VEC], int (&cellv)[VEC]) {
    const float yf = static_cast<float>(y);
    // the keys of one row of candidates at a time: smallest and middle of
    // three (one instruction each), then of the three rows
    unsigned lo[3][VEC], mid[3][VEC];
#pragma unroll
    for (int cr = 0; cr < 3; ++cr) {
        unsigned key[3][VEC];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            const int li = base + cr * ncx + cc;
            const float4 q = cen4[li];
            const float dy = ceny[li] - yf;
            const float dy2 = dy * dy;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const float xf = static_cast<float>(x + v);
                const float d =
                    DIST == 1 ? dist_squared(q.x, q.y, q.z, q.w, dy2, pl[v], pa[v], pb[v], xf, wgt)
                              : eq1_fast(q.x, q.y, q.z, q.w, dy2, pl[v], pa[v], pb[v], xf, wgt);
                key[cc][v] = (__float_as_uint(d) & kKeyBits) | static_cast<unsigned>(4 * cr + cc);
            }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            lo[cr][v] = umin3(key[0][v], key[1][v], key[2][v]);
            mid[cr][v] = umed3(key[0][v], key[1][v], key[2][v]);
        }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        const unsigned best = umin3(lo[0][v], lo[1][v], lo[2][v]);
        const unsigned second = umin3(umed3(lo[0][v], lo[1][v], lo[2][v]),
                                      umin3(mid[0][v], mid[1][v], mid[2][v]), kNoKey);
        near[v] = DIST == 1 ? (second ^ best) < 16u
                            : static_cast<int>(second - best) < static_cast<int>(kCertify);
        cellv[v] = base + static_cast<int>((best >> 2) & 3u) * ncx + static_cast<int>(best & 3u);
    }
}

// The window cell of the centre nearest to each pixel of the thread (rows yb
// .. yb + ROWS - 1, columns x .. x + VEC - 1).  cen4, ceny, kidx: the staged
// window of ncx columns; gx_rel: window column of the left candidates.
template <int VEC, int ROWS, int DIST>
__device__ __forceinline__ void find_cells(const float4* cen4, const float* ceny, const int* kidx,
                                           int ncx, int gx_rel, int gy_lo, const AssignImage& g,
                                           int x, int yb, const float (&pl)[ROWS][VEC],
                                           const float (&pa)[ROWS][VEC],
                                           const float (&pb)[ROWS][VEC],
                                           int (&cellv)[ROWS][VEC]) {
    int rowbase[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        rowbase[r] = (g.by_S.quotient(min(yb + r, g.h - 1)) - gy_lo - 1) * ncx + gx_rel;
    bool near[ROWS][VEC];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        find_row<VEC, DIST>(cen4, ceny, ncx, rowbase[r], g.wgt, x, yb + r, pl[r], pa[r], pb[r],
                            near[r], cellv[r]);
    // near ties (a few pixels per frame): the reference argmin, after the
    // fast pass, whose keys are then dead, and inline (a call would pin the
    // fast pass's live values to the callee-saved registers)
    bool any = false;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int v = 0; v < VEC; ++v) any = any || near[r][v];
    if (any) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                if (!near[r][v]) continue;
                const float xf = static_cast<float>(x + v), yf = static_cast<float>(yb + r);
                const int slot = DIST == 1 ? squared_slot(cen4, ceny, rowbase[r], ncx, pl[r][v], pa[r][v],
                                                          pb[r][v], xf, yf, g.wgt)
                                           : reference_slot(cen4, ceny, rowbase[r], ncx, pl[r][v],
                                                            pa[r][v], pb[r][v], xf, yf, g.wgt);
                cellv[r][v] = rowbase[r] + (slot / 3) * ncx + (slot % 3);
                // (squared: a cell outside the grid comes first only where no
                // distance is finite; the own cell is then taken)
                if (DIST == 1 && kidx[cellv[r][v]] < 0) cellv[r][v] = rowbase[r] + ncx + 1;
            }
        }
    }
}

// Adds the thread's pixels (tile columns txp .. and rows typ ..; the first
// `rows_in` rows lie in the image) to the bins, runs of equal cells at once.
// Odd rows go from right to left, so that a run goes on into the next row.
// A run's positions are kept as its count and its sums of v << 8 and r << 16:
// one addition per pixel, expanded when the run ends.
template <int VEC, int ROWS>
__device__ __forceinline__ void accumulate(unsigned long long* bins, int ncells, const int (&cellv)[ROWS][VEC],
                                           const float (&pl)[ROWS][VEC],
                                           const float (&pa)[ROWS][VEC],
                                           const float (&pb)[ROWS][VEC], int txp, int typ,
                                           int rows_in) {
    const float scale = static_cast<float>(1 << kQShift);
    int run_cell = -1;
    int rl = 0, ra = 0, rb = 0;
    unsigned rpos = 0;
    auto flush = [&]() {
        const unsigned n = rpos & 255u;
        const unsigned sx = n * txp + ((rpos >> 8) & 255u);
        const unsigned sy = n * typ + (rpos >> 16);
        // at most 8 pixels in 64 x 32: sx stays below 2^24 and sy below 2^8,
        // so the low word holds both
        add_bin(bins, ncells, run_cell, rl, ra, rb,
                static_cast<unsigned long long>(sx | (sy << 24)) |
                    (static_cast<unsigned long long>(n << 16) << 32));
        rl = ra = rb = 0;
        rpos = 0;
    };
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if (r >= rows_in) continue;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int v = (r & 1) ? VEC - 1 - i : i;
            const int cell = cellv[r][v];
            if (cell != run_cell) {
                if (run_cell >= 0) flush();
                run_cell = cell;
            }
            rl += static_cast<int>(rintf(pl[r][v] * scale));
            ra += static_cast<int>(rintf(pa[r][v] * scale));
            rb += static_cast<int>(rintf(pb[r][v] * scale));
            rpos += 1u + (static_cast<unsigned>(v) << 8) + (static_cast<unsigned>(r) << 16);
        }
    }
    if (run_cell >= 0) flush();
}

}  // namespace
}  // namespace slic
