// Weight build of the MLBM on gfx950: space-filling-curve ordering, stencil
// and owner searches on a uniform cell grid, and the FP64 local RBF solves.
//
// This translation unit is compiled with -ffp-contract=off: squared distances
// are rounded exactly as written, so stencil ties are decided on bitwise equal
// distances and then by user index, as in the definition of the stencil.
#include <cfloat>
#include <climits>
#include <type_traits>
#include <utility>

#include "common.h"

namespace mlbm {
namespace {

__device__ __forceinline__ double min_image(double d, double L) {
    if (L > 0.0) {
        if (d > 0.5 * L) d -= L;
        else if (d < -0.5 * L) d += L;
    }
    return d;
}

__device__ __forceinline__ double dist2(double ax, double ay, double bx, double by,
                                        double Lx, double Ly) {
    double dx = min_image(bx - ax, Lx);
    double dy = min_image(by - ay, Ly);
    return dx * dx + dy * dy;
}

// Index of cell (x, y) along the Hilbert curve of a 2^order x 2^order grid
// (the classic quadrant-rotation construction).
__device__ uint32_t hilbert_index(uint32_t x, uint32_t y, int order) {
    uint32_t d = 0;
    const uint32_t side = 1u << order;
    for (uint32_t s = side >> 1; s > 0; s >>= 1) {
        uint32_t rx = (x & s) ? 1u : 0u;
        uint32_t ry = (y & s) ? 1u : 0u;
        d += s * s * ((3u * rx) ^ ry);
        if (ry == 0) {
            if (rx == 1) {
                x = side - 1 - x;
                y = side - 1 - y;
            }
            uint32_t t = x;
            x = y;
            y = t;
        }
    }
    return d;
}

__device__ __forceinline__ void cell_of(const Geo &g, double x, double y, int &cx, int &cy) {
    double fx = floor((x - g.x0) / g.cw);
    double fy = floor((y - g.y0) / g.ch);
    cx = fx < 0 ? 0 : (fx >= g.gx ? g.gx - 1 : (int)fx);
    cy = fy < 0 ? 0 : (fy >= g.gy ? g.gy - 1 : (int)fy);
}

// Bounding box of an open cloud (one workgroup).
__global__ __launch_bounds__(1024) void k_geo_bbox(Geo *geo, const double *x, const double *y,
                                                   int n, int gx, int gy, int hb) {
    __shared__ double s[4][1024];
    double mnx = DBL_MAX, mny = DBL_MAX, mxx = -DBL_MAX, mxy = -DBL_MAX;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        mnx = fmin(mnx, x[i]);
        mxx = fmax(mxx, x[i]);
        mny = fmin(mny, y[i]);
        mxy = fmax(mxy, y[i]);
    }
    s[0][threadIdx.x] = mnx;
    s[1][threadIdx.x] = mxx;
    s[2][threadIdx.x] = mny;
    s[3][threadIdx.x] = mxy;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s[0][threadIdx.x] = fmin(s[0][threadIdx.x], s[0][threadIdx.x + w]);
            s[1][threadIdx.x] = fmax(s[1][threadIdx.x], s[1][threadIdx.x + w]);
            s[2][threadIdx.x] = fmin(s[2][threadIdx.x], s[2][threadIdx.x + w]);
            s[3][threadIdx.x] = fmax(s[3][threadIdx.x], s[3][threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double ex = s[1][0] - s[0][0], ey = s[3][0] - s[2][0];
        double e = fmax(fmax(ex, ey), 1e-300);
        Geo g;
        g.x0 = s[0][0] - 1e-9 * e;
        g.y0 = s[2][0] - 1e-9 * e;
        g.cw = (ex + 2e-9 * e) / gx;
        g.ch = (ey + 2e-9 * e) / gy;
        if (!(g.cw > 0)) g.cw = 1.0;
        if (!(g.ch > 0)) g.ch = 1.0;
        g.Lx = 0.0;
        g.Ly = 0.0;
        g.gx = gx;
        g.gy = gy;
        g.hb = hb;
        g.pad = 0;
        *geo = g;
    }
}

// First kernel of a cloud's build: the cells and the counters empty, and the
// geometry of a periodic cloud, whose values the host knows.
__global__ __launch_bounds__(256) void k_begin(Geo *geo, Geo periodic, int ncells, int32_t *cstart,
                                               int32_t *cend, int nkeys, int32_t *cnt) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ncells) cstart[i] = cend[i] = 0;
    if (i < nkeys) cnt[i] = 0;
    if (i == 0 && periodic.Lx > 0.0) *geo = periodic;
}

// Hilbert key of every node's cell. With counters a node also takes the next
// place in its key (vals[u]), without them vals[u] = u.
__global__ __launch_bounds__(256) void k_keys(const Geo *__restrict__ geo,
                                              const double *__restrict__ x,
                                              const double *__restrict__ y, int n, uint32_t *keys,
                                              int32_t *vals, int32_t *cnt) {
    int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    Geo g = *geo;
    int cx, cy;
    cell_of(g, x[u], y[u], cx, cy);
    const uint32_t k = hilbert_index((uint32_t)cx, (uint32_t)cy, g.hb);
    keys[u] = k;
    vals[u] = cnt ? atomicAdd(&cnt[k], 1) : u;
}

// Counting sort: the nodes of key k, in no order, at off[k] and up.
__global__ __launch_bounds__(256) void k_place(int n, const uint32_t *__restrict__ keys,
                                               const int32_t *__restrict__ vals,
                                               const int32_t *__restrict__ off,
                                               int32_t *__restrict__ placed) {
    const int u = blockIdx.x * blockDim.x + threadIdx.x;
    if (u < n) placed[off[keys[u]] + vals[u]] = u;
}

// Nodes in internal order: by key, nodes of one key by user index. COUNTED: the
// order is found here from the placed nodes and the keys' offsets, a node's rank
// in its key being the number of smaller user indices there (two nodes a cell on
// average; the stencil search scans the same cells). Otherwise perm and the
// sorted keys hold it. Also empties the owner lists' counters and the search's
// list (redo).
template <bool COUNTED>
__global__ __launch_bounds__(256) void k_scatter_sorted(
    const Geo *__restrict__ geo, const double *__restrict__ x, const double *__restrict__ y,
    const uint8_t *__restrict__ nt, int32_t *__restrict__ perm, const uint32_t *__restrict__ keys,
    const int32_t *__restrict__ placed, const int32_t *__restrict__ off, int nkeys, int n, double *xs,
    double *ys, uint8_t *ntype, int32_t *iperm, int32_t *cstart, int32_t *cend, int32_t *owned,
    int32_t *redo) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    owned[t] = 0;
    if (t == 0) redo[0] = 0;
    const Geo g = *geo;
    const int u = COUNTED ? placed[t] : perm[t];
    const double px = x[u], py = y[u];
    int cx, cy;
    cell_of(g, px, py, cx, cy);
    const int c = cy * g.gx + cx;
    int p = t;
    if (COUNTED) {
        const uint32_t k = keys[u];   // by user index
        const int b = off[k], e = (int)k + 1 < nkeys ? off[k + 1] : n;
        p = b;
        for (int q = b; q < e; ++q) p += placed[q] < u ? 1 : 0;
        perm[p] = u;
        if (t == b) {
            cstart[c] = b;
            cend[c] = e;
        }
    } else {
        const uint32_t k = keys[p];   // sorted
        if (p == 0 || keys[p - 1] != k) cstart[c] = p;
        if (p == n - 1 || keys[p + 1] != k) cend[c] = p + 1;
    }
    xs[p] = px;
    ys[p] = py;
    ntype[p] = nt ? nt[u] : (uint8_t)0;
    iperm[u] = p;
}

// Error words to "none" (no singular node, no flags, no reported node), records to 0.
__global__ __launch_bounds__(256) void k_reset(int32_t *err, int32_t *stats, int nstats) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 3) err[i] = i == kErrFlags ? 0 : INT_MAX;
    if (i < nstats) stats[i] = 0;
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Cell of Chebyshev ring r around (cx, cy) number t (0 <= t < 8r, or t = 0 for
// r = 0): its index, or -1 where an open axis has no such cell. Periodic axes
// wrap.
__device__ __forceinline__ int ring_cell(const Geo &g, int cx, int cy, int r, int t) {
    const int span = 2 * r + 1;
    int dx, dy;
    if (r == 0) {
        dx = 0;
        dy = 0;
    } else if (t < span) {        // bottom row
        dx = t - r;
        dy = -r;
    } else if (t < 2 * span) {    // top row
        dx = t - span - r;
        dy = r;
    } else {                      // left and right columns without corners
        const int v = t - 2 * span;
        dx = (v & 1) ? r : -r;
        dy = (v >> 1) - r + 1;
    }
    int ix = cx + dx, iy = cy + dy;
    if (g.Lx > 0.0) ix = (ix % g.gx + g.gx) % g.gx;
    else if (ix < 0 || ix >= g.gx) return -1;
    if (g.Ly > 0.0) iy = (iy % g.gy + g.gy) % g.gy;
    else if (iy < 0 || iy >= g.gy) return -1;
    return iy * g.gx + ix;
}

// Scan the cells of Chebyshev ring r around (cx, cy); `body(q)` runs for every
// node q in those cells.
template <class F>
__device__ __forceinline__ void for_ring(const Geo &g, const int32_t *__restrict__ cstart,
                                         const int32_t *__restrict__ cend, int cx, int cy,
                                         int r, F &&body) {
    const int count = r == 0 ? 1 : 8 * r;
    for (int t = 0; t < count; ++t) {
        const int c = ring_cell(g, cx, cy, r, t);
        if (c < 0) continue;
        const int e = cend[c];
        for (int q = cstart[c]; q < e; ++q) body(q);
    }
}

// LDS of the group of lanes that looks for one node's stencil.
struct KnnList {
    double *d;       // [CAP] squared distances of the listed nodes
    int *q;          // [CAP] the nodes
    int *cnt;
    unsigned *occ;   // [2]
};

// Stencil of node p: p itself, then the K - 1 closest other nodes by (squared
// distance, user index), by G lanes of a wavefront (all of its lanes take part;
// groups of lanes have nodes of their own, and live tells whether there is one).
// The nodes within a radius that should hold a few more than K - 1 (from the count
// of the 5 x 5 cells around) are listed in LDS; a list that comes out short, or
// longer than CAP, is taken again with another radius. The place of an entry in
// the stencil is then the number of entries before it, counted by comparing it with
// all of them: CAP / G entries a lane and one LDS read for every entry of the list.
// Equal distances are decided by the user index in a second pass, which only lists
// that have them (lattices) take.
// A whole wavefront (G = 64) shares crowded cells among its lanes, takes the third
// and later radii from the counts of 32 shells between radii known to hold too few
// and too many (a node outside a dense part of an uneven cloud meets hundreds of
// nodes within a thousandth of the radius), and where no radius brings the list
// into [K - 1, CAP] (more than CAP nodes at one distance) finds the nodes one after
// another. Eight lanes give up, and return false with nothing written, after four
// radii, at a crowded cell, or at a block of cells too large for them.
constexpr int kCrowded = 64;        // nodes of a cell
constexpr int kManyCells = 1024;    // cells of a block; also nodes where a block would wrap
template <int CAP, int G>
__device__ __forceinline__ bool knn_by_radius(const Geo &g, const double *__restrict__ xs,
                                              const double *__restrict__ ys,
                                              const int32_t *__restrict__ perm,
                                              const int32_t *__restrict__ cstart,
                                              const int32_t *__restrict__ cend, int n, int K, int p,
                                              bool live, const KnnList &l,
                                              int32_t *__restrict__ nbr) {
    constexpr bool WAVE = G == 64;
    constexpr int E = (CAP + G - 1) / G, TRIES = WAVE ? 16 : 4;
    const int gl = threadIdx.x % G;
    const double px = xs[p], py = ys[p];
    const bool perx = g.Lx > 0.0, pery = g.Ly > 0.0;
    int cx, cy;
    cell_of(g, px, py, cx, cy);
    // cell (ix, iy) of the grid, or -1 outside an open one
    auto cell = [&](int ix, int iy) {
        if (perx) ix += ix < 0 ? g.gx : ix >= g.gx ? -g.gx : 0;
        if (pery) iy += iy < 0 ? g.gy : iy >= g.gy ? -g.gy : 0;
        return ix < 0 || iy < 0 || ix >= g.gx || iy >= g.gy ? -1 : iy * g.gx + ix;
    };
    const int need = K - 1;
    double lim2;   // squared radius of the list
    {
        int sum = 0, cells = 0;
        if (g.gx >= 5 && g.gy >= 5) {
#pragma unroll
            for (int t = 0; t < (24 + G) / G; ++t) {
                const int i = gl + t * G;
                const int c = i < 25 ? cell(cx + i % 5 - 2, cy + i / 5 - 2) : -1;
                if (c >= 0) {
                    sum += cend[c] - cstart[c];
                    ++cells;
                }
            }
        }
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
            sum += __shfl_xor(sum, off);
            cells += __shfl_xor(cells, off);
        }
        const double per_cell = cells ? (double)sum / cells : (double)n / ((double)g.gx * g.gy);
        lim2 = (1.15 * need + 5.0) / (3.14159265 * per_cell) * g.cw * g.ch;
    }
    // take(q) for every node closer than the radius, and for some beyond it; false if
    // this is not for eight lanes
    auto each_near = [&](auto &&take) {
        // they lie at most rx, ry cells away (the margin covers the rounding of a
        // node's cell)
        const double lim = sqrt(lim2) * (1.0 + 1e-9);
        const double fx = floor(lim / g.cw) + 1.0, fy = floor(lim / g.ch) + 1.0;
        if ((perx && 2.0 * fx + 1.0 > g.gx) || (pery && 2.0 * fy + 1.0 > g.gy)) {
            if (!WAVE && n > kManyCells) return false;
            for (int q = gl; q < n; q += G) take(q);   // a block would meet cells twice
            return true;
        }
        // (an open grid: the block ends at its edge)
        const int rx = (int)fmin(fx, (double)g.gx), ry = (int)fmin(fy, (double)g.gy);
        const int x0 = perx ? cx - rx : max(cx - rx, 0);
        const int x1 = perx ? cx + rx : min(cx + rx, g.gx - 1);
        const int y0 = pery ? cy - ry : max(cy - ry, 0);
        const int y1 = pery ? cy + ry : min(cy + ry, g.gy - 1);
        const int w = x1 - x0 + 1, count = w * (y1 - y0 + 1);
        if (!WAVE && count > kManyCells) return false;
        int ix = gl % w, iy = gl / w;
        const int sx = G % w, sy = G / w;
        bool crowded = false;
        for (int t = gl; (WAVE ? t - gl : t) < count; t += G) {
            int b = 0, e = 0;
            if (!WAVE || t < count) {
                const int c = cell(x0 + ix, y0 + iy);
                b = cstart[c];
                e = cend[c];
            }
            const bool shared = WAVE && e - b > 8;
            if (!WAVE && e - b > kCrowded) {
                crowded = true;
                e = b;
            }
            if (!shared)
                for (int q = b; q < e; ++q) take(q);
            if (WAVE) {
                for (uint64_t m = __ballot(shared); m != 0; m &= m - 1) {
                    const int from = __builtin_ctzll(m);
                    const int be = __builtin_amdgcn_readlane(e, from);
                    for (int q = __builtin_amdgcn_readlane(b, from) + gl; q < be; q += G) take(q);
                }
            }
            ix += sx;
            iy += sy;
            if (ix >= w) {
                ix -= w;
                ++iy;
            }
        }
        return !crowded;
    };
    constexpr int BINS = 32;   // (in the list's place)
    int cnt = 0, below = 0;
    bool ok = false;
    double lo2 = 0.0, hi2 = DBL_MAX;   // squared radii known to hold too few (below), too many
    for (int tries = 0; tries < TRIES && !ok; ++tries) {
        if (WAVE && tries >= 2 && hi2 < DBL_MAX) {
            for (int b = gl; b < BINS; b += G) l.q[b] = 0;
            wave_lds_sync();
            const double width = (hi2 - lo2) / BINS;
            lim2 = hi2;
            each_near([&](int q) {
                const double d = dist2(px, py, xs[q], ys[q], g.Lx, g.Ly);
                if (d >= lo2 && d < hi2 && q != p)
                    atomicAdd(&l.q[(int)fmin((d - lo2) / width, BINS - 1.0)], 1);
            });
            wave_lds_sync();
            int b = 0;
            while (b < BINS - 1 && below + l.q[b] < need) below += l.q[b++];
            const bool few = below + l.q[b] <= CAP;
            wave_lds_sync();
            if (b < BINS - 1) hi2 = lo2 + (b + 1) * width;
            lo2 += b * width;
            if (!few) continue;
            lim2 = hi2;
        }
        if (gl == 0) *l.cnt = 0;
        wave_lds_sync();
        constexpr int kGiveUp = 1 << 30;   // (above any count of nodes)
        if (!each_near([&](int q) {
                const double d = dist2(px, py, xs[q], ys[q], g.Lx, g.Ly);
                if (d < lim2 && q != p) {
                    const int at = atomicAdd(l.cnt, 1);
                    if (at < CAP) {
                        l.d[at] = d;
                        l.q[at] = q;
                    }
                }
            }))
            atomicOr(reinterpret_cast<unsigned *>(l.cnt), (unsigned)kGiveUp);
        wave_lds_sync();
        cnt = *l.cnt;
        wave_lds_sync();
        if (cnt >= kGiveUp) break;
        ok = cnt >= need && cnt <= CAP;
        if (!ok) {
            if (cnt < need) {
                lo2 = lim2;
                below = cnt;
            } else {
                hi2 = lim2;
            }
            const double f = (1.15 * need + 5.0) / (cnt > 0 ? cnt : 1);
            lim2 *= cnt < need ? fmin(fmax(f, 1.1), 4.0) : fmin(fmax(f, 0.25), 0.95);
            if (!(lim2 > lo2 && lim2 < hi2)) lim2 = sqrt(lo2) * sqrt(hi2);
        }
    }
    if (WAVE && !ok) {   // each next node: the closest one behind the last
        if (live && gl == 0) nbr[p] = p;
        double ld = -1.0;
        int lu = -1;
        lim2 = hi2;
        for (int k = 1; k < K; ++k) {
            double bd = DBL_MAX;
            int bu = INT_MAX, bq = p;   // (p: there is none, coordinates are not finite)
            each_near([&](int q) {
                const double d = dist2(px, py, xs[q], ys[q], g.Lx, g.Ly);
                if (!(d <= bd) || d < ld || q == p) return;
                const int u = perm[q];
                if ((d == ld && u <= lu) || (d == bd && u > bu)) return;
                bd = d;
                bu = u;
                bq = q;
            });
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const double od = __shfl_xor(bd, off);
                const int ou = __shfl_xor(bu, off), oq = __shfl_xor(bq, off);
                if (od < bd || (od == bd && ou < bu)) {
                    bd = od;
                    bu = ou;
                    bq = oq;
                }
            }
            ld = bd;
            lu = bu;
            if (live && gl == 0) nbr[(int64_t)k * n + p] = bq;
        }
        return true;
    }
    if (!ok) cnt = 0;   // (the lanes stay: the steps below work across the wavefront)
    double d[E];
    int rank[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        d[e] = e * G + gl < cnt ? l.d[e * G + gl] : -1.0;
        rank[e] = 0;
    }
    int top = cnt;   // the wavefront's longest list
#pragma unroll
    for (int off = G; off < 64; off <<= 1) top = max(top, __shfl_xor(top, off));
    top = __builtin_amdgcn_readfirstlane(top);
#pragma unroll 4
    for (int j = 0; j < cnt; ++j) {
        const double dj = l.d[j];
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e * G < top) rank[e] += dj < d[e];
    }
    // two entries at one place: equal distances
    if (gl < 2) l.occ[gl] = 0u;
    wave_lds_sync();
    bool tie = false;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * G + gl < cnt && rank[e] < need) {
            const unsigned bit = 1u << (rank[e] & 31);
            if (atomicOr(&l.occ[rank[e] >> 5], bit) & bit) tie = true;
        }
    if (__any(tie)) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e * G + gl < cnt) {
                const int u = perm[l.q[e * G + gl]];
                for (int j = 0; j < cnt; ++j)
                    if (l.d[j] == d[e] && perm[l.q[j]] < u) ++rank[e];
            }
    }
    if (!live || !ok) return ok;
    if (gl == 0) nbr[p] = p;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e * G + gl < cnt && rank[e] < need)
            nbr[(int64_t)(rank[e] + 1) * n + p] = l.q[e * G + gl];
    return ok;
}

// Stencils of all nodes, eight lanes a node; k_knn_redo serves those that give up
// (none on lattices). Inserting each candidate into a sorted list in registers
// costs every lane of a wavefront a pass over the list whenever one lane takes it,
// and one lane a node leaves a small cloud's few wavefronts waiting for cells and
// nodes in turn: 909 us against 209 on 262,144 nodes, K 30, and 182 against 20 on
// 10,201, K 25.
constexpr int kKnnLanes = 8;
template <int CAP>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(CAP == 32 ? 7 : CAP == 64 ? 6 : 4))) void k_knn(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ cstart,
    const int32_t *__restrict__ cend, int n, int K, int32_t *__restrict__ redo,
    int32_t *__restrict__ nbr) {
    constexpr int G = kKnnLanes, QB = 256 / G;
    __shared__ double s_d[QB][CAP + 1];   // (odd strides: the groups read distinct banks)
    __shared__ int s_q[QB][CAP + 1];
    __shared__ int s_cnt[QB];
    __shared__ unsigned s_occ[QB][2];
    const int64_t nb = ((int64_t)n + QB - 1) / QB, blk = xcd_tile(nb);
    if (blk >= nb) return;
    const int grp = threadIdx.x / G;
    const int64_t pt = blk * QB + grp;
    const bool live = pt < n;
    const int p = live ? (int)pt : n - 1;
    const KnnList l{s_d[grp], s_q[grp], &s_cnt[grp], s_occ[grp]};
    if (!knn_by_radius<CAP, G>(*geo, xs, ys, perm, cstart, cend, n, K, p, live, l, nbr) &&
        live && threadIdx.x % G == 0)
        redo[1 + atomicAdd(&redo[0], 1)] = p;
}

// The nodes that k_knn left, a wavefront each: redo[0] of them, from redo[1] on.
// The search of 20,000 nodes, ms, with this, with sixteen radii by eight lanes, and
// by rings of cells, one lane a node: eight dense clusters K 12 1.1, 19, 12, K 45
// 1.4, 32, 40; a strip of 0.003 of the domain and 20 nodes outside, K 12 0.8, 98, 36;
// one node far off the others 0.4, 10, 17. An empty list costs a launch of 5 us.
__global__ __launch_bounds__(64) void k_knn_redo(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ cstart,
    const int32_t *__restrict__ cend, int n, int K, const int32_t *__restrict__ redo,
    int32_t *__restrict__ nbr) {
    constexpr int CAP = 96;
    __shared__ double s_d[CAP];
    __shared__ int s_q[CAP];
    __shared__ int s_cnt;
    __shared__ unsigned s_occ[2];
    const int count = min(redo[0], n);
    const KnnList l{s_d, s_q, &s_cnt, s_occ};
    for (int i = blockIdx.x; i < count; i += gridDim.x) {
        knn_by_radius<CAP, 64>(*geo, xs, ys, perm, cstart, cend, n, K, redo[1 + i], true, l, nbr);
        wave_lds_sync();   // the next node takes the list's place
    }
}

// Owner of each departure point x_p - e_k dx (k = 1..8): the closest node,
// ties to the lower user index. One thread a departure point: the cells of a
// ring are loads that wait for one another, so a small cloud needs every
// wavefront it can get (10,201 nodes: 126 us with one thread a node, 18 now;
// 262,144 nodes: 176 and 117). A departure point also takes the next place in its
// owner's list.
__global__ __launch_bounds__(256) void k_owner(const Geo *__restrict__ geo,
                                               const double *__restrict__ xs,
                                               const double *__restrict__ ys,
                                               const int32_t *__restrict__ perm,
                                               const int32_t *__restrict__ cstart,
                                               const int32_t *__restrict__ cend, int n,
                                               double dx, int32_t *__restrict__ owner,
                                               int32_t *__restrict__ cnt,
                                               int32_t *__restrict__ slot) {
    // eight directions of 32 nodes a workgroup, which share their cells
    const int64_t nb = ((int64_t)n + 31) / 32, blk = xcd_tile(nb);
    if (blk >= nb) return;
    const int p = (int)(blk * 32) + (threadIdx.x & 31), k = (threadIdx.x >> 5) + 1;
    if (p >= n) return;
    const Geo g = *geo;
    const double cmin = fmin(g.cw, g.ch);
    const double qx = xs[p] - lat_ex(k) * dx;
    const double qy = ys[p] - lat_ey(k) * dx;
    // cell of the departure point (wrapped into the periodic box)
    double wx = qx, wy = qy;
    if (g.Lx > 0.0) wx = wx - g.Lx * floor(wx / g.Lx);
    if (g.Ly > 0.0) wy = wy - g.Ly * floor(wy / g.Ly);
    int cx, cy;
    cell_of(g, wx, wy, cx, cy);
    double bd = DBL_MAX;
    int bu = INT_MAX, bq = 0;
    auto take = [&](int q) {
        const double d = dist2(qx, qy, xs[q], ys[q], g.Lx, g.Ly);
        if (!(d <= bd)) return;
        const int u = perm[q];
        if (d < bd || u < bu) {
            bd = d;
            bu = u;
            bq = q;
        }
    };
    for (int r = 0;; ++r) {
        bool wraps = (g.Lx > 0.0 && 2 * r + 1 > g.gx) || (g.Ly > 0.0 && 2 * r + 1 > g.gy);
        if (wraps) {
            bd = DBL_MAX;
            bu = INT_MAX;
            for (int q = 0; q < n; ++q) take(q);
            break;
        }
        for_ring(g, cstart, cend, cx, cy, r, take);
        double reach = r * cmin;
        if (bd < reach * reach) break;
        if (r > g.gx && r > g.gy) break;
    }
    owner[(int64_t)(k - 1) * n + p] = bq;
    slot[(int64_t)(k - 1) * n + p] = atomicAdd(&cnt[bq], 1);
}

// x^e for 0 <= e <= 4, without branches on e, so that a lane-dependent
// exponent costs no divergent code.
__device__ __forceinline__ double pow_upto4(double x, int e) {
    double p = 1.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) p = t < e ? p * x : p;
    return p;
}

__device__ __forceinline__ double cube_dist(double ax, double ay, double bx, double by) {
    double dx = ax - bx, dy = ay - by;
    double r = sqrt(dx * dx + dy * dy);
    return r * r * r;
}

// Departure point t of the right-hand-side list of owner s: node p and
// direction k. Own-node stencils: the eight departure points of s itself.
// Paper stencils: the points whose closest node is s (CSR list pts).
struct RhsList {
    const int32_t *ptr, *pts;   // null for own-node stencils
};

__device__ __forceinline__ void rhs_point(const RhsList &L, int s, int t, int &p, int &k) {
    if (!L.ptr) {
        p = s;
        k = t + 1;
    } else {
        const int e = L.pts[L.ptr[s] + t];
        p = e >> 3;
        k = (e & 7) + 1;
    }
}

// Largest 32-bit key over the lanes of a wavefront (all active), the same in
// every lane: DPP exchanges inside each row of 16 lanes (swap neighbours, swap
// pairs, mirror the half-rows, mirror the row) leave the row's largest key in
// all its lanes; the rows are then combined from scalar reads.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
    const uint32_t r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const uint32_t r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return max(max(r0, r1), max(r2, r3));
}

// The double in lane l of a wavefront (l uniform), in scalar registers.
__device__ __forceinline__ double readlane_d(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// 1/x to within about an ulp: the hardware estimate (about 2^-23 relative
// error for the magnitudes met here) refined by two Newton steps r += r(1 - xr),
// each of which squares the relative error. Zero gives NaN, which the
// singularity test catches where it matters (a zero pivot).
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return r;
}

// One wavefront solves the local system of an owner node, Phi w = phi(p)
// (eqs. rbf_interp_set_augmented and shape_vector) of owner s for every
// departure point that uses the stencil of s, by Gauss-Jordan elimination with
// partial pivoting. Lane r holds row r of the system (K RBF rows, M polynomial
// rows, then identity rows that pad the system to NB unknowns) in registers.
// Rows are never moved: the pivot of column k is a not-yet-used lane with the
// largest |a_k|, compared on the upper 32 bits of its binary64 encoding
// (exponent and 20 mantissa bits, so within a factor 1 + 2^-20 of the largest,
// which keeps the growth bound of partial pivoting; ties: lowest lane). Its row
// and its reciprocal 1/a_k are broadcast, and every other lane, pivot rows of
// earlier steps included, subtracts its multiple of that row and keeps the
// multiplier in a_k. At the end the pivot row of step j holds a_j x_j = b, so
// unknown j (the weight of stencil member j, j < K) is one product with the
// kept reciprocal away, with no back substitution. The right-hand sides
// (departure points) are taken R at a time: the first group is eliminated
// along with the matrix, later groups by replaying the stored multipliers.
template <int NB, int R, bool REPLAY>
__device__ __forceinline__ void rbf_solve(const Geo *__restrict__ geo,
                                          const double *__restrict__ xs,
                                          const double *__restrict__ ys,
                                          const int32_t *__restrict__ perm,
                                          const int32_t *__restrict__ nbr, RhsList L, int n,
                                          int K, int m, double dx, double *__restrict__ W64,
                                          int32_t *__restrict__ dev_err) {
    constexpr int MP = 15;   // monomials of degree <= 4 (table row stride, odd)
    __shared__ double2 s_c[4][64];
    __shared__ double s_P[4][kMaxK * MP];
    __shared__ double2 s_q[4][R];
    __shared__ int2 s_pk[4][R];
    const int lane = threadIdx.x & 63, ll = lane;   // lane: row of the system
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // each XCD takes a contiguous range of owners: the shape vectors they
    // store land at neighbouring nodes, so the L2 of one XCD collects whole
    // lines of them (grid xcd_grid of the workgroup count)
    const int64_t blk = xcd_tile(((int64_t)n + 3) / 4);
    const int64_t so = blk * 4 + wv;
    if (so >= n) return;   // uniform across the wavefront
    const int s = (int)so;
    // (without REPLAY every owner has at most R departure points)
    const int count = __builtin_amdgcn_readfirstlane(L.ptr ? L.ptr[s + 1] - L.ptr[s] : 8);
    if (count == 0) return;
    const Geo g = *geo;
    const int M = (m + 1) * (m + 2) / 2;
    const int nn = K + M;
    double *P = s_P[wv];
    const double2 *cw = s_c[wv];
    double2 *qw = s_q[wv];
    int2 *pkw = s_pk[wv];

    // stencil member coordinates relative to the centre s, scaled by the
    // stencil radius (the interpolant is invariant to this; it helps the
    // conditioning)
    double rx = 0.0, ry = 0.0;
    if (ll < K) {
        int q = nbr[(int64_t)ll * n + s];
        rx = min_image(xs[q] - xs[s], g.Lx);
        ry = min_image(ys[q] - ys[s], g.Ly);
    }
    double rad = sqrt(rx * rx + ry * ry);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rad = fmax(rad, __shfl_xor(rad, off));
    if (!(rad > 0.0)) rad = 1.0;
    const double sx = rx / rad, sy = ry / rad;
    s_c[wv][lane] = make_double2(sx, sy);
    // monomials of each member (eq. poly_sets, graded order 1, x, y, x^2, xy,
    // y^2, x^3, ..., y^4: monomial q of degree d at offset j is x^(d-j) y^j),
    // row `ll` of the table
    if (ll < K) {
        double xp[5], yp[5];
        xp[0] = yp[0] = 1.0;
#pragma unroll
        for (int e = 1; e < 5; ++e) {
            xp[e] = xp[e - 1] * sx;
            yp[e] = yp[e - 1] * sy;
        }
        int q = 0;
#pragma unroll
        for (int d = 0; d <= 4; ++d)
#pragma unroll
            for (int j = 0; j <= d; ++j) P[ll * MP + q++] = xp[d - j] * yp[j];
    }
    wave_lds_sync();
    const bool rbf_row = ll < K;
    const bool poly_row = ll >= K && ll < nn;
    const int qrow = ll - K;
    // table entries this lane reads: polynomial q of every member (polynomial
    // rows), every polynomial of its own member (RBF rows)
    const int pcol = poly_row ? qrow : 0;
    const int prow = (rbf_row ? ll : 0) * MP - K;

    // row `ll` of the padded system; the branches on the column are uniform
    double a[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        if (c < K) {
            const double2 cc = cw[c];
            const double r3 = cube_dist(sx, sy, cc.x, cc.y);
            const double pc = P[c * MP + pcol];
            a[c] = rbf_row ? r3 : (poly_row ? pc : 0.0);
        } else if (c < nn) {
            const double pr = P[prow + c];
            a[c] = rbf_row ? pr : 0.0;
        } else {
            a[c] = c == ll ? 1.0 : 0.0;
        }
    }
    // infinity norm for the singularity threshold
    double rs = 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c) rs += fabs(a[c]);
    if (ll >= NB) rs = 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rs = fmax(rs, __shfl_xor(rs, off));
    const double tiny = 1e3 * DBL_EPSILON * rs;
    bool singular = false;
    // elimination step at which this lane was the pivot (-1: padding lane)
    // and the reciprocal of its pivot value
    int pstep = ll < NB ? NB : -1;
    double pinv = 1.0;

    // right-hand sides c0 .. c0+R-1 (row `ll` of each). Lane t < R of each
    // group first locates departure point c0 + t (node p, direction k) and its
    // position x_p - e_k dx relative to s, scaled, for the whole group.
    const double irad = 1.0 / rad;
    // exponents of monomial qrow (degree qd, offset qey within it)
    const int qd = (qrow >= 1) + (qrow >= 3) + (qrow >= 6) + (qrow >= 10);
    const int qey = poly_row ? qrow - qd * (qd + 1) / 2 : 0;
    const int qex = poly_row ? qd - qey : 0;
    auto load_rhs = [&](int c0, double(&b)[R]) {
        if (ll < R) {
            double qx = 0.0, qy = 0.0;
            int p = 0, k = 1;
            if (c0 + ll < count) {
                rhs_point(L, s, c0 + ll, p, k);
                qx = (L.ptr ? min_image(xs[p] - lat_ex(k) * dx - xs[s], g.Lx)
                            : -lat_ex(k) * dx) * irad;
                qy = (L.ptr ? min_image(ys[p] - lat_ey(k) * dx - ys[s], g.Ly)
                            : -lat_ey(k) * dx) * irad;
            }
            qw[ll] = make_double2(qx, qy);
            pkw[ll] = make_int2(p, k);
        }
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < R; ++t) {
            const double2 q = qw[t];
            const double r3 = cube_dist(sx, sy, q.x, q.y);
            const double pq = pow_upto4(q.x, qex) * pow_upto4(q.y, qey);
            b[t] = c0 + t < count ? (rbf_row ? r3 : (poly_row ? pq : 0.0)) : 0.0;
        }
    };
    // the pivot row of step j < K holds a_j x_j = b: x_j is the weight of
    // stencil member j for each departure point
    auto store = [&](int c0, const double(&b)[R]) {
        if (pstep >= 0 && pstep < K) {
#pragma unroll
            for (int t = 0; t < R; ++t) {
                if (c0 + t < count) {
                    const int2 pk = pkw[t];
                    W64[w64_at(pk.y, pstep, n, pk.x)] = b[t] * pinv;
                }
            }
        }
    };

    double b[R];
    load_rhs(0, b);
    // The pivot row is broadcast through scalar
    // registers (two lane reads per value, used directly as the scalar
    // operand of the updates) instead of LDS, which the four SIMDs of a
    // compute unit share and which every lane would otherwise read the
    // whole row from. Lane k keeps the pivot lane of step k for the
    // replay of further groups.
    // Steps from nn on pivot on the identity rows that pad the system
    // and change nothing, and columns from nn on stay zero in every row
    // that holds a pivot before (a zero pivot there only happens in a
    // singular system, which is reported): both are skipped with uniform
    // branches.
    int plog = 0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        if (k >= nn) continue;
        const uint32_t key =
            pstep > k ? ((uint32_t)(__double_as_longlong(a[k]) >> 32) & 0x7FFFFFFFu) | 1u : 0u;
        const double rk = recip(a[k]);
        const uint32_t km = wave_max_u32(key);
        const int pl = __builtin_amdgcn_readfirstlane(__builtin_ctzll(__ballot(key == km)));
        const double pv = readlane_d(a[k], pl), pi = readlane_d(rk, pl);
        if (!(fabs(pv) > tiny)) singular = true;
        if (lane == pl) {
            pstep = k;
            pinv = pi;
        }
        if (lane == k) plog = pl;
        const double l = lane != pl ? a[k] * pi : 0.0;
        // (four lane reads ahead of their updates, so that the scalar
        // results are not waited for one by one)
#pragma unroll
        for (int c = k + 1; c < NB; c += 4) {
            if (c >= nn) continue;
            const double r0 = readlane_d(a[c], pl);
            const double r1 = c + 1 < NB ? readlane_d(a[c + 1], pl) : 0.0;
            const double r2 = c + 2 < NB ? readlane_d(a[c + 2], pl) : 0.0;
            const double r3 = c + 3 < NB ? readlane_d(a[c + 3], pl) : 0.0;
            a[c] = __builtin_fma(-l, r0, a[c]);
            if (c + 1 < NB) a[c + 1] = __builtin_fma(-l, r1, a[c + 1]);
            if (c + 2 < NB) a[c + 2] = __builtin_fma(-l, r2, a[c + 2]);
            if (c + 3 < NB) a[c + 3] = __builtin_fma(-l, r3, a[c + 3]);
        }
#pragma unroll
        for (int t = 0; t < R; t += 2) {
            const double r0 = readlane_d(b[t], pl), r1 = readlane_d(b[t + 1], pl);
            b[t] = __builtin_fma(-l, r0, b[t]);
            b[t + 1] = __builtin_fma(-l, r1, b[t + 1]);
        }
        if (lane != pl) a[k] = l;
    }
    store(0, b);
    for (int c0 = R; REPLAY && c0 < count; c0 += R) {
        load_rhs(c0, b);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            if (k >= nn) continue;
            const int pk = __builtin_amdgcn_readlane(plog, k);
            const double l = lane != pk ? a[k] : 0.0;
#pragma unroll
            for (int t = 0; t < R; ++t) b[t] = __builtin_fma(-l, readlane_d(b[t], pk), b[t]);
        }
        store(c0, b);
    }
    if (singular && ll == 0) atomicMin(dev_err, perm[s] + 1);
}

// Two wavefronts per SIMD with the replay, three without it, which keeps fewer
// registers alive (a small spill costs less than the latency that fewer
// wavefronts leave exposed).
template <int NB, int R, int WPE, bool REPLAY>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WPE))) void k_rbf(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ nbr, RhsList L, int n, int K,
    int m, double dx, double *__restrict__ W64, int32_t *__restrict__ dev_err) {
    rbf_solve<NB, R, REPLAY>(geo, xs, ys, perm, nbr, L, n, K, m, dx, W64, dev_err);
}

// ---- the same solve with the FP64 matrix cores ------------------------------
// The systems and the elimination of rbf_solve (Gauss-Jordan, partial
// pivoting on the upper 32 bits of |a_k|, ties to the lowest row, rows never
// moved, pivot rows left unscaled), taken four pivot columns at a time so that
// the bulk of the arithmetic runs on v_mfma_f64_16x16x4:
//  - the augmented matrix [Phi | b_0 .. b_15] (NB = 16 RT unknowns, up to 16
//    departure points) lives in the registers of one wavefront as RT x (RT+1)
//    tiles of 16 x 16 in the result layout of that instruction (register i of
//    lane l holds row l / 16 + 4 i, column l % 16 of its tile);
//  - a panel of four columns is copied to LDS and eliminated with one row per
//    lane, pivot search and row reads as in rbf_solve but on four columns. Its
//    four steps E_j = I - l_j e_{p_j}^T (l_j the multipliers, zero at the pivot
//    row p_j) multiply to I - Lt S^T, S^T selecting the pivot rows; the new
//    column of Lt is the step's multipliers and the earlier ones are reduced
//    by the step like matrix columns;
//  - every column right of the panel, right-hand sides included, then takes
//    the rank-4 product -Lt U, U the four pivot rows as they stood before the
//    panel: RT x (tiles right of the panel) matrix-core products, with Lt in
//    the A layout (lane 16 k + r holds row r, column k) and U in the B layout
//    (lane 16 k + c holds row k, column c).
// The pivot row of step j ends as d_j e_j on the matrix part, so unknown j is
// its right-hand-side entry times 1/d_j. Owners with more than 16 departure
// points solve again for each further group of 16. Each lane assembles its own
// tile entries (monomials from a per-member table in LDS).
// It serves 33 to 48 unknowns beyond the sizes of k_rbf_null, and what that
// one leaves. The FP64 matrix-core rate of gfx950 equals its FP64 vector rate: what the
// products save is issue slots (108 products a system at 48 unknowns against
// about 2,700 vector FMAs). The pivot steps (reduction, lane reads) stay
// serial and dominate what remains.
typedef double dbl4 __attribute__((ext_vector_type(4)));

// v from the lane CTRL names (a DPP row pattern), both halves of a double
template <int CTRL> __device__ __forceinline__ double dpp_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Three wavefronts per SIMD at 48 unknowns (167 VGPRs, a 20-byte spill);
// without the hint the compiler keeps the tiles in 460 registers and runs one.
template <int RT>
__device__ __forceinline__ void rbf_mfma_solve(const int s, const Geo &g,
                                               const double *__restrict__ xs,
                                               const double *__restrict__ ys,
                                               const int32_t *__restrict__ perm,
                                               const int32_t *__restrict__ nbr, RhsList L, int n,
                                               int K, int m, double dx, double *__restrict__ W64,
                                               int32_t *__restrict__ dev_err) {
    constexpr int NB = 16 * RT, CT = RT + 1, NC = 16 * CT;
    __shared__ double2 s_c[64];          // scaled stencil members
    __shared__ double2 s_q[16];          // scaled departure points of the group
    __shared__ int2 s_pk[16];            // their (node, direction)
    __shared__ double s_pan[4][NB + 4];  // panel columns (rows padded: see below)
    __shared__ double s_L[4][NB];        // Lt, column-major
    // the row groups that hold the pivot rows; element e of column c sits at
    // e ^ ((c >> 2) & 3), so that the sixteen lanes of a row group, which
    // read one element of sixteen consecutive columns, hit distinct banks
    // (unswizzled they read 32 bytes apart, four to a bank); the panel rows
    // are padded for the same reason. Both measured 4.7 % off the solve.
    __shared__ double s_U[4][NC][4];
    __shared__ int s_step[NB];
    __shared__ double s_pinv[NB];
    constexpr int PQ = NB * 15;          // the departure points' monomials follow the members'
    static_assert(PQ + 16 * 15 <= 4 * NC * 4, "the monomial tables fit in s_U");
    const int lane = threadIdx.x;
    const int count = L.ptr ? L.ptr[s + 1] - L.ptr[s] : 8;
    if (count == 0) return;
    const int M = (m + 1) * (m + 2) / 2;
    const int nn = K + M;

    double rx = 0.0, ry = 0.0;
    if (lane < K) {
        const int q = nbr[(int64_t)lane * n + s];
        rx = min_image(xs[q] - xs[s], g.Lx);
        ry = min_image(ys[q] - ys[s], g.Ly);
    }
    double rad = sqrt(rx * rx + ry * ry);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rad = fmax(rad, __shfl_xor(rad, off));
    if (!(rad > 0.0)) rad = 1.0;
    const double sx = rx / rad, sy = ry / rad, irad = 1.0 / rad;
    s_c[lane] = make_double2(sx, sy);
    bool singular = false;

    for (int c0 = 0; c0 < count; c0 += 16) {
        const int cnt = min(16, count - c0);
        if (lane < 16) {
            double qx = 0.0, qy = 0.0;
            int p = 0, k = 1;
            if (lane < cnt) {
                rhs_point(L, s, c0 + lane, p, k);
                qx = (L.ptr ? min_image(xs[p] - lat_ex(k) * dx - xs[s], g.Lx) : -lat_ex(k) * dx) *
                     irad;
                qy = (L.ptr ? min_image(ys[p] - lat_ey(k) * dx - ys[s], g.Ly) : -lat_ey(k) * dx) *
                     irad;
            }
            s_q[lane] = make_double2(qx, qy);
            s_pk[lane] = make_int2(p, k);
        }
        wave_lds_sync();

        // monomials of the stencil members (lanes below K) and of the group's
        // departure points (lanes 48 + t), row stride 15, in the space that
        // the elimination uses for U; powers first, then each product
        double *tab = &s_U[0][0][0];
        // the lane index again, opaque to the compiler: what depends on it is
        // recomputed for each group rather than kept live from the first
        int lid = lane;
        __asm__ volatile("" : "+v"(lid));
        const int g4 = lid >> 4, cl = lid & 15;
        {
            const int t = lid - 48;
            const bool mem = lid < K, dep = t >= 0 && t < cnt;
            double px = sx, py = sy;
            if (dep) {
                const double2 q = s_q[t];
                px = q.x;
                py = q.y;
            }
            double xp[5], yp[5];
            xp[0] = yp[0] = 1.0;
#pragma unroll
            for (int e = 1; e < 5; ++e) {
                xp[e] = xp[e - 1] * px;
                yp[e] = yp[e - 1] * py;
            }
            double *row = tab + (mem ? lid * 15 : PQ + (dep ? t : 0) * 15);
            if (mem || dep) {
#pragma unroll
                for (int d = 0, q = 0; d <= 4; ++d)
#pragma unroll
                    for (int ey = 0; ey <= d; ++ey, ++q)
                        if (q < M) row[q] = xp[d - ey] * yp[ey];
            }
        }
        wave_lds_sync();

        // assembly: every lane computes its own entries of the tiles; the
        // branches on a tile's place against K are uniform
        dbl4 T[RT][CT];
        double rsum[RT][4];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * rt + g4 + 4 * i;
                const double2 xr = s_c[r];
                const bool rr = r < K, pr = r >= K && r < nn;
                double acc = 0.0;
#pragma unroll
                for (int ct = 0; ct < RT; ++ct) {
                    const int c = 16 * ct + cl;
                    const bool rc = c < K, pc = c >= K && c < nn;
                    double r3 = 0.0;
                    if (16 * rt < K && 16 * ct < K) {
                        const double2 xc = s_c[c];
                        r3 = cube_dist(xr.x, xr.y, xc.x, xc.y);
                    }
                    const int ti = rr && pc ? r * 15 + (c - K) : pr && rc ? c * 15 + (r - K) : 0;
                    const double tv = tab[ti];
                    const double a = rr ? (rc ? r3 : (pc ? tv : 0.0))
                                        : pr ? (rc ? tv : 0.0) : (r == c ? 1.0 : 0.0);
                    T[rt][ct][i] = a;
                    acc += fabs(a);
                }
                rsum[rt][i] = acc;
                {
                    const int t = cl;
                    double r3 = 0.0;
                    if (16 * rt < K) {
                        const double2 q = s_q[t];
                        r3 = cube_dist(xr.x, xr.y, q.x, q.y);
                    }
                    const double tv = tab[pr ? PQ + t * 15 + (r - K) : 0];
                    T[rt][RT][i] = t < cnt ? (rr ? r3 : (pr ? tv : 0.0)) : 0.0;
                }
                // one row at a time: keeps the compiler from hoisting every
                // row's table reads (and their registers) to the start
                __asm__ volatile("" ::: "memory");
            }
        // infinity norm of the matrix: row sums over the sixteen lanes that
        // share a row group, then the largest row
        double rs = 0.0;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double v = rsum[rt][i];
                v += dpp_d<0x128>(v);
                v += dpp_d<0x124>(v);
                v += dpp_d<0x122>(v);
                v += dpp_d<0x121>(v);
                rs = fmax(rs, v);
            }
        rs = fmax(fmax(readlane_d(rs, 0), readlane_d(rs, 16)),
                  fmax(readlane_d(rs, 32), readlane_d(rs, 48)));
        const double tiny = 1e3 * DBL_EPSILON * rs;
        wave_lds_sync();   // the table's space is U's from here on

        int pstep = lane < NB ? NB : -1;
        double pinv = 1.0;
        // panels: the column tile of the panel is unrolled (register tiles
        // take compile-time indices), the four panels inside it are not; the
        // products cover the panel's own tile too (for its last panel only
        // finished columns change there)
#pragma unroll
        for (int ctp = 0; ctp < RT; ++ctp) {
#pragma unroll 1
            for (int cp0 = 0; cp0 < 16; cp0 += 4) {
                const int k0 = 16 * ctp + cp0;
                if (k0 >= nn) break;                  // uniform
                if (cl >= cp0 && cl < cp0 + 4) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            s_pan[cl - cp0][16 * rt + g4 + 4 * i] = T[rt][ctp][i];
                }
                wave_lds_sync();
                double pv[4] = {0.0, 0.0, 0.0, 0.0}, Lt[4] = {0.0, 0.0, 0.0, 0.0};
                if (lane < NB) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) pv[j] = s_pan[j][lane];
                }
                int plist[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = k0 + j;
                    plist[j] = -1;
                    if (k >= nn) continue;            // uniform
                    const uint32_t key =
                        pstep > k
                            ? ((uint32_t)(__double_as_longlong(pv[j]) >> 32) & 0x7FFFFFFFu) | 1u
                            : 0u;
                    const double rk = recip(pv[j]);
                    const uint32_t km = wave_max_u32(key);
                    const int pl =
                        __builtin_amdgcn_readfirstlane(__builtin_ctzll(__ballot(key == km)));
                    const double pvv = readlane_d(pv[j], pl), pi = readlane_d(rk, pl);
                    if (!(fabs(pvv) > tiny)) singular = true;
                    if (lane == pl) {
                        pstep = k;
                        pinv = pi;
                    }
                    const double l = lane != pl ? pv[j] * pi : 0.0;
#pragma unroll
                    for (int jj = j + 1; jj < 4; ++jj)
                        pv[jj] = __builtin_fma(-l, readlane_d(pv[jj], pl), pv[jj]);
#pragma unroll
                    for (int jj = 0; jj < j; ++jj)
                        Lt[jj] = __builtin_fma(-l, readlane_d(Lt[jj], pl), Lt[jj]);
                    Lt[j] = l;
                    plist[j] = pl;
                }
                if (lane < NB) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) s_L[j][lane] = Lt[j];
                }
                // U: the row group of each pivot row writes its four rows of
                // every tile from the panel's on; a step past nn gives a zero row
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int p = plist[j];
                    if (p < 0) {
                        if (g4 == 0) {
#pragma unroll
                            for (int ct = ctp; ct < CT; ++ct)
                                *reinterpret_cast<dbl4 *>(&s_U[j][16 * ct + cl][0]) =
                                    dbl4{0.0, 0.0, 0.0, 0.0};
                        }
                        continue;
                    }
                    const int rtp = p >> 4, gp = p & 3;
                    // one branch per row tile (uniform); the empty asm keeps
                    // the compiler from merging the stores into one store of
                    // a value selected across every tile
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        if (rt == rtp) {
                            __asm__ volatile("" ::: "memory");
                            if (g4 == gp) {
#pragma unroll
                                for (int ct = ctp; ct < CT; ++ct)
#pragma unroll
                                    for (int e = 0; e < 4; ++e)
                                        s_U[j][16 * ct + cl][e ^ ((cl >> 2) & 3)] = T[rt][ct][e];
                            }
                        }
                    }
                }
                wave_lds_sync();
                const int pk =
                    g4 == 0 ? plist[0] : g4 == 1 ? plist[1] : g4 == 2 ? plist[2] : plist[3];
                const int ik = pk < 0 ? 0 : ((pk & 15) >> 2);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const double a = -s_L[g4][16 * rt + cl];
#pragma unroll
                    for (int ct = ctp; ct < CT; ++ct) {
                        const double b = s_U[g4][16 * ct + cl][ik ^ ((cl >> 2) & 3)];
                        T[rt][ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, T[rt][ct], 0, 0, 0);
                    }
                }
                wave_lds_sync();
            }
        }
        if (lane < NB) {
            s_step[lane] = pstep;
            s_pinv[lane] = pinv;
        }
        wave_lds_sync();
        if (cl < cnt) {
            const int2 pk = s_pk[cl];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 16 * rt + g4 + 4 * i;
                    const int j = s_step[r];
                    if (j < K) W64[w64_at(pk.y, j, n, pk.x)] = T[rt][RT][i] * s_pinv[r];
                }
        }
        wave_lds_sync();
    }
    if (singular && lane == 0) atomicMin(dev_err, perm[s] + 1);
}

template <int RT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_rbf_mfma(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ nbr, RhsList L, int n, int K,
    int m, double dx, double *__restrict__ W64, int32_t *__restrict__ dev_err) {
    // owners in XCD-contiguous ranges, as in k_rbf (grid xcd_grid(n))
    const int64_t s = xcd_tile(n);
    if (s >= n) return;
    rbf_mfma_solve<RT>((int)s, *geo, xs, ys, perm, nbr, L, n, K, m, dx, W64, dev_err);
}

// The same for the owners that k_rbf_null left: redo[0] of them, from redo[1]
// on, in whatever order. Usually none, so the grid is small and walks the list.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_rbf_redo(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ perm, const int32_t *__restrict__ nbr, RhsList L, int n, int K,
    int m, double dx, const int32_t *__restrict__ redo, double *__restrict__ W64,
    int32_t *__restrict__ dev_err) {
    const int count = min(redo[0], n);
    for (int i = blockIdx.x; i < count; i += gridDim.x)
        rbf_mfma_solve<3>(redo[1 + i], *geo, xs, ys, perm, nbr, L, n, K, m, dx, W64, dev_err);
}

// ---- the same systems by the null space of the polynomials --------------------
// Phi = [[R, P], [P^T, 0]] with r^3 positive definite on the null space of P^T
// (r^3 is conditionally positive definite of order 2 and the polynomials hold
// the linear ones), so only the M columns of P need a pivot search:
//  1. P = L U with row pivoting (M steps over the K members); the M pivot
//     members are "set 1", the other N2 = K - M "set 2", X = P2 P1^-1;
//  2. S = R22 - X R12 - (R21 - X R11) X^T, symmetric positive definite, is
//     factored without a search;
//  3. per departure point y = p P1^-1 (two triangular solves with L and U),
//     S w2 = phi2 - X phi1 - (R21 - X R11) y^T and w1 = y - w2 X.
// At K 30, degree 4 that is 15 pivot searches and about 24k multiply-adds a
// system with its eight points, against 45 and 62k for the elimination of Phi.
//
// Sixteen lanes take a system, four systems a wavefront. After step 1 the
// members are dealt out again, set 1 in pivot order, so that everything that
// follows names its lanes at compile time: the matrices are held a row per
// lane, and every multiply-add takes its second factor from a fixed lane of
// the sixteen as it goes (v_fmac_f64 with DPP row_newbcast, the one DPP
// pattern that double precision has), without LDS and without a broadcast of
// its own. Departure points are a lane each, sixteen at a time.
// The pivot rows of step 1, which only become known there, go through LDS,
// straight to their place in pivot order.
//
// Bound by issue: about 7,000 instructions a wavefront, a third of them FP64
// multiply-adds, two wavefronts a SIMD. 262,144 nodes, K 30, degree 4, paper
// rule: 4.46 -> 0.92 ms for the solves against the elimination of Phi on the
// matrix cores. The shape vectors' error against a solve with refinement falls
// too, on the lattices of the studies from 4.3e-16 - 1.7e-15 to 2.9e-16 -
// 5.0e-16 of an interpolated field. Blocks of eight multiply-adds instead of
// four (fewer wait states) measured the same.
//
// A system that may be singular by the rule of the general elimination (a pivot
// of at most 1e3 eps |Phi|) is left to k_rbf_redo, which decides by that rule:
// `redo` gets its owner. Nodes nearly on one curve of the polynomials' degree
// leave a small pivot u in P; the elimination of Phi then meets a pivot near u^2
// (its inverse holds R / u^2), so the line for u lies at 1e-4, where u^2 is a
// hundred times the largest threshold. Nodes close together leave a small pivot
// in S, which is of the size of Phi's: its line is 1e6 eps (8 K + M), at least
// 1e3 times the threshold (distances are at most 2 stencil radii). Over 40,000
// systems of pairs, clusters, strips and curves of all sizes, 12,641 of them
// refused, the refused ones had u below 5e-7 or a pivot of S below 2e-4 of its
// line. Jittered lattices have u above 2e-2 from K = M + 3 on and above 2e-4 at
// K = M.
constexpr double kSetPivot = 1e-4;

// acc[i] += (NEG ? -1 : 1) src(lane L0 + i) m for i < C <= 4, the lane taken within each
// group of sixteen. The wait states that a DPP read of a fresh result needs
// come first, inside the block.
#define MLBM_BC " row_mask:0xf bank_mask:0xf"
template <int L0, int C, bool NEG>
__device__ __forceinline__ void fmac_lanes(double *acc, double src, double m) {
    if constexpr (C == 4) {
        if constexpr (NEG)
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, -%4, %5 row_newbcast:%6" MLBM_BC
                "\n\tv_fmac_f64_dpp %1, -%4, %5 row_newbcast:%7" MLBM_BC
                "\n\tv_fmac_f64_dpp %2, -%4, %5 row_newbcast:%8" MLBM_BC
                "\n\tv_fmac_f64_dpp %3, -%4, %5 row_newbcast:%9" MLBM_BC
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
                : "v"(src), "v"(m), "i"(L0), "i"(L0 + 1), "i"(L0 + 2), "i"(L0 + 3));
        else
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, %4, %5 row_newbcast:%6" MLBM_BC
                "\n\tv_fmac_f64_dpp %1, %4, %5 row_newbcast:%7" MLBM_BC
                "\n\tv_fmac_f64_dpp %2, %4, %5 row_newbcast:%8" MLBM_BC
                "\n\tv_fmac_f64_dpp %3, %4, %5 row_newbcast:%9" MLBM_BC
                : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
                : "v"(src), "v"(m), "i"(L0), "i"(L0 + 1), "i"(L0 + 2), "i"(L0 + 3));
    } else if constexpr (C > 0) {
        if constexpr (NEG)
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, -%1, %2 row_newbcast:%3" MLBM_BC
                : "+&v"(acc[0]) : "v"(src), "v"(m), "i"(L0));
        else
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3" MLBM_BC
                : "+&v"(acc[0]) : "v"(src), "v"(m), "i"(L0));
        fmac_lanes<L0 + 1, C - 1, NEG>(acc + 1, src, m);
    }
}

// acc[i] += (NEG ? -1 : 1) src[i / 16](lane i % 16) m for I0 <= i < I1.
template <int I0, int I1, bool NEG>
__device__ __forceinline__ void fmac_rows(double *acc, const double *src, double m) {
    if constexpr (I0 < I1) {
        constexpr int end = I1 < (I0 / 16 + 1) * 16 ? I1 : (I0 / 16 + 1) * 16;
        constexpr int C = end - I0 < 4 ? end - I0 : 4;
        fmac_lanes<I0 % 16, C, NEG>(acc + I0, src[I0 / 16], m);
        fmac_rows<I0 + C, I1, NEG>(acc, src, m);
    }
}

// acc += (NEG ? -1 : 1) sum over I0 <= i < I1 of src[i / 16](lane i % 16) m[i].
template <int I0, int I1, bool NEG>
__device__ __forceinline__ void fmac_dot(double &acc, const double *src, const double *m) {
    if constexpr (I0 < I1) {
        constexpr int end = I1 < (I0 / 16 + 1) * 16 ? I1 : (I0 / 16 + 1) * 16;
        constexpr int C = end - I0 < 4 ? 1 : 4;
        constexpr int L0 = I0 % 16;
        if constexpr (C == 4 && NEG)
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, -%1, %2 row_newbcast:%6" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, -%1, %3 row_newbcast:%7" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, -%1, %4 row_newbcast:%8" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, -%1, %5 row_newbcast:%9" MLBM_BC
                : "+&v"(acc)
                : "v"(src[I0 / 16]), "v"(m[I0]), "v"(m[I0 + 1]), "v"(m[I0 + 2]), "v"(m[I0 + 3]),
                  "i"(L0), "i"(L0 + 1), "i"(L0 + 2), "i"(L0 + 3));
        else if constexpr (C == 4)
            asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%6" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, %1, %3 row_newbcast:%7" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, %1, %4 row_newbcast:%8" MLBM_BC
                "\n\tv_fmac_f64_dpp %0, %1, %5 row_newbcast:%9" MLBM_BC
                : "+&v"(acc)
                : "v"(src[I0 / 16]), "v"(m[I0]), "v"(m[I0 + 1]), "v"(m[I0 + 2]), "v"(m[I0 + 3]),
                  "i"(L0), "i"(L0 + 1), "i"(L0 + 2), "i"(L0 + 3));
        else
            fmac_lanes<L0, 1, NEG>(&acc, src[I0 / 16], m[I0]);
        fmac_dot<I0 + C, I1, NEG>(acc, src, m);
    }
}

// acc[c] += src[c](lane L) m for C0 <= c < C1.
template <int L, int C0, int C1>
__device__ __forceinline__ void fmac_lane(double *acc, const double *src, double m) {
    if constexpr (C1 - C0 >= 4) {
        asm("s_nop 1\n\tv_fmac_f64_dpp %0, %4, %8 row_newbcast:%9" MLBM_BC
            "\n\tv_fmac_f64_dpp %1, %5, %8 row_newbcast:%9" MLBM_BC
            "\n\tv_fmac_f64_dpp %2, %6, %8 row_newbcast:%9" MLBM_BC
            "\n\tv_fmac_f64_dpp %3, %7, %8 row_newbcast:%9" MLBM_BC
            : "+&v"(acc[C0]), "+&v"(acc[C0 + 1]), "+&v"(acc[C0 + 2]), "+&v"(acc[C0 + 3])
            : "v"(src[C0]), "v"(src[C0 + 1]), "v"(src[C0 + 2]), "v"(src[C0 + 3]), "v"(m), "i"(L));
        fmac_lane<L, C0 + 4, C1>(acc, src, m);
    } else if constexpr (C0 < C1) {
        asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3" MLBM_BC
            : "+&v"(acc[C0]) : "v"(src[C0]), "v"(m), "i"(L));
        fmac_lane<L, C0 + 1, C1>(acc, src, m);
    }
}

// The same on rows of their own: acc[c] += acc[c](lane L) m.
template <int L, int C0, int C1>
__device__ __forceinline__ void fmac_self(double *acc, double m) {
    if constexpr (C1 - C0 >= 4) {
        asm("s_nop 1\n\tv_fmac_f64_dpp %0, %0, %4 row_newbcast:%5" MLBM_BC
            "\n\tv_fmac_f64_dpp %1, %1, %4 row_newbcast:%5" MLBM_BC
            "\n\tv_fmac_f64_dpp %2, %2, %4 row_newbcast:%5" MLBM_BC
            "\n\tv_fmac_f64_dpp %3, %3, %4 row_newbcast:%5" MLBM_BC
            : "+&v"(acc[C0]), "+&v"(acc[C0 + 1]), "+&v"(acc[C0 + 2]), "+&v"(acc[C0 + 3])
            : "v"(m), "i"(L));
        fmac_self<L, C0 + 4, C1>(acc, m);
    } else if constexpr (C0 < C1) {
        asm("s_nop 1\n\tv_fmac_f64_dpp %0, %0, %1 row_newbcast:%2" MLBM_BC
            : "+&v"(acc[C0]) : "v"(m), "i"(L));
        fmac_self<L, C0 + 1, C1>(acc, m);
    }
}

// v of lane L of each group of sixteen.
template <int L> __device__ __forceinline__ double lane_of(double v) {
    double r;
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2" MLBM_BC : "=v"(r) : "v"(v), "i"(L));
    return r;
}
template <int L> __device__ __forceinline__ int lane_of(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + L, 0xF, 0xF, true);
}
#undef MLBM_BC

// r^3 for the offset (dx, dy): the hardware's estimate y of 1 / sqrt(d2) gives
// g = d2 y and h = y / 2, one step with the residual 1/2 - g h doubles the
// digits of both, and g + (d2 - g^2) h is the root to the last place or two.
// 1e-300 keeps a zero distance off the pole.
__device__ __forceinline__ double cube_of(double dx, double dy) {
    const double d2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, 1e-300));
    const double y = __builtin_amdgcn_rsq(d2);
    double g = d2 * y, h = 0.5 * y;
    const double e = __builtin_fma(-g, h, 0.5);
    g = __builtin_fma(g, e, g);
    h = __builtin_fma(h, e, h);
    g = __builtin_fma(__builtin_fma(-g, g, d2), h, g);
    return d2 * g;
}

// f(0), ..., f(N - 1) with the index as a compile-time constant.
template <class F, int... I>
__device__ __forceinline__ void each_index(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void each(F &&f) {
    each_index(static_cast<F &&>(f), std::make_integer_sequence<int, N>{});
}

// The M monomials of (x, y), in the order of eq. poly_sets.
template <int M> __device__ __forceinline__ void monomials(double x, double y, double (&q)[M]) {
    constexpr int D = M == 6 ? 2 : M == 10 ? 3 : 4;
    double xp[D + 1], yp[D + 1];
    xp[0] = yp[0] = 1.0;
#pragma unroll
    for (int e = 1; e <= D; ++e) {
        xp[e] = xp[e - 1] * x;
        yp[e] = yp[e - 1] * y;
    }
#pragma unroll
    for (int d = 0, i = 0; d <= D; ++d)
#pragma unroll
        for (int j = 0; j <= d; ++j, ++i) q[i] = xp[d - j] * yp[j];
}

// M polynomials, at most NP members beyond them (N2 <= NP, rows past N2 are an
// identity), K <= 32.
template <int M, int NP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_rbf_null(
    const Geo *__restrict__ geo, const double *__restrict__ xs, const double *__restrict__ ys,
    const int32_t *__restrict__ nbr, RhsList L, int n, int K, double dx,
    double *__restrict__ W64, int32_t *__restrict__ redo) {
    constexpr int NS = (NP + 15) / 16;      // members of set 2 per lane
    constexpr int RS = (M + 4) / 2 * 2;     // a member's row: LU row, x, y, slot (16-byte aligned)
    constexpr int SS = 32 * RS + 2;         // a system's rows; its neighbours use other banks
    __shared__ __align__(16) double s_rows[4 * SS];
    const int lane = threadIdx.x, grp = lane >> 4, ll = lane & 15;
    // owners in XCD-contiguous ranges, as in k_rbf (grid xcd_grid of the wavefronts)
    const int64_t s0 = xcd_tile(((int64_t)n + 3) / 4) * 4;
    if (s0 >= n) return;
    const bool live = s0 + grp < n;
    const int s = (int)(live ? s0 + grp : n - 1);
    const int count = live ? (L.ptr ? L.ptr[s + 1] - L.ptr[s] : 8) : 0;
    const int cmax = max(max(__builtin_amdgcn_readlane(count, 0), __builtin_amdgcn_readlane(count, 16)),
                         max(__builtin_amdgcn_readlane(count, 32), __builtin_amdgcn_readlane(count, 48)));
    if (cmax == 0) return;
    const Geo g = *geo;
    const int N2 = K - M;
    double *rows = s_rows + grp * SS;

    // members ll and ll + 16, relative to the owner and scaled by the radius
    double sx[2], sy[2], P[2][M];
    bool used[2];
    const double cx = xs[s], cy = ys[s];
    double far = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = ll + 16 * h;
        used[h] = r >= K;
        sx[h] = sy[h] = 0.0;
        if (r < K) {
            const int q = nbr[(int64_t)r * n + s];
            sx[h] = min_image(xs[q] - cx, g.Lx);
            sy[h] = min_image(ys[q] - cy, g.Ly);
        }
        far = fmax(far, sx[h] * sx[h] + sy[h] * sy[h]);
    }
    far = fmax(far, dpp_d<0xB1>(far));
    far = fmax(far, dpp_d<0x4E>(far));
    far = fmax(far, dpp_d<0x141>(far));
    far = fmax(far, dpp_d<0x140>(far));
    const double irad = far > 0.0 ? recip(sqrt(far)) : 1.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        sx[h] *= irad;
        sy[h] *= irad;
        monomials<M>(sx[h], sy[h], P[h]);
    }
    const double line = 1e6 * DBL_EPSILON * (8 * K + M);   // for the pivots of S
    auto store_row = [&](int at, int h) {
        double *o = rows + at * RS;
#pragma unroll
        for (int c = 0; c < M; ++c) o[c] = P[h][c];
        o[M] = sx[h];
        o[M + 1] = sy[h];
        reinterpret_cast<int *>(o + M + 2)[0] = ll + 16 * h;
    };

    // 1. P = L U: the pivot row goes to its place in pivot order, every lane
    // reads it back; rows that were pivots before are updated along and ignored
    double uinv = 0.0;
    each<M>([&](auto T) {
        constexpr int t = T;
        uint32_t key[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            key[h] = used[h] ? 0u : ((uint32_t)(__double_as_longlong(P[h][t]) >> 32) & 0x7FFFFFFFu) | 1u;
        uint32_t top = max(key[0], key[1]);
        top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0xB1, 0xF, 0xF, true));
        top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x4E, 0xF, 0xF, true));
        top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x141, 0xF, 0xF, true));
        top = max(top, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)top, 0x140, 0xF, 0xF, true));
        const bool hit0 = key[0] == top, hit1 = key[1] == top;
        const uint64_t hits = __ballot(hit0 || hit1);
        const bool me = ll == __builtin_ctz((uint32_t)(hits >> (16 * grp)) | 0x10000u);
        if (me && hit0) {
            store_row(t, 0);
            used[0] = true;
        }
        if (me && !hit0) {
            store_row(t, 1);
            used[1] = true;
        }
        wave_lds_sync();
        double U[M];
#pragma unroll
        for (int c = 0; c < M; ++c)
            if (c >= t) U[c] = rows[t * RS + c];
        const double pi = recip(U[t]);
        if (ll == t) uinv = pi;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double l = P[h][t] * pi;
            P[h][t] = l;
#pragma unroll
            for (int c = 0; c < M; ++c)
                if (c > t) P[h][c] = __builtin_fma(-l, U[c], P[h][c]);
        }
    });
    bool bad = !(fabs(uinv) < 1.0 / kSetPivot);   // lane t: pivot t
    // set 2 behind set 1, in stencil order
    {
        const uint32_t f0 = (uint32_t)(__ballot(!used[0]) >> (16 * grp)) & 0xFFFFu;
        const uint32_t f1 = (uint32_t)(__ballot(!used[1]) >> (16 * grp)) & 0xFFFFu;
        const uint32_t below = (1u << ll) - 1u;
        if (!used[0]) store_row(M + __popc(f0 & below), 0);
        if (!used[1]) store_row(M + __popc(f0) + __popc(f1 & below), 1);
    }
    wave_lds_sync();
    double LU[M], x1, y1, X[NS][M], x2[NS], y2[NS];
    int slot1, slot2[NS];
    {
        const double *o = rows + min(ll, M - 1) * RS;
#pragma unroll
        for (int c = 0; c < M; ++c) LU[c] = o[c];
        x1 = o[M];
        y1 = o[M + 1];
        slot1 = reinterpret_cast<const int *>(o + M + 2)[0];
    }
#pragma unroll
    for (int r = 0; r < NS; ++r) {
        const bool in = ll + 16 * r < N2;
        const double *o = rows + (in ? M + ll + 16 * r : 0) * RS;
#pragma unroll
        for (int c = 0; c < M; ++c) X[r][c] = in ? o[c] : 0.0;
        x2[r] = o[M];
        y2[r] = o[M + 1];
        slot2[r] = reinterpret_cast<const int *>(o + M + 2)[0];
    }
    // X = L2 L1^-1
    each<M>([&](auto T) {
        constexpr int t = M - 1 - T;
#pragma unroll
        for (int r = 0; r < NS; ++r) fmac_dot<t + 1, M, true>(X[r][t], &LU[t], X[r]);
    });

    // 2. S, row ll + 16 r in lane ll, with T1 = R21 - X R11 on the way
    double S[NS][NP], T1[M][NS];
    each<NP>([&](auto C) {
        constexpr int c = C;
        const double bx = lane_of<c % 16>(x2[c / 16]), by = lane_of<c % 16>(y2[c / 16]);
#pragma unroll
        for (int r = 0; r < NS; ++r) S[r][c] = cube_of(x2[r] - bx, y2[r] - by);
    });
    double XT[M][NS];   // X by column, as the broadcasts take it
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int r = 0; r < NS; ++r) XT[j][r] = X[r][j];
    each<M>([&](auto J) {
        constexpr int j = J;
        const double bx = lane_of<j>(x1), by = lane_of<j>(y1);
        const double r11 = cube_of(x1 - bx, y1 - by);
        double r21[NS];
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            r21[r] = cube_of(x2[r] - bx, y2[r] - by);
            T1[j][r] = r21[r];
            fmac_dot<0, M, true>(T1[j][r], &r11, X[r]);
        }
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            fmac_rows<0, NP, true>(S[r], r21, X[r][j]);
            fmac_rows<0, NP, true>(S[r], XT[j], T1[j][r]);
        }
    });
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < NS; ++r)
            if (c >= N2) S[r][c] = ll + 16 * r == c ? 1.0 : 0.0;
    // S = L D L^T without a search: -L below the diagonal, D L^T on and above it
    double dinv[NS];
#pragma unroll
    for (int r = 0; r < NS; ++r) dinv[r] = 0.0;
    each<NP>([&](auto Kc) {
        constexpr int k = Kc, rk = k / 16;
        const double d = lane_of<k % 16>(S[rk][k]);
        if (!(d > line)) bad = true;
        const double di = recip(d);
        if (ll == k % 16) dinv[rk] = di;
        double nl[NS];
#pragma unroll
        for (int r = rk; r < NS; ++r) {
            const bool under = ll + 16 * r > k;
            nl[r] = under ? -S[r][k] * di : 0.0;
            S[r][k] = under ? nl[r] : S[r][k];
        }
#pragma unroll
        for (int r = NS - 1; r > rk; --r) fmac_lane<k % 16, k + 1, NP>(S[r], S[rk], nl[r]);
        fmac_self<k % 16, k + 1, NP>(S[rk], nl[rk]);
    });
    if (((uint32_t)(__ballot(bad) >> (16 * grp)) & 0xFFFFu) != 0 && count > 0 && ll == 0)
        redo[1 + atomicAdd(&redo[0], 1)] = s;
    double ST[NP][NS];   // S by column
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
        for (int r = 0; r < NS; ++r) ST[c][r] = S[r][c];

    // 3. departure points, one a lane
    for (int c0 = 0; c0 < cmax; c0 += 16) {
        const bool on = c0 + ll < count;
        int p = 0, dir = 1;
        double qx = 0.0, qy = 0.0;
        if (on) {
            rhs_point(L, s, c0 + ll, p, dir);
            qx = (L.ptr ? min_image(xs[p] - lat_ex(dir) * dx - cx, g.Lx) : -lat_ex(dir) * dx) * irad;
            qy = (L.ptr ? min_image(ys[p] - lat_ey(dir) * dx - cy, g.Ly) : -lat_ey(dir) * dx) * irad;
        }
        double y[M], b[NP];
        monomials<M>(qx, qy, y);
        each<M>([&](auto T) {   // y U
            constexpr int t = T;
            fmac_dot<0, t, true>(y[t], &LU[t], y);
            y[t] *= lane_of<t>(uinv);
        });
        each<M>([&](auto T) {   // y L1
            constexpr int t = M - 1 - T;
            fmac_dot<t + 1, M, true>(y[t], &LU[t], y);
        });
        each<NP>([&](auto I) {
            constexpr int i = I;
            b[i] = cube_of(qx - lane_of<i % 16>(x2[i / 16]), qy - lane_of<i % 16>(y2[i / 16]));
        });
        each<M>([&](auto J) {
            constexpr int j = J;
            const double f1 = cube_of(qx - lane_of<j>(x1), qy - lane_of<j>(y1));
            fmac_rows<0, NP, true>(b, XT[j], f1);
            fmac_rows<0, NP, true>(b, T1[j], y[j]);
        });
        each<NP>([&](auto Kc) {
            constexpr int k = Kc;
            fmac_rows<k + 1, NP, false>(b, ST[k], b[k]);
        });
        each<NP>([&](auto Kc) {
            constexpr int k = NP - 1 - Kc;
            b[k] *= lane_of<k % 16>(dinv[k / 16]);
            fmac_rows<0, k, true>(b, ST[k], b[k]);
        });
        each<M>([&](auto J) {
            constexpr int j = J;
            fmac_dot<0, NP, true>(y[j], XT[j], b);
        });
        each<M>([&](auto J) {
            constexpr int j = J;
            const int at = lane_of<j>(slot1);
            if (on) W64[w64_at(dir, at, n, p)] = y[j];
        });
        each<NP>([&](auto I) {
            constexpr int i = I;
            const int at = lane_of<i % 16>(slot2[i / 16]);
            if (on && i < N2) W64[w64_at(dir, at, n, p)] = b[i];
        });
    }
}

// Owner -> departure-point lists of the paper's stencil rule (CSR): every point
// to the place it took in its owner's list (the order inside a list does not
// affect the solved weights). The counters are done with: their first word
// becomes the empty list of owners to solve again.
__global__ __launch_bounds__(256) void k_owned_fill(int n, const int32_t *__restrict__ owner,
                                                    int32_t *__restrict__ ptr,
                                                    const int32_t *__restrict__ slot,
                                                    int32_t *__restrict__ pts,
                                                    int32_t *__restrict__ redo) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)8 * n) return;
    const int k0 = (int)(i / n), p = (int)(i - (int64_t)k0 * n);   // owner is [8][n]
    pts[ptr[owner[i]] + slot[i]] = p * 8 + k0;
    if (i == 0) {
        ptr[n] = 8 * n;
        redo[0] = 0;
    }
}

// FP32 copy of the shape vectors in the streaming layout [K][2][n][4]
// (directions 1..4 and 5..8 as float4). After rounding, the weights of each
// (node, direction) no longer sum to one; the defect 1 - sum (evaluated in
// FP64) is added to one weight, the smallest in magnitude among those at least
// 64 times larger than the defect, so the rounded weights keep the partition
// of unity that the deviation-stored populations rely on. One thread per
// (node, direction), numbered like the FP32 layout: four consecutive lanes
// fill one node's float4, so a wavefront stores whole lines of each member
// plane (numbered like the FP64 layout instead, two far-apart workgroups each
// wrote half of every float4, and the partly written lines doubled the
// writes). Its loads are two 256-byte runs per wavefront and member, one in
// each direction pair's plane of the FP64 layout. The weights stay in
// registers between the three passes.
template <int KB>
__global__ __launch_bounds__(256) void k_pack_w32(const double *__restrict__ W64, int n, int K,
                                                  float *__restrict__ W32) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)8 * n) return;
    const int64_t plane = (int64_t)8 * n;   // distance between members j and j+1
    const int c = (int)(t & 3);              // direction within the half
    const int64_t hp = t >> 2;
    const int hh = (int)(hp / n);            // half: directions 1-4 or 5-8
    const int p = (int)(hp - (int64_t)hh * n);
    const int k = 4 * hh + c + 1;
    const int64_t src = w64_at(k, 0, n, p);
    double w[KB];
    double sum = 0.0;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
        w[j] = j < K ? W64[j * plane + src] : 0.0;
        sum += (double)(float)w[j];
    }
    const double defect = 1.0 - sum;
    int jstar = -1;
    double best = DBL_MAX;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
        const double a = fabs(w[j]);
        if (j < K && a >= 64.0 * fabs(defect) && a < best) {
            best = a;
            jstar = j;
        }
    }
    float *out = W32 + ((int64_t)hh * n + p) * 4 + c;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
        if (j < K) {
            float f = (float)w[j];
            if (j == jstar) f = (float)((double)f + defect);
            out[(int64_t)j * 8 * n] = f;
        }
    }
}

// Constant azimuthal acceleration about the origin (Sec. 3): a = g (-y, x)/r at
// fluid nodes, zero at wall nodes.
__global__ void k_force(const double *__restrict__ xs, const double *__restrict__ ys,
                        const uint8_t *__restrict__ nt, int n, double mag, float *f32,
                        double *f64) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double x = xs[p], y = ys[p];
    double r = sqrt(x * x + y * y);
    double ax = 0.0, ay = 0.0;
    if (!(nt && nt[p]) && r > 0.0) {
        ax = -mag * y / r;
        ay = mag * x / r;
    }
    if (f32) {
        f32[p] = (float)ax;
        f32[n + p] = (float)ay;
    }
    if (f64) {
        f64[p] = ax;
        f64[n + p] = ay;
    }
}

// Bounce-back link masks (Sec. 3): at wall node p (internal order), bit k-1
// is set when e_k . n < 0 for the outward normal n of the fluid domain, i.e.
// population k enters the fluid from outside the wall.
__global__ void k_links(const uint8_t *__restrict__ ntype, const int32_t *__restrict__ perm,
                        const double *__restrict__ nx, const double *__restrict__ ny, int n,
                        uint8_t *__restrict__ links) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    unsigned m = 0;
    if (ntype[p]) {
        const int u = perm[p];
        const double a = nx[u], b = ny[u];
        for (int k = 1; k < kQ; ++k)
            if (lat_ex(k) * a + lat_ey(k) * b < 0.0) m |= 1u << (k - 1);
    }
    links[p] = (uint8_t)m;
}

}  // namespace

hipError_t launch_links(const uint8_t *ntype, const int32_t *perm, const double *nx,
                        const double *ny, int n, uint8_t *links, hipStream_t s) {
    hipLaunchKernelGGL(k_links, dim3(blocks_for(n, 256)), dim3(256), 0, s, ntype, perm, nx, ny,
                       n, links);
    return hipGetLastError();
}

hipError_t launch_reset(int32_t *err, int32_t *stats, int nstats, hipStream_t s) {
    hipLaunchKernelGGL(k_reset, dim3(blocks_for(std::max(nstats, 1), 256)), dim3(256), 0, s, err, stats,
                       nstats);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

// Workspace of the search and the solve: owner counts [n] (then the list of
// owners to solve again, n + 1), list offsets [n + 1] (the search's list before
// that), points [8 n] (the sort's counters before that), scan. Counts and
// offsets share what n and n + 1 words take when each starts a 256-byte line:
// a fixed workspace that held a build without the lists still holds it.
struct OwnedLists {
    int32_t *cnt, *ptr, *pts;
    char *scan;
    size_t scan_bytes;
    static size_t lines(size_t bytes) { return (bytes + 255) & ~size_t(255); }
    static size_t head(int n) { return lines((size_t)n * 4) + lines(((size_t)n + 1) * 4); }
    static size_t points(int n) { return lines((size_t)8 * n * 4); }
    OwnedLists(void *tmp, size_t bytes, int n) {
        cnt = (int32_t *)tmp;
        ptr = cnt + (((size_t)n + 1 + 3) & ~size_t(3));
        pts = (int32_t *)((char *)tmp + head(n));
        scan = (char *)pts + points(n);
        scan_bytes = bytes - (size_t)(scan - (char *)tmp);
    }
};

// Internal order of the nodes: Hilbert key of the cell, then user index. A
// counting sort where the keys are at most four a node (square domains have half
// a key to one, 1:4 ones four; their counters and offsets then fit the place of
// the point lists) and the sort's temporary memory holds the scan's; longer
// domains sort the keys. Both give the same order. A build of a small cloud is
// bound by its launches (about 5 us each), and the library's sort took five of
// them at 10,201 nodes and sixteen at 262,144; the counting sort takes three or
// four, the clearing of counters and lists one more, where it took six. Whole
// builds, with the lists' counts in k_owner: 10,201 nodes 27 launches to 16, 252
// to 199 us; 262,144 nodes 1,651 to 1,538 us.
hipError_t launch_order(const BuildOrder &o, hipStream_t s) {
    const int n = o.n;
    const OwnedLists lists(o.rbf_tmp, o.rbf_bytes, n);
    const int64_t all = (int64_t)1 << (2 * o.hb);
    const bool counted = o.hb < 15 && all <= (int64_t)4 * n && scan_temp_bytes((int)all) <= o.sort_bytes;
    const int nkeys = counted ? (int)all : 0, ncells = o.gx * o.gy;
    int32_t *cnt = counted ? lists.pts : nullptr, *off = lists.pts + nkeys;
    Geo g{};
    if (o.Lx > 0 && o.Ly > 0) {
        g.cw = o.Lx / o.gx;
        g.ch = o.Ly / o.gy;
        g.Lx = o.Lx;
        g.Ly = o.Ly;
        g.gx = o.gx;
        g.gy = o.gy;
        g.hb = o.hb;
    } else {
        hipLaunchKernelGGL(k_geo_bbox, dim3(1), dim3(1024), 0, s, o.geo, o.x, o.y, n, o.gx, o.gy, o.hb);
    }
    const dim3 grid(blocks_for(n, 256)), block(256);
    hipLaunchKernelGGL(k_begin, dim3(blocks_for(std::max(ncells, std::max(nkeys, 1)), 256)), block, 0, s,
                       o.geo, g, ncells, o.cstart, o.cend, nkeys, cnt);
    hipLaunchKernelGGL(k_keys, grid, block, 0, s, o.geo, o.x, o.y, n, o.keys, o.vals, cnt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (counted) {
        if ((e = exclusive_scan(o.sort_tmp, o.sort_bytes, cnt, off, nkeys, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_place, grid, block, 0, s, n, o.keys, o.vals, off, (int32_t *)o.skeys);
        hipLaunchKernelGGL(k_scatter_sorted<true>, grid, block, 0, s, o.geo, o.x, o.y, o.nt, o.perm,
                           o.keys, (const int32_t *)o.skeys, off, nkeys, n, o.xs, o.ys, o.ntype, o.iperm,
                           o.cstart, o.cend, lists.cnt, lists.ptr);
    } else {
        if ((e = sort_pairs(o.sort_tmp, o.sort_bytes, o.keys, o.skeys, o.vals, o.perm, n,
                            std::max(1, 2 * o.hb), s)) != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_scatter_sorted<false>, grid, block, 0, s, o.geo, o.x, o.y, o.nt, o.perm,
                           o.skeys, nullptr, nullptr, 0, n, o.xs, o.ys, o.ntype, o.iperm, o.cstart,
                           o.cend, lists.cnt, lists.ptr);
    }
    return hipGetLastError();
}

hipError_t launch_knn(const Geo *geo, const double *xs, const double *ys,
                      const int32_t *perm, const int32_t *cstart,
                      const int32_t *cend, int n, int K, void *tmp, size_t tmp_bytes, int32_t *nbr,
                      hipStream_t s) {
    int32_t *redo = OwnedLists(tmp, tmp_bytes, n).ptr;   // emptied by launch_order
    const dim3 grid(xcd_grid(blocks_for(n, 256 / kKnnLanes)));
    auto kernel = K <= 16 ? k_knn<32> : K <= 32 ? k_knn<64> : k_knn<96>;   // room for a third more
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, geo, xs, ys, perm, cstart, cend, n, K, redo, nbr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_knn_redo, dim3(1024), dim3(64), 0, s, geo, xs, ys, perm, cstart, cend, n, K,
                       redo, nbr);
    return hipGetLastError();
}

hipError_t launch_owner(const Geo *geo, const double *xs, const double *ys,
                        const int32_t *perm, const int32_t *cstart, const int32_t *cend, int n,
                        double dx, int32_t *owner, void *tmp, size_t tmp_bytes, int32_t *slot,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_owner, dim3(xcd_grid(blocks_for(n, 32))), dim3(256), 0, s, geo, xs, ys,
                       perm, cstart, cend, n, dx, owner, OwnedLists(tmp, tmp_bytes, n).cnt, slot);
    return hipGetLastError();
}

// Sizes of k_rbf_null: N2 = K - M members beyond the polynomials, rounded up.
template <int M>
static hipError_t launch_rbf_null(const Geo *geo, const double *xs, const double *ys,
                                  const int32_t *perm, const int32_t *nbr, RhsList L, int n, int K,
                                  int m, double dx, int32_t *redo, double *W64, int32_t *dev_err,
                                  hipStream_t s) {
    const int N2 = K - M;
    auto kernel = N2 <= 8 ? k_rbf_null<M, 8> : N2 <= 12 ? k_rbf_null<M, 12> : k_rbf_null<M, 16>;
    if constexpr (M == 10)
        if (N2 > 16) kernel = N2 <= 20 ? k_rbf_null<M, 20> : k_rbf_null<M, 24>;
    if constexpr (M == 6)
        if (N2 > 16) kernel = N2 <= 20 ? k_rbf_null<M, 20> : k_rbf_null<M, 28>;
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(blocks_for(n, 4))), dim3(64), 0, s, geo, xs, ys, nbr, L,
                       n, K, dx, W64, redo);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rbf_redo, dim3(256), dim3(64), 0, s, geo, xs, ys, perm, nbr, L, n, K, m, dx,
                       redo, W64, dev_err);
    return hipGetLastError();
}

size_t rbf_temp_bytes(int n) {
    return OwnedLists::head(n) + OwnedLists::points(n) + scan_temp_bytes(n) + 256;
}

hipError_t launch_rbf(const Geo *geo, const double *xs, const double *ys,
                      const int32_t *perm, const int32_t *nbr, const int32_t *owner,
                      int n, int K, int m, double dx, int mode, void *tmp, size_t tmp_bytes,
                      double *W64, int32_t *dev_err, hipStream_t s) {
    RhsList L{nullptr, nullptr};
    const OwnedLists lists(tmp, tmp_bytes, n);
    if (mode == MLBM_STENCIL_PAPER) {
        hipError_t e = exclusive_scan(lists.scan, lists.scan_bytes, lists.cnt, lists.ptr, n, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_owned_fill, dim3(blocks_for((int64_t)8 * n, 256)), dim3(256), 0, s, n,
                           owner, lists.ptr, (const int32_t *)W64, lists.pts, lists.cnt);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        L.ptr = lists.ptr;
        L.pts = lists.pts;
    }
    // Stencils of up to 32 nodes take the null-space solver (31 at degree 4,
    // where its registers end): 262,144 nodes, whole build, before -> with it,
    // K 30 degree 4 5.7 -> 2.3 ms, K 25 degree 3 4.9 -> 1.8, K 25 degree 2
    // 3.3 -> 1.9, K 20 degree 3 3.1 -> 1.6, K 15 degree 2 2.0 -> 1.1, K 12
    // degree 2 (own stencils) 1.5 -> 0.7. Its list of owners to solve again
    // takes the place of the owners' counters, which are done with.
    int32_t *redo = lists.cnt;
    if (K <= (m == 4 ? 31 : 32)) {
        if (m == 2)
            return launch_rbf_null<6>(geo, xs, ys, perm, nbr, L, n, K, m, dx, redo, W64, dev_err, s);
        if (m == 3)
            return launch_rbf_null<10>(geo, xs, ys, perm, nbr, L, n, K, m, dx, redo, W64, dev_err, s);
        return launch_rbf_null<15>(geo, xs, ys, perm, nbr, L, n, K, m, dx, redo, W64, dev_err, s);
    }
    // Larger ones the general elimination: up to 48 unknowns on the matrix
    // cores (10 % faster than a row per lane, 262,144 nodes, 45 unknowns); at
    // 64 the register tiles leave two wavefronts per SIMD and a row per lane
    // is faster (K 47: 10.3 against 11.2 ms build)
    if (K + poly_count(m) <= 48) {
        hipLaunchKernelGGL(k_rbf_mfma<3>, dim3(xcd_grid(n)), dim3(64), 0, s, geo, xs, ys, perm, nbr, L,
                           n, K, m, dx, W64, dev_err);
        return hipGetLastError();
    }
    // own-node stencils (exactly 8 departure points per owner) take the
    // kernel without the replay, which need not keep the multipliers (the
    // register allocator would park them in scratch memory). Splitting the
    // paper rule's owners the same way (at most 8 departure points, then the
    // rest) measured slower: the second launch runs a sparse tail.
    const dim3 grid(xcd_grid(blocks_for(n, 4))), block(256);
    if (L.ptr)
        hipLaunchKernelGGL((k_rbf<64, 8, 2, true>), grid, block, 0, s, geo, xs, ys, perm, nbr, L, n, K,
                           m, dx, W64, dev_err);
    else
        hipLaunchKernelGGL((k_rbf<64, 8, 3, false>), grid, block, 0, s, geo, xs, ys, perm, nbr, L, n, K,
                           m, dx, W64, dev_err);
    return hipGetLastError();
}

hipError_t launch_pack_w32(const double *W64, int n, int K, float *W32, hipStream_t s) {
    const dim3 grid(blocks_for((int64_t)8 * n, 256)), block(256);
    if (K <= 16)
        hipLaunchKernelGGL(k_pack_w32<16>, grid, block, 0, s, W64, n, K, W32);
    else if (K <= 32)
        hipLaunchKernelGGL(k_pack_w32<32>, grid, block, 0, s, W64, n, K, W32);
    else
        hipLaunchKernelGGL(k_pack_w32<kMaxK>, grid, block, 0, s, W64, n, K, W32);
    return hipGetLastError();
}

hipError_t launch_force(const double *xs, const double *ys, const uint8_t *ntype, int n,
                        int kind, double mag, float *f32, double *f64, hipStream_t s) {
    if (kind == 0) return hipSuccess;
    hipLaunchKernelGGL(k_force, dim3(blocks_for(n, 256)), dim3(256), 0, s, xs, ys, ntype, n,
                       mag, f32, f64);
    return hipGetLastError();
}

}  // namespace mlbm
