// Time stepping of the MLBM on gfx950: initial equilibrium, the fused
// stream + collide step, moments and error reductions.
//
// One lane owns one node. Per step and node the kernel
//   1. interpolates every moving population k = 1..8 at its departure point:
//      f_k(i) = sum_j W[k][j][i] * g_k(nbr[j][s]), s the stencil owner
//      (Sec. 2.3; Appendix A, STREAM); k = 0 departs from the node itself;
//   2. imposes the wall rule at wall nodes;
//   3. takes the moments (eq. macro_var) and applies BGK collision with the
//      optional body force (eqs. LBM_collision, feq; Sec. 3);
//   4. writes the post-collision populations g for the next step.
// The state g is kept post-collision, so one kernel per step reads each
// population once and writes it once; this is the paper's COLLIDE-STREAM order
// shifted by half a step.
//
// The FP32 form stores every population as its deviation from w_k rho0 (the
// populations are O(1) while the flow lives in O(u) corrections); the weights
// reproduce constants, so the streamed deviation is the interpolated
// deviation. The FP64 form stores plain populations.
//
// Memory: the stencil weights dominate the traffic (8K per node per step); they
// are read once, unit-stride across the lanes of a wavefront. The populations
// gathered through nbr are re-used by neighbouring nodes and are served from
// L2; nodes are in Hilbert order so the gathers of a workgroup stay local.
#include <algorithm>

#include "common.h"

namespace mlbm {
namespace {

// ------------------------------------------------------------------------
// FP32, deviation-stored populations
// ------------------------------------------------------------------------

// Bounce-back wall rule (Sec. 3): each population flagged in the node's link
// mask (bit k-1: it enters the fluid from outside the wall) takes the
// streamed value of the opposite direction. Flagged directions point into the
// fluid, so their opposites are never flagged.
template <class T>
__device__ __forceinline__ void bounce_back(unsigned links, T (&f)[kQ]) {
    if (!links) return;
    T g[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) g[k] = f[k];
#pragma unroll
    for (int k = 1; k < kQ; ++k)
        if ((links >> (k - 1)) & 1u) f[k] = g[lat_opp(k)];
}

// Moments, wall rule, BGK collision with force, and the stores of one node.
// WALL: 0 none; 1 equilibrium wall nodes (node = its type); 2 bounce-back
// (node = its link mask). (ax, ay): the node's body force.
// Directions k0 <= k < k1 are stored (all of them by default; the two lanes
// of a node in the split step store one part each).
template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void collide_at32(int n, int p, float (&f)[kQ],
                                                float *__restrict__ go, unsigned node, float ax,
                                                float ay, float rtau, float rho0, float rho_w,
                                                float *__restrict__ frec, int32_t *err,
                                                const int32_t *perm, int uoff, int k0 = 0,
                                                int k1 = kQ) {
    if (WALL == 1 && node) {
#pragma unroll
        for (int k = 0; k < kQ; ++k) {
            if (k < k0 || k >= k1) continue;
            const float v = lat_wmul(k, rho_w - rho0);
            go[(int64_t)k * n + p] = v;
            if (REC) frec[(int64_t)k * n + p] = v;
        }
        return;
    }
    if (WALL == 2) bounce_back(node, f);
    float drho = 0.0f, jx = 0.0f, jy = 0.0f;
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        drho += f[k];
        jx += f[k] * (float)lat_ex(k);
        jy += f[k] * (float)lat_ey(k);
    }
    const float rho = rho0 + drho;
    const float ux = jx / rho, uy = jy / rho;
    const float uu = ux * ux + uy * uy;
    if (k0 == 0) check_speed(err, uu, perm, p, uoff);
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        if (k < k0 || k >= k1) continue;
        const float eu = (float)lat_ex(k) * ux + (float)lat_ey(k) * uy;
        const float feq = lat_wmul(k, drho + rho * (3.0f * eu + 4.5f * eu * eu - 1.5f * uu));
        float v = f[k] - (f[k] - feq) * rtau;
        if (FORCE) v += lat_wmul(k, 3.0f * ((float)lat_ex(k) * ax + (float)lat_ey(k) * ay));
        go[(int64_t)k * n + p] = v;
        if (REC) frec[(int64_t)k * n + p] = f[k];
    }
}

// The same with the node's mark and force read here.
template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void collide_store32(int n, int p, float (&f)[kQ],
                                                float *__restrict__ go,
                                                const float *__restrict__ force,
                                                const uint8_t *__restrict__ ntype, float rtau,
                                                float rho0, float rho_w,
                                                float *__restrict__ frec, int32_t *err,
                                                const int32_t *perm, int uoff, int k0 = 0,
                                                int k1 = kQ) {
    collide_at32<FORCE, WALL, REC>(n, p, f, go, WALL ? ntype[p] : 0u, FORCE ? force[p] : 0.0f,
                                   FORCE ? force[n + p] : 0.0f, rtau, rho0, rho_w, frec, err, perm,
                                   uoff, k0, k1);
}

// One workgroup per tile of kTile nodes. Tiles with gather tables (tdesc
// |H_t| > 0) stage the 8 moving populations of the tile's halo H_t and the
// tile-local stencils of its owners in LDS, then every interpolation reads LDS
// only; HBM sees the weights, the tile tables and the halo rows, all
// contiguous. Tiles without tables gather through global memory.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// One row of four FP32 weights; non-temporal loads do not keep the line in
// the caches.
__device__ __forceinline__ float4 load_w(const float4 *p, bool nt) {
    const f32x4 *q = reinterpret_cast<const f32x4 *>(p);
    const f32x4 v = nt ? __builtin_nontemporal_load(q) : *q;
    return make_float4(v.x, v.y, v.z, v.w);
}

// One pair of FP64 weights, non-temporal.
__device__ __forceinline__ double2 load_w2(const double2 *p) {
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    const f64x2 v = __builtin_nontemporal_load(reinterpret_cast<const f64x2 *>(p));
    return make_double2(v.x, v.y);
}

// Staging of a tile (before its barrier), NTH threads. Every load of a lane
// is issued before the first LDS store, so the L2 round trips overlap
// instead of following one another: the halo populations (a halo holds at
// most kHaloCap nodes, so at most kHaloCap / NTH per lane) and the index
// words (in batches of four per lane).
template <int NTH>
__device__ __forceinline__ void stage_halo32(const float *__restrict__ g, int n,
                                             const int32_t *__restrict__ hl, int nh,
                                             float *__restrict__ gl, int32_t *err, int tid) {
    constexpr int U = (kHaloCap + NTH - 1) / NTH;
    int q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int h = tid + u * NTH;
        int v = h < nh ? hl[h] : 0;
        if ((unsigned)v >= (unsigned)n) {   // a bad table must not fault
            v = 0;
            report_index(err);
        }
        q[u] = v;
    }
    float v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int d = 0; d < 8; ++d)
            v[u][d] = tid + u * NTH < nh ? g[(int64_t)(d + 1) * n + q[u]] : 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int h = tid + u * NTH;
        if (h < nh) {
#pragma unroll
            for (int d = 0; d < 8; ++d) gl[d * nh + h] = v[u][d];
        }
    }
}

template <int NTH>
__device__ __forceinline__ void stage_words(uint32_t *__restrict__ dst,
                                            const uint32_t *__restrict__ src, int count,
                                            int tid) {
    for (int b = 0; b < count; b += 4 * NTH) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int w = b + tid + u * NTH;
            v[u] = w < count ? src[w] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int w = b + tid + u * NTH;
            if (w < count) dst[w] = v[u];
        }
    }
}

// Halo size of a tile that stages its tables, 0 for one that gathers from
// global memory: no tables, or tables larger than the launch's LDS (a plan
// built inside a graph capture sizes its LDS before the tables exist).
__device__ __forceinline__ int tile_halo(const Step32Args &a, int64_t tile) {
    if (!a.tdesc) return 0;
    const int nh = a.tdesc[2 * tile + 1];
    const int no = a.tdesc[2 * tile];
    return nh > 0 && 32 * nh + 4 * no * ((a.K + 2) / 3) <= a.lcap ? nh : 0;
}

template <int MODE, bool FORCE, int WALL, bool REC, int UNROLL, bool NT>
__device__ __forceinline__ void step32_tile(const Step32Args &a, const float *__restrict__ g,
                                            float *__restrict__ go, int64_t tile,
                                            unsigned char *smem) {
    const int n = a.n, K = a.K;
    const int base = (int)(tile * kTile);
    const int cnt = min(kTile, n - base);
    const int tid = threadIdx.x;
    const int nh = tile_halo(a, tile);
    const float4 *__restrict__ W = a.W;

    float acc[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] = 0.0f;

    if (nh > 0) {
        const int no = a.tdesc[2 * tile];
        const int Kw = (K + 2) / 3;                                  // index words per owner
        float *gl = reinterpret_cast<float *>(smem);                 // [8][nh]
        uint32_t *nl = reinterpret_cast<uint32_t *>(gl + 8 * nh);    // [no][Kw]
        const int32_t *hl = a.hlist + tile * (int64_t)a.hcap;
        stage_halo32<kTile>(g, n, hl, nh, gl, a.err, tid);
        stage_words<kTile>(nl, a.nbrL + tile * (int64_t)a.ocap * Kw, no * Kw, tid);
        __syncthreads();
        if (tid >= cnt) return;
        const int p = base + tid;
        int ol[8];
#pragma unroll
        for (int d = 0; d < 8; ++d)
            ol[d] = (MODE == MLBM_STENCIL_OWN ? tid : (int)a.ownerL[(int64_t)d * n + p]) * Kw;
        // stencil slots j = 3w, 3w+1, 3w+2 share index word w (10 bits each)
#pragma unroll UNROLL
        for (int w = 0; w < Kw; ++w) {
            uint32_t word[8];
#pragma unroll
            for (int d = 0; d < 8; ++d)
                word[d] = (MODE == MLBM_STENCIL_OWN && d > 0) ? word[0] : nl[ol[d] + w];
#pragma unroll
            for (int sft = 0; sft < 3; ++sft) {
                const int jj = 3 * w + sft;
                if (jj < K) {
                    const float4 wa = load_w(W + ((int64_t)jj * 2) * n + p, NT);
                    const float4 wb = load_w(W + ((int64_t)jj * 2 + 1) * n + p, NT);
                    const float wv[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
#pragma unroll
                    for (int d = 0; d < 8; ++d)
                        acc[d] = __builtin_fmaf(
                            wv[d], gl[d * nh + (int)((word[d] >> (10 * sft)) & 1023u)], acc[d]);
                }
            }
        }
        float f[kQ];
        f[0] = g[p];
#pragma unroll
        for (int d = 0; d < 8; ++d) f[d + 1] = acc[d];
        collide_store32<FORCE, WALL, REC>(n, p, f, go, a.force, a.ntype, a.rtau, a.rho0,
                                          a.rho_w, a.frec, a.err, a.perm, a.uoff);
        return;
    }

    if (tid >= cnt) return;
    const int p = base + tid;
    constexpr int UJ = 3 * UNROLL;
    int s[8];
#pragma unroll
    for (int d = 0; d < 8; ++d)
        s[d] = MODE == MLBM_STENCIL_OWN ? p : a.owner[(int64_t)d * n + p];
#pragma unroll UJ
    for (int j = 0; j < K; ++j) {
        const float4 wa = load_w(W + ((int64_t)j * 2) * n + p, NT);
        const float4 wb = load_w(W + ((int64_t)j * 2 + 1) * n + p, NT);
        const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
        if (MODE == MLBM_STENCIL_OWN) {
            const int q = a.nbr[(int64_t)j * n + p];
#pragma unroll
            for (int d = 0; d < 8; ++d)
                acc[d] = __builtin_fmaf(w[d], g[(int64_t)(d + 1) * n + q], acc[d]);
        } else {
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const int q = a.nbr[(int64_t)j * n + s[d]];
                acc[d] = __builtin_fmaf(w[d], g[(int64_t)(d + 1) * n + q], acc[d]);
            }
        }
    }
    float f[kQ];
    f[0] = g[p];
#pragma unroll
    for (int d = 0; d < 8; ++d) f[d + 1] = acc[d];
    collide_store32<FORCE, WALL, REC>(n, p, f, go, a.force, a.ntype, a.rtau, a.rho0, a.rho_w,
                                      a.frec, a.err, a.perm, a.uoff);
}

// The same tile with two lanes per node (adjacent lanes; 2 kTile threads):
// lane h of node l interpolates directions 4h+1 .. 4h+4, the pair swaps its
// four sums with a DPP exchange, and both lanes finish the node identically
// (same values, same order), lane 0 storing directions 0..4 and lane 1 5..8.
// The tile's LDS is unchanged, so a compute unit holds twice the wavefronts
// for the same tiles. Per direction the sums run in the same order as in
// step32_tile, so the results are bitwise the same.
__device__ __forceinline__ float swap_pair(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF,
                                                      false));   // quad_perm [1,0,3,2]
}

template <int MODE, bool FORCE, int WALL, bool REC, bool NT, int UNROLL>
__device__ __forceinline__ void step32_tile_split(const Step32Args &a,
                                                  const float *__restrict__ g,
                                                  float *__restrict__ go, int64_t tile,
                                                  unsigned char *smem) {
    const int n = a.n, K = a.K;
    const int base = (int)(tile * kTile);
    const int cnt = min(kTile, n - base);
    const int tid = threadIdx.x, l = tid >> 1, h = tid & 1;
    const int nh = tile_halo(a, tile);
    const float4 *__restrict__ W = a.W;
    float acc[4];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) acc[dd] = 0.0f;

    if (nh > 0) {
        const int no = a.tdesc[2 * tile];
        const int Kw = (K + 2) / 3;
        float *gl = reinterpret_cast<float *>(smem);                 // [8][nh]
        uint32_t *nl = reinterpret_cast<uint32_t *>(gl + 8 * nh);    // [no][Kw]
        const int32_t *hl = a.hlist + tile * (int64_t)a.hcap;
        stage_halo32<2 * kTile>(g, n, hl, nh, gl, a.err, tid);
        stage_words<2 * kTile>(nl, a.nbrL + tile * (int64_t)a.ocap * Kw, no * Kw, tid);
        __syncthreads();
        if (l >= cnt) return;   // both lanes of a node leave together
        const int p = base + l;
        int ol[4];
#pragma unroll
        for (int dd = 0; dd < 4; ++dd)
            ol[dd] = (MODE == MLBM_STENCIL_OWN ? l
                                               : (int)a.ownerL[(int64_t)(4 * h + dd) * n + p]) * Kw;
        const float *glh = gl + 4 * h * nh;
#pragma unroll UNROLL
        for (int w = 0; w < Kw; ++w) {
            uint32_t word[4];
#pragma unroll
            for (int dd = 0; dd < 4; ++dd)
                word[dd] = (MODE == MLBM_STENCIL_OWN && dd > 0) ? word[0] : nl[ol[dd] + w];
#pragma unroll
            for (int sft = 0; sft < 3; ++sft) {
                const int jj = 3 * w + sft;
                if (jj < K) {
                    const float4 wv = load_w(W + ((int64_t)jj * 2 + h) * n + p, NT);
                    const float wt[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
                    for (int dd = 0; dd < 4; ++dd)
                        acc[dd] = __builtin_fmaf(
                            wt[dd], glh[dd * nh + (int)((word[dd] >> (10 * sft)) & 1023u)], acc[dd]);
                }
            }
        }
    } else {
        if (l >= cnt) return;
        const int p = base + l;
        int s[4];
#pragma unroll
        for (int dd = 0; dd < 4; ++dd)
            s[dd] = MODE == MLBM_STENCIL_OWN ? p : a.owner[(int64_t)(4 * h + dd) * n + p];
        for (int j = 0; j < K; ++j) {
            const float4 wv = load_w(W + ((int64_t)j * 2 + h) * n + p, NT);
            const float wt[4] = {wv.x, wv.y, wv.z, wv.w};
#pragma unroll
            for (int dd = 0; dd < 4; ++dd) {
                const int q = a.nbr[(int64_t)j * n + s[dd]];
                acc[dd] = __builtin_fmaf(wt[dd], g[(int64_t)(4 * h + dd + 1) * n + q], acc[dd]);
            }
        }
    }
    const int p = base + l;
    float oth[4];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) oth[dd] = swap_pair(acc[dd]);
    float f[kQ];
    f[0] = g[p];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        f[1 + dd] = h ? oth[dd] : acc[dd];
        f[5 + dd] = h ? acc[dd] : oth[dd];
    }
    collide_store32<FORCE, WALL, REC>(n, p, f, go, a.force, a.ntype, a.rtau, a.rho0, a.rho_w,
                                      a.frec, a.err, a.perm, a.uoff, h ? 5 : 0, h ? kQ : 5);
}

template <int MODE, bool FORCE, int WALL, bool REC, bool NT, int UNROLL>
__global__ __launch_bounds__(2 * kTile) void k_step32s(Step32Args a, const float *__restrict__ g,
                                                       float *__restrict__ go, int64_t nblocks) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t tile = xcd_tile(nblocks);
    if (tile >= nblocks) return;
    step32_tile_split<MODE, FORCE, WALL, REC, NT, UNROLL>(a, g, go, tile, smem);
}

template <int MODE, bool FORCE, int WALL, bool REC, int UNROLL, bool NT>
__global__ __launch_bounds__(kTile) void k_step32(Step32Args a, const float *__restrict__ g,
                                                  float *__restrict__ go, int64_t nblocks) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t tile = xcd_tile(nblocks);
    if (tile >= nblocks) return;
    step32_tile<MODE, FORCE, WALL, REC, UNROLL, NT>(a, g, go, tile, smem);
}

// All tiles of all clouds of a batched plan in one launch: the tile's cloud
// comes from tile2cloud, its arrays and parameters from the descriptor table;
// the state of cloud c starts soff elements into g and go.
template <int MODE, int UNROLL, bool NT>
__global__ __launch_bounds__(kTile) void k_step32_batch(const Step32Args *__restrict__ descs,
                                                        const int32_t *__restrict__ tile2cloud,
                                                        const float *__restrict__ g,
                                                        float *__restrict__ go,
                                                        XcdSplit xs) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t t = xcd_split_tile(xs);
    if (t < 0) return;
    const Step32Args a = descs[tile2cloud[t]];
    step32_tile<MODE, false, false, false, UNROLL, NT>(a, g + a.soff, go + a.soff,
                                                        t - a.tile_begin, smem);
}

template <int MODE, bool NT, int UNROLL>
__global__ __launch_bounds__(2 * kTile) void k_step32s_batch(const Step32Args *__restrict__ descs,
                                                             const int32_t *__restrict__ tile2cloud,
                                                             const float *__restrict__ g,
                                                             float *__restrict__ go,
                                                             XcdSplit xs) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t t = xcd_split_tile(xs);
    if (t < 0) return;
    const Step32Args a = descs[tile2cloud[t]];
    step32_tile_split<MODE, false, false, false, NT, UNROLL>(a, g + a.soff, go + a.soff,
                                                             t - a.tile_begin, smem);
}

// Writes one batch descriptor (a kernel, so that graph capture records it).
__global__ void k_set_desc(Step32Args *dst, Step32Args v) { *dst = v; }

// ------------------------------------------------------------------------
// FP64, plain populations
// ------------------------------------------------------------------------
template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void collide_at64(int n, int p, double (&f)[kQ],
                                                double *__restrict__ go, unsigned node,
                                                double ax, double ay, double rtau,
                                                double rho_w, double *__restrict__ frec,
                                                int32_t *err, const int32_t *perm, int uoff,
                                                int k0 = 0, int k1 = kQ) {
    if (WALL == 1 && node) {
#pragma unroll
        for (int k = 0; k < kQ; ++k) {
            if (k < k0 || k >= k1) continue;
            const double v = lat_w(k) * rho_w;
            go[(int64_t)k * n + p] = v;
            if (REC) frec[(int64_t)k * n + p] = v;
        }
        return;
    }
    if (WALL == 2) bounce_back(node, f);
    double rho = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        rho += f[k];
        jx += f[k] * lat_ex(k);
        jy += f[k] * lat_ey(k);
    }
    const double ux = jx / rho, uy = jy / rho;
    const double uu = ux * ux + uy * uy;
    if (k0 == 0) check_speed(err, uu, perm, p, uoff);
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        if (k < k0 || k >= k1) continue;
        const double eu = lat_ex(k) * ux + lat_ey(k) * uy;
        const double feq = lat_w(k) * rho * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        double v = f[k] - (f[k] - feq) * rtau;
        if (FORCE) v += 3.0 * lat_w(k) * (lat_ex(k) * ax + lat_ey(k) * ay);
        go[(int64_t)k * n + p] = v;
        if (REC) frec[(int64_t)k * n + p] = f[k];
    }
}

template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void collide_store64(int n, int p, double (&f)[kQ],
                                                double *__restrict__ go,
                                                const double *__restrict__ force,
                                                const uint8_t *__restrict__ ntype, double rtau,
                                                double rho_w, double *__restrict__ frec,
                                                int32_t *err, const int32_t *perm, int uoff) {
    collide_at64<FORCE, WALL, REC>(n, p, f, go, WALL ? ntype[p] : 0u, FORCE ? force[p] : 0.0,
                                   FORCE ? force[n + p] : 0.0, rtau, rho_w, frec, err, perm, uoff);
}

// Same structure as the FP32 step, with the same tile tables: a tile stages
// its halo four directions at a time (4 x |H_t| doubles take the LDS that 8 x
// |H_t| floats take), so the directions are interpolated in two passes. (One
// pass over 8 x |H_t| doubles fits the LDS too, but the larger footprint
// lowers the workgroups per CU and measured slower.)
template <int MODE, bool FORCE, int WALL, bool REC>
__global__ __launch_bounds__(kTile) void k_step64(
    int n, int K, int64_t nblocks, const double *__restrict__ g, double *__restrict__ go,
    const double *__restrict__ W, const int32_t *__restrict__ nbr,
    const int32_t *__restrict__ owner, const double *__restrict__ force,
    const uint8_t *__restrict__ ntype, double rtau, double rho_w, double *__restrict__ frec,
    const int32_t *__restrict__ tdesc, const uint16_t *__restrict__ ownerL,
    const uint32_t *__restrict__ nbrL, const int32_t *__restrict__ hlist, int ocap, int hcap,
    int32_t *err, const int32_t *__restrict__ perm, int uoff) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t tile = xcd_tile(nblocks);
    if (tile >= nblocks) return;
    const int base = (int)(tile * kTile);
    const int cnt = min(kTile, n - base);
    const int tid = threadIdx.x;
    const int p = base + tid;
    const int nh = tdesc ? tdesc[2 * tile + 1] : 0;

    double acc[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) acc[d] = 0.0;
    const double2 *W2 = reinterpret_cast<const double2 *>(W);   // [K][4][n] pairs

    if (nh > 0) {
        const int no = tdesc[2 * tile];
        const int Kw = (K + 2) / 3;
        double *gl = reinterpret_cast<double *>(smem);               // [4][nh]
        uint32_t *nl = reinterpret_cast<uint32_t *>(gl + 4 * nh);    // [no][Kw]
        const int32_t *hl = hlist + tile * (int64_t)hcap;
        const uint32_t *src = nbrL + tile * (int64_t)ocap * Kw;
        for (int w = tid; w < no * Kw; w += kTile) nl[w] = src[w];
        int ol[8];
#pragma unroll
        for (int d = 0; d < 8; ++d)
            ol[d] = tid < cnt ? (MODE == MLBM_STENCIL_OWN ? tid : (int)ownerL[(int64_t)d * n + p]) * Kw
                              : 0;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
            if (pass) __syncthreads();   // the first half is read by everyone
            for (int h = tid; h < nh; h += kTile) {
                int q = hl[h];
                if ((unsigned)q >= (unsigned)n) {   // a bad table must not fault
                    q = 0;
                    report_index(err);
                }
#pragma unroll
                for (int dd = 0; dd < 4; ++dd)
                    gl[dd * nh + h] = g[(int64_t)(4 * pass + dd + 1) * n + q];
            }
            __syncthreads();
            if (tid < cnt) {
#pragma unroll 2
                for (int w = 0; w < Kw; ++w) {
                    uint32_t word[4];
#pragma unroll
                    for (int dd = 0; dd < 4; ++dd)
                        word[dd] = nl[ol[MODE == MLBM_STENCIL_OWN ? 0 : 4 * pass + dd] + w];
#pragma unroll
                    for (int sft = 0; sft < 3; ++sft) {
                        const int jj = 3 * w + sft;
                        if (jj < K) {
                            // directions 4 pass + 1 .. 4 pass + 4 as two pairs
                            // streamed once per step: non-temporal
                            const double2 wa = load_w2(W2 + ((int64_t)jj * 4 + 2 * pass) * n + p);
                            const double2 wb =
                                load_w2(W2 + ((int64_t)jj * 4 + 2 * pass + 1) * n + p);
                            const double wt[4] = {wa.x, wa.y, wb.x, wb.y};
#pragma unroll
                            for (int dd = 0; dd < 4; ++dd)
                                acc[4 * pass + dd] = __builtin_fma(
                                    wt[dd], gl[dd * nh + (int)((word[dd] >> (10 * sft)) & 1023u)],
                                    acc[4 * pass + dd]);
                        }
                    }
                }
            }
        }
        if (tid >= cnt) return;
    } else {
        if (tid >= cnt) return;
        int s[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) s[d] = MODE == MLBM_STENCIL_OWN ? p : owner[(int64_t)d * n + p];
        for (int j = 0; j < K; ++j) {
            int qo = 0;
            if (MODE == MLBM_STENCIL_OWN) qo = nbr[(int64_t)j * n + p];
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const double w = W[w64_at(d + 1, j, n, p)];
                const int q = MODE == MLBM_STENCIL_OWN ? qo : nbr[(int64_t)j * n + s[d]];
                acc[d] = __builtin_fma(w, g[(int64_t)(d + 1) * n + q], acc[d]);
            }
        }
    }
    double f[kQ];
    f[0] = g[p];
#pragma unroll
    for (int d = 0; d < 8; ++d) f[d + 1] = acc[d];
    collide_store64<FORCE, WALL, REC>(n, p, f, go, force, ntype, rtau, rho_w, frec, err, perm,
                                      uoff);
}

// ------------------------------------------------------------------------
// Small clouds, both precisions
// ------------------------------------------------------------------------

// Arguments of the small-cloud step.
template <class T> struct WideArgs {
    int n, K, ocap, hcap;
    const T *W;
    const int32_t *nbr, *owner;
    const T *force;
    const uint8_t *ntype;
    T rtau, rho0, rho_w;
    T *frec;
    const int32_t *tdesc;
    const uint16_t *ownerL;
    const uint32_t *nbrL;
    const int32_t *hlist;
    int32_t *err;
    const int32_t *perm;
    int uoff;
    int nhcap;   // halo nodes that the launch's LDS holds
    int direct;  // longest own-node stencil that gathers from memory (wide_direct)
};

// A value at a byte offset from a uniform base: a scalar address and a 32-bit
// lane offset, without 64-bit vector arithmetic.
template <class V>
__device__ __forceinline__ V load_at(const void *base, uint32_t off) {
    return *reinterpret_cast<const V *>(static_cast<const char *>(base) + off);
}

__device__ __forceinline__ float wide_fma(float w, float x, float acc) {
    return __builtin_fmaf(w, x, acc);
}
__device__ __forceinline__ double wide_fma(double w, double x, double acc) {
    return __builtin_fma(w, x, acc);
}

template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void wide_finish(const WideArgs<float> &a, int p, float (&f)[kQ],
                                            float *go, unsigned node, float ax, float ay,
                                            int k0, int k1) {
    collide_at32<FORCE, WALL, REC>(a.n, p, f, go, node, ax, ay, a.rtau, a.rho0, a.rho_w, a.frec,
                                   a.err, a.perm, a.uoff, k0, k1);
}
template <bool FORCE, int WALL, bool REC>
__device__ __forceinline__ void wide_finish(const WideArgs<double> &a, int p, double (&f)[kQ],
                                            double *go, unsigned node, double ax, double ay,
                                            int k0, int k1) {
    collide_at64<FORCE, WALL, REC>(a.n, p, f, go, node, ax, ay, a.rtau, a.rho_w, a.frec, a.err,
                                   a.perm, a.uoff, k0, k1);
}

// The step for clouds that leave the chip mostly idle (wide_dirs). There the
// tile kernels spend their time waiting: one workgroup per 256 nodes leaves
// most CUs empty, and each of its lanes goes through its weights in turn, a
// wait for memory and for LDS per slot. Here 32 D nodes make a workgroup and
// a lane takes D directions of one node, so the same work is spread over
// eight (D = 1) or four times the CUs; a lane asks for the weights of its
// first 36 slots and for its tables before it waits for anything, so that
// their round trips run under the halo's (tables, then populations); and the
// slots are taken six at a time without branches. Every workgroup stages the
// halo of its whole tile. Sums and collision are in the tile kernels' order,
// so the states are bitwise the same. 6,400 nodes, K 25: FP64 32.4 -> 6.1 us
// a step, FP32 8.3 -> 5.4; 1,600 nodes, K 12: FP32 5.6 -> 4.7, FP64 8.8 -> 4.8.
// Of those, 2.7 us go by for a launch and one trip to memory, two more for the
// halo's. Short own-node stencils gather from global memory instead (wide_direct):
// 1,600 nodes, K 12, 4.7 -> 4.0 (FP32) and 4.8 -> 4.5 us (FP64); at K 20 both
// ways cost the same, at K 30 the halo is cheaper (FP64 6.0 against 6.3), and
// with two directions a lane it is at every K (22,500 nodes FP64 6.4 / 8.4).
template <class T, int MODE, bool FORCE, int WALL, bool REC, int D>
__device__ __forceinline__ void wide_group(const WideArgs<T> &a, const T *__restrict__ g,
                                           T *__restrict__ go, int64_t tile, int first,
                                           unsigned char *smem) {
    typedef T TD __attribute__((ext_vector_type(D)));
    constexpr int NN = 32 * D;          // nodes of the workgroup
    constexpr int CH = 6, NC = 6;       // weight slots per chunk, chunks held
    constexpr int U = kHaloCap / 256;
    // FP32 rows of weights are two float4 a slot, FP64 rows four double2
    constexpr int RPS = sizeof(T) == 4 ? 2 : 4, EPR = 8 / RPS, LPR = EPR / D;
    const int n = a.n, K = a.K, Kw = (K + 2) / 3;
    if (tile * kTile + first >= n) return;          // uniform
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // LPR lanes share a node's row of EPR weights; a wavefront holds 64 / LPR
    // nodes of one row, and the rows follow one another over the wavefronts
    constexpr int WPR = NN * LPR / 64;              // wavefronts per row
    const int row = wv / WPR;
    const int nd = (wv % WPR) * (64 / LPR) + lane / LPR;    // node within the workgroup
    const int d0 = row * EPR + (lane % LPR) * D;            // first of this lane's directions, from 0
    const int pt = (int)(tile * kTile) + first + nd;
    const int p = min(pt, n - 1);                   // a lane past the last node repeats it
    const T *wbase = a.W + (int64_t)row * n * EPR;
    const uint32_t woff = (uint32_t)(p * EPR + (lane % LPR) * D) * sizeof(T);
    auto weights = [&](int j) { return load_at<TD>(wbase + (int64_t)j * 8 * n, woff); };
    // short own-node stencils: a lane's populations are fewer than its share of the
    // halo, and need the stencil alone (no halo list, no LDS)
    const bool direct = MODE == MLBM_STENCIL_OWN && D == 1 && K <= a.direct;
    int q[U] = {};
    if (a.tdesc && !direct) {   // (every tile has room for kHaloCap entries: no wait for its count)
        const int32_t *hl = a.hlist + tile * (int64_t)a.hcap;
#pragma unroll
        for (int u = 0; u < U; ++u) q[u] = load_at<int32_t>(hl, (uint32_t)(tid + u * 256) * 4);
    }
    const int nh0 = a.tdesc && !direct ? a.tdesc[2 * tile + 1] : 0;
    const int nh = nh0 <= a.nhcap ? nh0 : 0;
    T acc[D];
#pragma unroll
    for (int i = 0; i < D; ++i) acc[i] = 0;
    // the values of the node this lane finishes, asked for with the tables
    const int fn = tid & (NN - 1), part = tid / NN;   // 256 / NN lanes finish a node
    const int fp = (int)(tile * kTile) + first + fn;
    const int fq = min(fp, n - 1);
    const T f0 = g[fq];
    const unsigned node = WALL ? a.ntype[fq] : 0u;
    const T ax = FORCE ? a.force[fq] : (T)0, ay = FORCE ? a.force[n + fq] : (T)0;
    T *gl = reinterpret_cast<T *>(smem);                // [8][nh]
    if (nh > 0) {
        int ol[D];
#pragma unroll
        for (int i = 0; i < D; ++i)
            ol[i] = MODE == MLBM_STENCIL_OWN ? p - (int)(tile * kTile)
                                             : (int)a.ownerL[(int64_t)(d0 + i) * n + p];
        // Chunks of six slots, without branches inside a chunk, so that its
        // loads and LDS reads are in flight together. Slots from K on repeat
        // the weights of slot K - 1 and read the zero cell behind the halo
        // (adding a zero to a sum that starts at +0 changes nothing).
        TD w[NC][CH];
        uint32_t wd[NC][2][D];
        const uint32_t *nl = a.nbrL + tile * (int64_t)a.ocap * Kw;
        auto load = [&](int c) {
#pragma unroll
            for (int j = 0; j < CH; ++j) w[c % NC][j] = weights(min(c * CH + j, K - 1));
        };
        auto words = [&](int c) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < D; ++i)
                    wd[c % NC][h][i] =
                        MODE == MLBM_STENCIL_OWN && i
                            ? wd[c % NC][h][0]
                            : load_at<uint32_t>(nl + min(2 * c + h, Kw - 1), (uint32_t)(ol[i] * Kw) * 4);
        };
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c * CH < K) load(c);
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c * CH < K) words(c);
        T v[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = tid + u * 256 < nh;
            if (in && (unsigned)q[u] >= (unsigned)n) {   // a bad table must not fault
                q[u] = 0;
                report_index(a.err);
            }
            if (in) {
#pragma unroll
                for (int d = 0; d < 8; ++d)
                    v[u][d] = load_at<T>(g + (int64_t)(d + 1) * n, (uint32_t)q[u] * sizeof(T));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (tid + u * 256 < nh) {
#pragma unroll
                for (int d = 0; d < 8; ++d) gl[d * nh + tid + u * 256] = v[u][d];
            }
        if (tid == 0) gl[8 * nh] = 0;
        __syncthreads();
        const T *glp = gl + d0 * nh;
        const int zero = (8 - d0) * nh;
#pragma unroll
        for (int c = 0; c < kMaxK / CH; ++c) {
            if (c * CH < K) {
                T x[CH][D];
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int i = 0; i < D; ++i) {
                        const int at = (int)((wd[c % NC][j / 3][i] >> (10 * (j % 3))) & 1023u);
                        x[j][i] = glp[c * CH + j < K ? i * nh + at : zero];
                    }
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int i = 0; i < D; ++i) acc[i] = wide_fma(w[c % NC][j][i], x[j][i], acc[i]);
                if (c + NC < kMaxK / CH && (c + NC) * CH < K) {
                    load(c + NC);
                    words(c + NC);
                }
            }
        }
        __syncthreads();   // the halo is read by everyone: its space takes the sums
    } else if (direct) {
        TD w[3][CH];
        int at[3][CH];
        T x[3][CH][D];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c * CH < K) {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int jj = min(c * CH + j, K - 1);
                    at[c][j] = load_at<int32_t>(a.nbr + (int64_t)jj * n, (uint32_t)p * 4);
                    w[c][j] = weights(jj);
                }
            }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c * CH < K) {
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int i = 0; i < D; ++i)
                        x[c][j][i] = load_at<T>(g + (int64_t)(d0 + i + 1) * n,
                                                (uint32_t)at[c][j] * sizeof(T));
            }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            if (c * CH < K) {
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int i = 0; i < D; ++i)
                        acc[i] = wide_fma(w[c][j][i], c * CH + j < K ? x[c][j][i] : (T)0, acc[i]);
            }
    } else {
        int s[D];
#pragma unroll
        for (int i = 0; i < D; ++i)
            s[i] = MODE == MLBM_STENCIL_OWN ? p : a.owner[(int64_t)(d0 + i) * n + p];
        for (int j = 0; j < K; ++j) {
            const TD wt = weights(j);
#pragma unroll
            for (int i = 0; i < D; ++i)
                acc[i] = wide_fma(wt[i], g[(int64_t)(d0 + i + 1) * n + a.nbr[(int64_t)j * n + s[i]]],
                                  acc[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < D; ++i) gl[(d0 + i) * NN + nd] = acc[i];
    __syncthreads();
    if (fp >= n) return;
    T f[kQ];
    f[0] = f0;
#pragma unroll
    for (int d = 0; d < 8; ++d) f[d + 1] = gl[d * NN + fn];
    wide_finish<FORCE, WALL, REC>(a, fp, f, go, node, ax, ay, part ? part * D + 1 : 0, part * D + D + 1);
}

template <class T, int MODE, bool FORCE, int WALL, bool REC, int D>
__global__ __launch_bounds__(256) void k_step_wide(WideArgs<T> a, const T *__restrict__ g,
                                                   T *__restrict__ go, int64_t nblocks) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int PER = kTile / (32 * D);   // workgroups per tile
    const int64_t b = xcd_tile(nblocks);
    if (b >= nblocks) return;
    wide_group<T, MODE, FORCE, WALL, REC, D>(a, g, go, b / PER, (int)(b % PER) * 32 * D, smem);
}

// The same over all tiles of a batched plan, as k_step32_batch.
template <int MODE, int D>
__global__ __launch_bounds__(256) void k_step_wide_batch(const Step32Args *__restrict__ descs,
                                                         const int32_t *__restrict__ tile2cloud,
                                                         const float *__restrict__ g,
                                                         float *__restrict__ go, int64_t nblocks,
                                                         int nhcap, int direct) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int PER = kTile / (32 * D);
    const int64_t b = xcd_tile(nblocks);
    if (b >= nblocks) return;
    const int64_t t = b / PER;
    const Step32Args &s = descs[tile2cloud[t]];
    WideArgs<float> a{};
    a.n = s.n;
    a.K = s.K;
    a.ocap = s.ocap;
    a.hcap = s.hcap;
    a.W = reinterpret_cast<const float *>(s.W);
    a.nbr = s.nbr;
    a.owner = s.owner;
    a.rtau = s.rtau;
    a.rho0 = s.rho0;
    a.rho_w = s.rho_w;
    a.tdesc = s.tdesc;
    a.ownerL = s.ownerL;
    a.nbrL = s.nbrL;
    a.hlist = s.hlist;
    a.err = s.err;
    a.perm = s.perm;
    a.uoff = s.uoff;
    a.nhcap = nhcap;
    a.direct = direct;
    wide_group<float, MODE, false, 0, false, D>(a, g + s.soff, go + s.soff, t - s.tile_begin,
                                                (int)(b % PER) * 32 * D, smem);
}

// ------------------------------------------------------------------------
// Initial state, moments, L2 sums
// ------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void init_node(int p, int n, const int32_t *__restrict__ perm,
                                          const double *__restrict__ rho,
                                          const double *__restrict__ ux,
                                          const double *__restrict__ uy,
                                          const uint8_t *__restrict__ ntype,
                                          const double *__restrict__ force, double rho0,
                                          double rho_w, int wall, int dev, int collide,
                                          T *__restrict__ g) {
    const int u = perm ? perm[p] : p;
    double r = rho ? rho[u] : rho0;
    double vx = ux ? ux[u] : 0.0, vy = uy ? uy[u] : 0.0;
    const bool is_wall = wall && ntype && ntype[p];
    if (is_wall) {
        r = rho_w;
        vx = vy = 0.0;
    }
    const double uu = vx * vx + vy * vy;
    for (int k = 0; k < kQ; ++k) {
        const double eu = lat_ex(k) * vx + lat_ey(k) * vy;
        // feq - w rho0 = w [(rho - rho0) + rho (3 eu + 4.5 eu^2 - 1.5 u^2)]
        double v = dev ? lat_w(k) * ((r - rho0) + r * (3.0 * eu + 4.5 * eu * eu - 1.5 * uu))
                       : lat_w(k) * r * (1.0 + 3.0 * eu + 4.5 * eu * eu - 1.5 * uu);
        if (collide && force && !is_wall)
            v += 3.0 * lat_w(k) * (lat_ex(k) * force[p] + lat_ey(k) * force[n + p]);
        g[(int64_t)k * n + p] = (T)v;
    }
}

template <class T>
__global__ void k_init(int n, const int32_t *__restrict__ perm, const double *__restrict__ rho,
                       const double *__restrict__ ux, const double *__restrict__ uy,
                       const uint8_t *__restrict__ ntype, const double *__restrict__ force,
                       double rho0, double rho_w, int wall, int dev, int collide,
                       T *__restrict__ g) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n)
        init_node<T>(p, n, perm, rho, ux, uy, ntype, force, rho0, rho_w, wall, dev, collide, g);
}

// Initial state (collided or not: a batched plan has no force) and moments of all
// clouds of a batched plan in one launch each, a workgroup a tile: with one
// launch a cloud, 24 clouds of 67,018 nodes together took 100 us of host time for
// the one and 92 for the other, now 14 and 15 with the call's own.
__global__ __launch_bounds__(kTile) void k_init_batch(const Step32Args *__restrict__ descs,
                                                      const int32_t *__restrict__ tile2cloud,
                                                      const double *__restrict__ rho,
                                                      const double *__restrict__ ux,
                                                      const double *__restrict__ uy,
                                                      float *__restrict__ g) {
    const int64_t t = blockIdx.x;
    const Step32Args &a = descs[tile2cloud[t]];
    const int p = (int)(t - a.tile_begin) * kTile + (int)threadIdx.x;
    if (p < a.n)
        init_node<float>(p, a.n, a.perm, rho ? rho + a.uoff : nullptr, ux ? ux + a.uoff : nullptr,
                         uy ? uy + a.uoff : nullptr, nullptr, nullptr, a.rho0_64, 0.0, 0, 1, 0,
                         g + a.soff);
}

template <class T>
__device__ __forceinline__ void moments_node(int p, int n, const int32_t *__restrict__ perm,
                                             const T *__restrict__ g,
                                             const float *__restrict__ f32,
                                             const double *__restrict__ f64,
                                             const uint8_t *__restrict__ ntype, double rho0,
                                             int dev, double *__restrict__ rho,
                                             double *__restrict__ ux, double *__restrict__ uy,
                                             int32_t *err, int uoff) {
    double r = 0.0, jx = 0.0, jy = 0.0;
    for (int k = 0; k < kQ; ++k) {
        const double v = (double)g[(int64_t)k * n + p];
        r += v;
        jx += v * lat_ex(k);
        jy += v * lat_ey(k);
    }
    if (dev) r += rho0;
    if (!(ntype && ntype[p])) {   // the force term added momentum a at fluid nodes
        if (f32) {
            jx -= (double)f32[p];
            jy -= (double)f32[n + p];
        } else if (f64) {
            jx -= f64[p];
            jy -= f64[n + p];
        }
    }
    const int u = perm ? perm[p] : p;
    const double vx = jx / r, vy = jy / r;
    check_speed(err, vx * vx + vy * vy, perm, p, uoff);
    if (rho) rho[u] = r;
    if (ux) ux[u] = vx;
    if (uy) uy[u] = vy;
}

template <class T>
__global__ void k_moments(int n, const int32_t *__restrict__ perm, const T *__restrict__ g,
                          const float *__restrict__ f32, const double *__restrict__ f64,
                          const uint8_t *__restrict__ ntype, double rho0, int dev,
                          double *__restrict__ rho, double *__restrict__ ux,
                          double *__restrict__ uy, int32_t *err, int uoff) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) moments_node<T>(p, n, perm, g, f32, f64, ntype, rho0, dev, rho, ux, uy, err, uoff);
}

__global__ __launch_bounds__(kTile) void k_moments_batch(const Step32Args *__restrict__ descs,
                                                         const int32_t *__restrict__ tile2cloud,
                                                         const float *__restrict__ g,
                                                         double *__restrict__ rho,
                                                         double *__restrict__ ux,
                                                         double *__restrict__ uy) {
    const int64_t t = blockIdx.x;
    const Step32Args &a = descs[tile2cloud[t]];
    const int p = (int)(t - a.tile_begin) * kTile + (int)threadIdx.x;
    if (p < a.n)
        moments_node<float>(p, a.n, a.perm, g + a.soff, nullptr, nullptr, nullptr, a.rho0_64, 1,
                            rho ? rho + a.uoff : nullptr, ux ? ux + a.uoff : nullptr,
                            uy ? uy + a.uoff : nullptr, a.err, a.uoff);
}

// Per-block partial sums, then a single workgroup adds the partials in a fixed
// order (deterministic, no floating-point atomics).
template <class T>
__global__ __launch_bounds__(256) void k_l2_partial(
    int n, const int32_t *__restrict__ perm, const T *__restrict__ g,
    const float *__restrict__ f32, const double *__restrict__ f64,
    const uint8_t *__restrict__ ntype, double rho0, int dev, const double *__restrict__ uxt,
    const double *__restrict__ uyt, double *__restrict__ part, int32_t *err, int uoff) {
    __shared__ double sh[4][256];
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    if (p < n) {
        double r = 0.0, jx = 0.0, jy = 0.0;
        for (int k = 0; k < kQ; ++k) {
            const double v = (double)g[(int64_t)k * n + p];
            r += v;
            jx += v * lat_ex(k);
            jy += v * lat_ey(k);
        }
        if (dev) r += rho0;
        if (!(ntype && ntype[p])) {
            if (f32) {
                jx -= (double)f32[p];
                jy -= (double)f32[n + p];
            } else if (f64) {
                jx -= f64[p];
                jy -= f64[n + p];
            }
        }
        const int u = perm[p];
        const double vx = jx / r, vy = jy / r;
        check_speed(err, vx * vx + vy * vy, perm, p, uoff);
        const double ex = vx - uxt[u], ey = vy - uyt[u];
        a0 = ex * ex + ey * ey;
        a1 = uxt[u] * uxt[u] + uyt[u] * uyt[u];
        a2 = ex * ex;
        a3 = uxt[u] * uxt[u];
    }
    sh[0][threadIdx.x] = a0;
    sh[1][threadIdx.x] = a1;
    sh[2][threadIdx.x] = a2;
    sh[3][threadIdx.x] = a3;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 4) part[(int64_t)blockIdx.x * 4 + threadIdx.x] = sh[threadIdx.x][0];
}

// Speed |u| of every node against the speed of an earlier check (user order,
// overwritten with the current speed): part[block] = (sum (|u| - |u_prev|)^2,
// sum |u|^2, 0, 0). The relative residual of the steady-state runs is
// sqrt(out[0] / out[1]).
template <class T>
__global__ __launch_bounds__(256) void k_residual_partial(
    int n, const int32_t *__restrict__ perm, const T *__restrict__ g,
    const float *__restrict__ f32, const double *__restrict__ f64,
    const uint8_t *__restrict__ ntype, double rho0, int dev, double *__restrict__ speed,
    double *__restrict__ part, int32_t *err, int uoff) {
    __shared__ double sh[2][256];
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    double a0 = 0, a1 = 0;
    if (p < n) {
        double r = 0.0, jx = 0.0, jy = 0.0;
        for (int k = 0; k < kQ; ++k) {
            const double v = (double)g[(int64_t)k * n + p];
            r += v;
            jx += v * lat_ex(k);
            jy += v * lat_ey(k);
        }
        if (dev) r += rho0;
        if (!(ntype && ntype[p])) {
            if (f32) {
                jx -= (double)f32[p];
                jy -= (double)f32[n + p];
            } else if (f64) {
                jx -= f64[p];
                jy -= f64[n + p];
            }
        }
        const int u = perm[p];
        const double U = sqrt(jx * jx + jy * jy) / r;
        check_speed(err, U * U, perm, p, uoff);
        const double d = U - speed[u];
        a0 = d * d;
        a1 = U * U;
        speed[u] = U;
    }
    sh[0][threadIdx.x] = a0;
    sh[1][threadIdx.x] = a1;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sh[0][threadIdx.x] += sh[0][threadIdx.x + w];
            sh[1][threadIdx.x] += sh[1][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x * 4 + 0] = sh[0][0];
        part[blockIdx.x * 4 + 1] = sh[1][0];
        part[blockIdx.x * 4 + 2] = 0.0;
        part[blockIdx.x * 4 + 3] = 0.0;
    }
}

__global__ __launch_bounds__(256) void k_l2_final(int64_t nparts, const double *__restrict__ part,
                                                  double *__restrict__ out) {
    __shared__ double sh[4][256];
    double a[4] = {0, 0, 0, 0};
    for (int64_t b = threadIdx.x; b < nparts; b += 256)
        for (int c = 0; c < 4; ++c) a[c] += part[b * 4 + c];
    for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] = a[c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 4) out[threadIdx.x] = sh[threadIdx.x][0];
}

// Collision only (g = C(f)), same arithmetic as the fused step after its
// streaming part.
template <class T>
__global__ void k_collide(int n, const T *__restrict__ f, T *__restrict__ g,
                          const double *__restrict__ force, const uint8_t *__restrict__ ntype,
                          int wall, double rtau, double rho0, double rho_w, int dev) {
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    if (wall && ntype && ntype[p]) {
        for (int k = 0; k < kQ; ++k)
            g[(int64_t)k * n + p] = (T)(dev ? lat_w(k) * (rho_w - rho0) : lat_w(k) * rho_w);
        return;
    }
    T fk[kQ];
    T drho = 0, jx = 0, jy = 0;
    for (int k = 0; k < kQ; ++k) {
        fk[k] = f[(int64_t)k * n + p];
        drho += fk[k];
        jx += fk[k] * (T)lat_ex(k);
        jy += fk[k] * (T)lat_ey(k);
    }
    const T rho = dev ? (T)rho0 + drho : drho;
    const T ux = jx / rho, uy = jy / rho, uu = ux * ux + uy * uy;
    for (int k = 0; k < kQ; ++k) {
        const T eu = (T)lat_ex(k) * ux + (T)lat_ey(k) * uy;
        const T poly = (T)3 * eu + (T)4.5 * eu * eu - (T)1.5 * uu;
        const T feq = dev ? lat_wmul(k, drho + rho * poly) : lat_wmul(k, rho * ((T)1 + poly));
        T v = fk[k] - (fk[k] - feq) * (T)rtau;
        if (force)
            v += (T)(3.0 * lat_w(k) * (lat_ex(k) * force[p] + lat_ey(k) * force[n + p]));
        g[(int64_t)k * n + p] = v;
    }
}

// Tuning variants of the FP32 step: unroll depth of the stencil loop over
// index words (1, 2 or 3 words = 3, 6 or 9 weight rows a lane has in flight)
// and non-temporal weight loads (the weights are streamed once per step and
// need not displace the halo rows in L2). Variant v < 6: one lane per node,
// unroll {1, 2, 3}[v / 2], non-temporal v % 2. Tiles without tables unroll
// their row loop 3x that. Variants 6-9: two lanes per node (directions split
// in halves), non-temporal v % 2, the index-word loop unrolled 2x from 8 on.
template <int MODE, bool FORCE, int WALL, bool REC, int UNROLL, bool NT>
void launch32(const CloudPlan &cp, const void *gin, void *gout, void *frec, int64_t nblocks,
              hipStream_t s) {
    const Step32Args a = step32_args(cp, frec);
    hipLaunchKernelGGL((k_step32<MODE, FORCE, WALL, REC, UNROLL, NT>), dim3(xcd_grid(nblocks)),
                       dim3(kTile), cp.lds_bytes, s, a, (const float *)gin, (float *)gout,
                       nblocks);
}

template <int MODE, bool FORCE, int WALL, bool REC, bool NT, int UNROLL = 1>
void launch32s(const CloudPlan &cp, const void *gin, void *gout, void *frec, int64_t nblocks,
               hipStream_t s) {
    const Step32Args a = step32_args(cp, frec);
    hipLaunchKernelGGL((k_step32s<MODE, FORCE, WALL, REC, NT, UNROLL>), dim3(xcd_grid(nblocks)),
                       dim3(2 * kTile), cp.lds_bytes, s, a, (const float *)gin, (float *)gout,
                       nblocks);
}

template <int MODE, bool NT, int UNROLL = 1>
void launch32s_batch(const mlbm_plan &plan, const void *gin, void *gout, hipStream_t s) {
    hipLaunchKernelGGL((k_step32s_batch<MODE, NT, UNROLL>), dim3(8 * plan.xcd_longest),
                       dim3(2 * kTile), plan.batch_lds, s, plan.descs, plan.tile2cloud,
                       (const float *)gin, (float *)gout, plan.xcd);
}

template <int MODE, int UNROLL, bool NT>
void launch32_batch(const mlbm_plan &plan, const void *gin, void *gout, hipStream_t s) {
    hipLaunchKernelGGL((k_step32_batch<MODE, UNROLL, NT>), dim3(8 * plan.xcd_longest),
                       dim3(kTile), plan.batch_lds, s, plan.descs, plan.tile2cloud,
                       (const float *)gin, (float *)gout, plan.xcd);
}

template <int MODE, bool FORCE, int WALL, bool REC>
void launch32_tuned(const CloudPlan &cp, const void *gin, void *gout, void *frec,
                    int64_t nblocks, hipStream_t s) {
    if (WALL == 2 || FORCE != (WALL == 1)) {   // other wall/force mixes: default variant
        launch32<MODE, FORCE, WALL, REC, 1, false>(cp, gin, gout, frec, nblocks, s);
        return;
    }
    switch (cp.variant) {
        case 1: launch32<MODE, FORCE, WALL, REC, 1, true>(cp, gin, gout, frec, nblocks, s); break;
        case 2: launch32<MODE, FORCE, WALL, REC, 2, false>(cp, gin, gout, frec, nblocks, s); break;
        case 3: launch32<MODE, FORCE, WALL, REC, 2, true>(cp, gin, gout, frec, nblocks, s); break;
        case 4: launch32<MODE, FORCE, WALL, REC, 3, false>(cp, gin, gout, frec, nblocks, s); break;
        case 5: launch32<MODE, FORCE, WALL, REC, 3, true>(cp, gin, gout, frec, nblocks, s); break;
        case 6: launch32s<MODE, FORCE, WALL, REC, false>(cp, gin, gout, frec, nblocks, s); break;
        case 7: launch32s<MODE, FORCE, WALL, REC, true>(cp, gin, gout, frec, nblocks, s); break;
        case 8: launch32s<MODE, FORCE, WALL, REC, false, 2>(cp, gin, gout, frec, nblocks, s); break;
        case 9: launch32s<MODE, FORCE, WALL, REC, true, 2>(cp, gin, gout, frec, nblocks, s); break;
        default: launch32<MODE, FORCE, WALL, REC, 1, false>(cp, gin, gout, frec, nblocks, s); break;
    }
}

// Halo nodes that a launch's LDS holds (64 KiB at most: a tile past that gathers
// from global memory).
template <class T> int wide_halo(int nh_max) {
    return std::min(nh_max, (int)(65536 / sizeof(T) - 2) / 8);
}

// Longest own-node stencils that gather from memory with one direction a lane. The
// more workgroups a CU has, the more of the halo's trip is covered. FP32, us a step,
// gathers / halo: K 6 3.5 / 4.1 at 16,384 nodes, 4.4 / 5.1 at 31,684; K 12 4.2 / 4.4 at
// 16,384, 5.0 / 4.9 at 18,225; K 15 4.3 / 4.4 at 8,100, 4.8 / 4.6 at 10,000, 6.0 / 5.3 at
// 24,336. FP64 K 12 4.1 / 4.4 at 8,100, K 15 4.7 / 4.7, K 30 at 6,400 6.3 / 6.0.
inline int wide_direct(int64_t n) {
    return n <= 8192 ? 18 : n <= 16384 ? 12 : n <= 32768 ? 6 : 0;
}

template <class T> WideArgs<T> wide_args(const CloudPlan &cp, void *frec) {
    WideArgs<T> a{};
    a.n = cp.n;
    a.K = cp.K;
    a.ocap = cp.ocap;
    a.hcap = cp.hcap;
    if constexpr (sizeof(T) == 8) {
        a.W = cp.W64;
        a.force = cp.force64;
    } else {
        a.W = cp.W32;
        a.force = cp.force32;
    }
    a.nbr = cp.nbr;
    a.owner = cp.owner;
    a.ntype = cp.prm.wall_kind == 2 ? cp.links : cp.ntype;
    a.rtau = (T)(1.0 / cp.prm.tau);
    a.rho0 = (T)cp.prm.rho0;
    a.rho_w = (T)cp.prm.rho_wall;
    a.frec = (T *)frec;
    a.tdesc = cp.lds_bytes ? cp.tdesc : nullptr;
    a.ownerL = cp.ownerL;
    a.nbrL = cp.nbrL;
    a.hlist = cp.hlist;
    a.err = cp.err;
    a.perm = cp.perm;
    a.uoff = (int)cp.off;
    a.nhcap = wide_halo<T>(cp.nh_max);
    a.direct = wide_direct(cp.n);
    return a;
}

// the halo's populations and a zero, then the sums of the workgroup's nodes in their place
template <class T> unsigned wide_lds(int nhcap, int nodes) {
    return (unsigned)(8 * std::max(nhcap, nodes) + 2) * sizeof(T);
}

template <class T, int MODE, bool FORCE, int WALL, bool REC>
void launch_wide(const CloudPlan &cp, int dirs, const void *gin, void *gout, void *frec,
                 hipStream_t s) {
    const int nodes = 32 * dirs;   // of a workgroup
    const int64_t nb = ((int64_t)cp.n + nodes - 1) / nodes;
    const WideArgs<T> a = wide_args<T>(cp, frec);
    const unsigned lds = wide_lds<T>(a.nhcap, nodes);
    auto kernel = dirs == 1 ? k_step_wide<T, MODE, FORCE, WALL, REC, 1>
                            : k_step_wide<T, MODE, FORCE, WALL, REC, 2>;
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(nb)), dim3(256), lds, s, a, (const T *)gin, (T *)gout,
                       nb);
}

// Directions a lane takes in the small-cloud step, 0 for the tile kernels: one (32
// nodes a workgroup) while that leaves few workgroups a CU, then two (64), until the
// halos that each workgroup stages for itself cost more than the tile kernels'
// unfilled chip. The lines lie where a CU takes another workgroup: 24,576, 32,768
// and 40,960 nodes are three to five of 32 nodes a CU, 81,920 and 98,304 five and
// six of 64. Work grows by chunks of six slots, the halo not at all with K, so short
// stencils return to the tile kernels earlier, and own-node stencils earlier still,
// whose tile kernels have smaller halos. us a step, one / two / tile kernels (of the
// FP32 ones the fastest variant), paper stencils:
//   FP32    16,384             28,900             36,481              48,841
//   K 6     4.3 / 4.2 / 4.9    5.4 / 4.8 / 5.0    6.7 / 5.5 / 5.1     7.4 / 5.6 / 5.2
//   K 10    4.7 / 4.7 / 5.6    6.0 / 5.7 / 5.7    7.4 / 6.8 / 5.8     8.2 / 6.9 / 5.9
//   K 12    4.7 / 4.8 / 5.8    6.1 / 5.8 / 6.0    7.4 / 6.8 / 6.1     8.6 / 7.1 / 7.0
//   K 13    5.1 / 5.3 / 6.1    6.7 / 6.7 / 6.2    8.0 / 7.8 / 6.4     9.5 / 8.2 / 7.7
//   K 15    5.1 / 5.3 / 6.3    6.7 / 6.7 / 6.8    8.0 / 7.9 / 7.1     10.0 / 8.4 / 9.1
//   K 17    5.2 / 5.4 / 6.9    6.7 / 6.8 / 8.3    8.5 / 8.1 / 9.0     10.4 / 8.7 / 10.8
//   K 25    6.2 / 7.5 / 7.9    8.5 / 9.0 / 12.9   10.7 / 11.1 / 13.7  13.5 / 13.1 / 14.8
//   FP64    8,100              65,536             84,100              98,596
//   K 6     4.3 / 4.3 / 7.7    13 / 10.4 / 13.0   17 / 14.7 / 14.8    19 / 16.7 / 15.4
//   K 8     4.6 / 4.8 / 8.5    15 / 13.2 / 15.7   19 / 17.5 / 17.7    22 / 19.4 / 18.5
//   K 12    4.8 / 5.0 / 10.4   17 / 15.1 / 20.6   21 / 19.5 / 24.6    23 / 21.5 / 25.7
//   K 30    6.0 / 6.8 / 21     27 / 26 / 44       33 / 33 / 47        37 / 36 / 49
//   K 48    8.3 / 9.9 / 47     40 / 40 / 65       57 / 59 / 72        76 / 75 / 75
// Own-node stencils, FP32 at 28,900 nodes: K 6 4.4 / 4.7 / 4.7, K 13 5.9 / 6.1 / 5.8,
// K 15 5.9 / 6.1 / 6.1; FP64, two / tile kernels: K 8 at 65,536 nodes 12.9 / 14.2 and at
// 68,644 16.2 / 15.3, K 9 at 78,961 16.6 / 17.2 and at 84,100 18.7 / 17.4, K 12 at
// 96,100 20.7 / 22.2 and at 98,596 23.0 / 22.2.
inline int wide_dirs(int64_t n, int K, int mode, int precision) {
    const bool own = mode == MLBM_STENCIL_OWN;
    if (precision == MLBM_FP64) {
        if (n <= 8192) return 1;
        const int most = own ? (K <= 8 ? 65536 : K <= 9 ? 81920 : K <= 14 ? 98304 : 102400)
                             : (K <= 7 ? 81920 : K <= 9 ? 98304 : 102400);
        return n <= (K > 45 ? 98304 : most) ? 2 : 0;
    }
    if (K <= 6) {
        if (n <= (own ? 32768 : 8192)) return 1;
        return n <= 32768 && !own ? 2 : 0;
    }
    if (n <= 24576) return 1;
    if (n <= 32768) return K >= 15 || (own && K >= 13) ? 1 : K == 11 || K == 12 ? 2 : 0;
    if (n <= 40960) return K >= 22 ? 1 : K >= 17 ? 2 : 0;
    return n <= 49152 && K >= 15 ? 2 : 0;
}

template <int MODE, int D>
void launch_wide_batch(const mlbm_plan &plan, const void *gin, void *gout, hipStream_t s) {
    const int64_t nb = plan.total_tiles * (kTile / (32 * D));
    int nh = 0;
    for (const CloudPlan &cp : plan.c) nh = std::max(nh, cp.nh_max);
    nh = wide_halo<float>(nh);
    hipLaunchKernelGGL((k_step_wide_batch<MODE, D>), dim3(xcd_grid(nb)), dim3(256),
                       wide_lds<float>(nh, 32 * D), s, plan.descs, plan.tile2cloud,
                       (const float *)gin, (float *)gout, nb, nh,
                       wide_direct(plan.total_tiles * kTile));
}

// Small batches take the small-cloud kernel by their nodes, counted in whole tiles, and
// shortest stencils, whatever the variant: one direction a lane up to 24,576 nodes,
// then two. us a step, this / best tile kernel: paper stencils of K 6 at 30,720 nodes
// (eight clouds) 4.8 / 5.1, K 10 5.7 / 5.9, K 12 5.8 / 6.3, K 15 6.6 / 6.8; K 12 at 36,864
// (sixteen) 6.8 / 6.3 and K 15 7.9 / 6.8; K 20 there 9.5 / 8.8, but 9.8 / 11.2 at 40,960
// (four) and 10.6 / 13.1 at 49,152. K 20 to 30, 2 clouds of 3,232 nodes together 5.1 /
// 9.5, 8 of 15,247 6.6 / 9.7, 4 of 38,054 12.9 / 16.7; 8 of 76,924 nodes stay with the
// tile kernels (18.5).
int wide_dirs_batch(const mlbm_plan &plan) {
    int K = kMaxK;
    for (const CloudPlan &cp : plan.c) K = std::min(K, cp.K);
    const int64_t n = plan.total_tiles * kTile;
    if (n <= 24576) return 1;
    return n <= (K < 18 ? 32768 : 49152) ? 2 : 0;
}

template <int MODE>
void launch32_batch_v(const mlbm_plan &plan, const void *gin, void *gout, hipStream_t s) {
    if (const int dirs = wide_dirs_batch(plan)) {
        if (dirs == 1) launch_wide_batch<MODE, 1>(plan, gin, gout, s);
        else launch_wide_batch<MODE, 2>(plan, gin, gout, s);
        return;
    }
    switch (plan.c[0].variant) {
        case 1: launch32_batch<MODE, 1, true>(plan, gin, gout, s); break;
        case 2: launch32_batch<MODE, 2, false>(plan, gin, gout, s); break;
        case 3: launch32_batch<MODE, 2, true>(plan, gin, gout, s); break;
        case 4: launch32_batch<MODE, 3, false>(plan, gin, gout, s); break;
        case 5: launch32_batch<MODE, 3, true>(plan, gin, gout, s); break;
        case 6: launch32s_batch<MODE, false>(plan, gin, gout, s); break;
        case 7: launch32s_batch<MODE, true>(plan, gin, gout, s); break;
        case 8: launch32s_batch<MODE, false, 2>(plan, gin, gout, s); break;
        case 9: launch32s_batch<MODE, true, 2>(plan, gin, gout, s); break;
        default: launch32_batch<MODE, 1, false>(plan, gin, gout, s); break;
    }
}

template <int MODE, bool FORCE, int WALL, bool REC>
hipError_t step_variant(const CloudPlan &cp, int precision, const void *gin, void *gout,
                        void *frec, hipStream_t s) {
    const int n = cp.n;
    const int64_t nblocks = (n + kTile - 1) / kTile;
    if (const int dirs = wide_dirs(n, cp.K, MODE, precision)) {
        if (precision == MLBM_FP64)
            launch_wide<double, MODE, FORCE, WALL, REC>(cp, dirs, gin, gout, frec, s);
        else
            launch_wide<float, MODE, FORCE, WALL, REC>(cp, dirs, gin, gout, frec, s);
        return hipGetLastError();
    }
    if (precision == MLBM_FP64) {
        hipLaunchKernelGGL((k_step64<MODE, FORCE, WALL, REC>), dim3(xcd_grid(nblocks)),
                           dim3(kTile), cp.lds_bytes, s, n, cp.K, nblocks, (const double *)gin,
                           (double *)gout, cp.W64, cp.nbr, cp.owner, cp.force64,
                           cp.prm.wall_kind == 2 ? cp.links : cp.ntype,
                           1.0 / cp.prm.tau, cp.prm.rho_wall, (double *)frec,
                           cp.lds_bytes ? cp.tdesc : nullptr, cp.ownerL, cp.nbrL, cp.hlist,
                           cp.ocap, cp.hcap, cp.err, cp.perm, (int)cp.off);
    } else {
        launch32_tuned<MODE, FORCE, WALL, REC>(cp, gin, gout, frec, nblocks, s);
    }
    return hipGetLastError();
}

template <int MODE, bool FORCE, int WALL>
hipError_t step_rec(const CloudPlan &cp, int precision, const void *gin, void *gout,
                    void *frec, hipStream_t s) {
    return frec ? step_variant<MODE, FORCE, WALL, true>(cp, precision, gin, gout, frec, s)
                : step_variant<MODE, FORCE, WALL, false>(cp, precision, gin, gout, frec, s);
}

template <int MODE, bool FORCE>
hipError_t step_wall(const CloudPlan &cp, int precision, const void *gin, void *gout,
                     void *frec, hipStream_t s) {
    switch (cp.prm.wall_kind) {
        case 1: return step_rec<MODE, FORCE, 1>(cp, precision, gin, gout, frec, s);
        case 2: return step_rec<MODE, FORCE, 2>(cp, precision, gin, gout, frec, s);
        default: return step_rec<MODE, FORCE, 0>(cp, precision, gin, gout, frec, s);
    }
}

template <int MODE>
hipError_t step_force(const CloudPlan &cp, int precision, const void *gin, void *gout,
                      void *frec, hipStream_t s) {
    return cp.prm.force_kind ? step_wall<MODE, true>(cp, precision, gin, gout, frec, s)
                             : step_wall<MODE, false>(cp, precision, gin, gout, frec, s);
}

// ------------------------------------------------------------------------
// Standard lattice Boltzmann (eq. LBM_streaming): the reference method of the
// paper on a periodic nx x ny lattice, state [9][ny][nx] with x fastest.
// Streaming is a pull by the index shift x - e_k (wrapped), followed by the
// same moments and BGK collision as the fused MLBM step. Workgroups cover 256
// consecutive nodes of a row; the XCD map keeps neighbouring rows, which read
// each other's populations, in one L2.
// ------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(256) void k_lbm_step(int nx, int ny, int64_t nblocks,
                                                  const T *__restrict__ g, T *__restrict__ go,
                                                  double rtau, double rho0) {
    const int64_t b = xcd_tile(nblocks);
    if (b >= nblocks) return;
    const int bx = (nx + 255) / 256;
    const int y = (int)(b / bx);
    const int x = (int)(b - (int64_t)y * bx) * 256 + threadIdx.x;
    if (x >= nx) return;
    const int64_t n = (int64_t)nx * ny;
    const int p = y * nx + x;
    T f[kQ];
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        int sx = x - (int)lat_ex(k), sy = y - (int)lat_ey(k);
        sx = sx < 0 ? sx + nx : (sx >= nx ? sx - nx : sx);
        sy = sy < 0 ? sy + ny : (sy >= ny ? sy - ny : sy);
        f[k] = g[(int64_t)k * n + (int64_t)sy * nx + sx];
    }
    if constexpr (sizeof(T) == 4)
        collide_store32<false, false, false>((int)n, p, f, go, nullptr, nullptr, (float)rtau,
                                             (float)rho0, 0.0f, nullptr, nullptr, nullptr, 0);
    else
        collide_store64<false, false, false>((int)n, p, f, go, nullptr, nullptr, rtau, 0.0,
                                             nullptr, nullptr, nullptr, 0);
}

// One collision with the step's arithmetic, in registers.
__device__ __forceinline__ void lbm_collide(float (&f)[kQ], float (&v)[kQ], float rtau, float rho0) {
    collide_at32<false, 0, false>(1, 0, f, v, 0u, 0.0f, 0.0f, rtau, rho0, 0.0f, nullptr, nullptr,
                                  nullptr, 0);
}
__device__ __forceinline__ void lbm_collide(double (&f)[kQ], double (&v)[kQ], double rtau, double) {
    collide_at64<false, 0, false>(1, 0, f, v, 0u, 0.0, 0.0, rtau, 0.0, nullptr, nullptr, nullptr, 0);
}

// S steps in one pass over memory. A workgroup makes a block of TX x TY nodes:
// the first step pulls from global memory for the block and S - 1 nodes around
// it, the next ones pull from LDS, each for one node less on every side, and
// the last writes the block. Every population is pulled by one node only, so
// LDS needs no copy of the input, and one buffer: the new values wait in
// registers until all have been read. The arithmetic is that of single steps
// and so are the bits.
// A step alone is bound by memory, 72 (FP32) or 144 bytes a node, or on a
// small lattice by its launch and two trips to memory; S steps share those.
// 3 or 4 of them: FP32 2048^2 49.0 -> 26.8 us a step, 1024^2 10.9 -> 8.4, 512^2
// 4.2 -> 3.8, 160^2 2.6 -> 1.6; FP64 115 -> 49.4, 23.2 -> 11.0, 6.6 -> 4.6, 2.9 ->
// 1.7. What bounds them now is the arithmetic of the block and the nodes around
// it, at 512 threads and three workgroups a CU.
template <class T, int TX, int CAP, int NTH, int S>
__global__ __launch_bounds__(NTH) void k_lbm_steps(int nx, int ny, int64_t nblocks,
                                                   const T *__restrict__ g, T *__restrict__ go,
                                                   T rtau, T rho0) {
    constexpr int R = S - 1, W = TX + 2 * R, H = CAP / W, TY = H - 2 * R, N = W * H;
    constexpr int NPT = (N + NTH - 1) / NTH;
    static_assert(TY > 0 && S > 1, "room for the block");
    __shared__ T s[kQ][N];
    const int64_t b = xcd_tile(nblocks);
    if (b >= nblocks) return;
    const int bx = (nx + TX - 1) / TX, by = (int)(b / bx);
    const int x0 = (int)(b - (int64_t)by * bx) * TX - R, y0 = by * TY - R;
    const int tid = threadIdx.x;
    const int64_t n = (int64_t)nx * ny;
    T v[NPT][kQ];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int at = tid + i * NTH;
        if (at < N) {
            // (blocks may reach past the lattice, and around a small one more than once)
            int x = (x0 + at % W) % nx, y = (y0 + at / W) % ny;
            x += x < 0 ? nx : 0;
            y += y < 0 ? ny : 0;
            T f[kQ];
#pragma unroll
            for (int k = 0; k < kQ; ++k) {
                int sx = x - (int)lat_ex(k), sy = y - (int)lat_ey(k);
                sx = sx < 0 ? sx + nx : (sx >= nx ? sx - nx : sx);
                sy = sy < 0 ? sy + ny : (sy >= ny ? sy - ny : sy);
                f[k] = g[(int64_t)k * n + (int64_t)sy * nx + sx];
            }
            lbm_collide(f, v[i], rtau, rho0);
        }
    }
#pragma unroll
    for (int i = 0; i < NPT; ++i)
        if (tid + i * NTH < N) {
#pragma unroll
            for (int k = 0; k < kQ; ++k) s[k][tid + i * NTH] = v[i][k];
        }
    __syncthreads();
#pragma unroll
    for (int m = 1; m < S; ++m) {
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int at = tid + i * NTH, lx = at % W, ly = at / W;
            if (lx >= m && lx < W - m && ly >= m && ly < H - m) {
                T f[kQ];
#pragma unroll
                for (int k = 0; k < kQ; ++k) f[k] = s[k][at - (int)lat_ey(k) * W - (int)lat_ex(k)];
                lbm_collide(f, v[i], rtau, rho0);
                if (m == S - 1 && x0 + lx < nx && y0 + ly < ny) {
#pragma unroll
                    for (int k = 0; k < kQ; ++k)
                        go[(int64_t)k * n + (int64_t)(y0 + ly) * nx + (x0 + lx)] = v[i][k];
                }
            }
        }
        if (m < S - 1) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
                const int at = tid + i * NTH, lx = at % W, ly = at / W;
                if (lx >= m && lx < W - m && ly >= m && ly < H - m) {
#pragma unroll
                    for (int k = 0; k < kQ; ++k) s[k][at] = v[i][k];
                }
            }
            __syncthreads();
        }
    }
}

template <class T, int TX, int CAP, int NTH, int S>
void launch_lbm_steps(int nx, int ny, double rtau, double rho0, const void *g, void *go,
                      hipStream_t s) {
    constexpr int TY = CAP / (TX + 2 * (S - 1)) - 2 * (S - 1);
    const int64_t nb = (int64_t)((nx + TX - 1) / TX) * ((ny + TY - 1) / TY);
    hipLaunchKernelGGL((k_lbm_steps<T, TX, CAP, NTH, S>), dim3(xcd_grid(nb)), dim3(NTH), 0, s, nx, ny,
                       nb, (const T *)g, (T *)go, (T)rtau, (T)rho0);
}

// Interpolation alone (Sec. 4, Fig. interp_test): the streaming operator of
// the plan applied to a scalar field, in FP64 with the FP64 shape vectors.
// out[k-1][u] = sum_j W_k[j](p) field[user(nbr[j][owner_k(p)])], u = user(p).
// One thread a departure point, six slots at a time: member, user index and
// value are three loads one after another, which one thread a node went
// through 8 K times in turn (10,201 nodes, K 25: 95 us, 11 now).
__global__ __launch_bounds__(256) void k_interpolate(int n, int K, int mode,
                                                     const double *__restrict__ W64,
                                                     const int32_t *__restrict__ nbr,
                                                     const int32_t *__restrict__ owner,
                                                     const int32_t *__restrict__ perm,
                                                     const double *__restrict__ field,
                                                     int64_t out_stride, double *__restrict__ out) {
    // pairs of directions side by side, as the shape vectors lie: 128 nodes a
    // workgroup and pair
    const int64_t nb = ((int64_t)n + 127) / 128, blk = xcd_tile(nb);
    if (blk >= nb) return;
    const int p = (int)(blk * 128) + (int)(threadIdx.x >> 1);
    const int k = 2 * (int)blockIdx.y + (int)(threadIdx.x & 1) + 1;
    if (p >= n) return;
    const int u = perm[p];
    const int s = mode == MLBM_STENCIL_OWN ? p : owner[(int64_t)(k - 1) * n + p];
    double acc = 0.0;
    constexpr int CH = 6;
    int j = 0;
    for (; j + CH <= K; j += CH) {
        int q[CH];
        double w[CH], v[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            q[i] = nbr[(int64_t)(j + i) * n + s];
            w[i] = W64[w64_at(k, j + i, n, p)];
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) q[i] = perm[q[i]];
#pragma unroll
        for (int i = 0; i < CH; ++i) v[i] = field[q[i]];
#pragma unroll
        for (int i = 0; i < CH; ++i) acc = __builtin_fma(w[i], v[i], acc);
    }
    for (; j < K; ++j)
        acc = __builtin_fma(W64[w64_at(k, j, n, p)], field[perm[nbr[(int64_t)j * n + s]]], acc);
    out[(int64_t)(k - 1) * out_stride + u] = acc;
}

}  // namespace

hipError_t launch_interpolate(const CloudPlan &cp, const double *field, int64_t out_stride,
                              double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_interpolate, dim3(xcd_grid(blocks_for(cp.n, 128)), 4), dim3(256), 0, s, cp.n, cp.K,
                       cp.prm.stencil_mode, cp.W64, cp.nbr, cp.owner, cp.perm, field, out_stride,
                       out);
    return hipGetLastError();
}

// Nodes whose populations carry no body force (so the moments need no
// correction there): the equilibrium wall nodes; with bounce-back, none.
inline const uint8_t *fmask(const CloudPlan &cp) { return cp.has_walls ? cp.ntype : nullptr; }

Step32Args step32_args(const CloudPlan &cp, void *frec) {
    Step32Args a{};
    a.n = cp.n;
    a.K = cp.K;
    a.ocap = cp.ocap;
    a.hcap = cp.hcap;
    a.W = reinterpret_cast<const float4 *>(cp.W32);
    a.nbr = cp.nbr;
    a.owner = cp.owner;
    a.force = cp.force32;
    a.ntype = cp.prm.wall_kind == 2 ? cp.links : cp.ntype;   // link masks for bounce-back
    a.rtau = (float)(1.0 / cp.prm.tau);
    a.rho0 = (float)cp.prm.rho0;
    a.rho0_64 = cp.prm.rho0;
    a.rho_w = (float)cp.prm.rho_wall;
    a.frec = (float *)frec;
    a.tdesc = cp.lds_bytes ? cp.tdesc : nullptr;
    a.lcap = (int)cp.lds_bytes;
    a.ownerL = cp.ownerL;
    a.nbrL = cp.nbrL;
    a.hlist = cp.hlist;
    a.soff = 0;
    a.tile_begin = 0;
    a.err = cp.err;
    a.perm = cp.perm;
    a.uoff = (int)cp.off;
    return a;
}

hipError_t launch_step_batch(const mlbm_plan &plan, const void *gin, void *gout,
                             hipStream_t s) {
    if (plan.batch_mode == MLBM_STENCIL_OWN)
        launch32_batch_v<MLBM_STENCIL_OWN>(plan, gin, gout, s);
    else
        launch32_batch_v<MLBM_STENCIL_PAPER>(plan, gin, gout, s);
    return hipGetLastError();
}

bool step_ignores_variant(const mlbm_plan &plan) {
    if (plan.batched) return wide_dirs_batch(plan) != 0;
    for (const CloudPlan &cp : plan.c)
        if (!wide_dirs(cp.n, cp.K, cp.prm.stencil_mode, plan.precision)) return false;
    return true;
}

hipError_t launch_init_batch(const mlbm_plan &plan, const double *rho, const double *ux,
                             const double *uy, void *g, hipStream_t s) {
    hipLaunchKernelGGL(k_init_batch, dim3((unsigned)plan.total_tiles), dim3(kTile), 0, s, plan.descs,
                       plan.tile2cloud, rho, ux, uy, (float *)g);
    return hipGetLastError();
}

hipError_t launch_moments_batch(const mlbm_plan &plan, const void *g, double *rho, double *ux,
                                double *uy, hipStream_t s) {
    hipLaunchKernelGGL(k_moments_batch, dim3((unsigned)plan.total_tiles), dim3(kTile), 0, s,
                       plan.descs, plan.tile2cloud, (const float *)g, rho, ux, uy);
    return hipGetLastError();
}

hipError_t launch_set_desc(Step32Args *dst, const Step32Args &v, hipStream_t s) {
    hipLaunchKernelGGL(k_set_desc, dim3(1), dim3(1), 0, s, dst, v);
    return hipGetLastError();
}

hipError_t launch_step(const CloudPlan &cp, int precision, const void *gin, void *gout,
                       void *frec, hipStream_t s) {
    return cp.prm.stencil_mode == MLBM_STENCIL_OWN
               ? step_force<MLBM_STENCIL_OWN>(cp, precision, gin, gout, frec, s)
               : step_force<MLBM_STENCIL_PAPER>(cp, precision, gin, gout, frec, s);
}

hipError_t launch_init(const CloudPlan &cp, int precision, const double *rho,
                       const double *ux, const double *uy, void *g, bool collide,
                       hipStream_t s) {
    const int n = cp.n;
    const int wall = cp.has_walls ? 1 : 0;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_init<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, rho, ux, uy, cp.ntype, cp.force64, cp.prm.rho0,
                           cp.prm.rho_wall, wall, 0, collide ? 1 : 0, (double *)g);
    else
        hipLaunchKernelGGL(k_init<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, rho, ux, uy, cp.ntype, cp.force64, cp.prm.rho0,
                           cp.prm.rho_wall, wall, 1, collide ? 1 : 0, (float *)g);
    return hipGetLastError();
}

hipError_t launch_moments(const CloudPlan &cp, int precision, const void *g, double *rho,
                          double *ux, double *uy, bool post_collision, hipStream_t s) {
    const int n = cp.n;
    const float *f32 = post_collision && precision != MLBM_FP64 ? cp.force32 : nullptr;
    const double *f64 = post_collision && precision == MLBM_FP64 ? cp.force64 : nullptr;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_moments<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, (const double *)g, f32, f64, fmask(cp), cp.prm.rho0, 0, rho,
                           ux, uy, cp.err, (int)cp.off);
    else
        hipLaunchKernelGGL(k_moments<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, (const float *)g, f32, f64, fmask(cp), cp.prm.rho0, 1, rho,
                           ux, uy, cp.err, (int)cp.off);
    return hipGetLastError();
}

hipError_t launch_l2(const CloudPlan &cp, int precision, const void *g, const double *uxt,
                     const double *uyt, double *out, double *part, hipStream_t s) {
    const int n = cp.n;
    const int64_t nb = blocks_for(n, 256);
    const float *f32 = precision != MLBM_FP64 ? cp.force32 : nullptr;
    const double *f64 = precision == MLBM_FP64 ? cp.force64 : nullptr;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_l2_partial<double>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const double *)g, f32, f64, fmask(cp), cp.prm.rho0, 0, uxt, uyt, part,
                           cp.err, (int)cp.off);
    else
        hipLaunchKernelGGL(k_l2_partial<float>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const float *)g, f32, f64, fmask(cp), cp.prm.rho0, 1, uxt, uyt, part,
                           cp.err, (int)cp.off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_l2_final, dim3(1), dim3(256), 0, s, nb, (const double *)part, out);
    return hipGetLastError();
}

hipError_t launch_residual(const CloudPlan &cp, int precision, const void *g, double *speed,
                           double *out, double *part, hipStream_t s) {
    const int n = cp.n;
    const int64_t nb = blocks_for(n, 256);
    const float *f32 = precision != MLBM_FP64 ? cp.force32 : nullptr;
    const double *f64 = precision == MLBM_FP64 ? cp.force64 : nullptr;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_residual_partial<double>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const double *)g, f32, f64, fmask(cp), cp.prm.rho0, 0, speed, part,
                           cp.err, (int)cp.off);
    else
        hipLaunchKernelGGL(k_residual_partial<float>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const float *)g, f32, f64, fmask(cp), cp.prm.rho0, 1, speed, part,
                           cp.err, (int)cp.off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_l2_final, dim3(1), dim3(256), 0, s, nb, (const double *)part, out);
    return hipGetLastError();
}

hipError_t launch_collide(const CloudPlan &cp, int precision, const void *f, void *g,
                          hipStream_t s) {
    const int n = cp.n;
    const int wall = cp.has_walls ? 1 : 0;
    const double *force = cp.prm.force_kind ? cp.force64 : nullptr;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_collide<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const double *)f, (double *)g, force, cp.ntype, wall,
                           1.0 / cp.prm.tau, cp.prm.rho0, cp.prm.rho_wall, 0);
    else
        hipLaunchKernelGGL(k_collide<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const float *)f, (float *)g, force, cp.ntype, wall,
                           1.0 / cp.prm.tau, cp.prm.rho0, cp.prm.rho_wall, 1);
    return hipGetLastError();
}

hipError_t launch_l2_final(const double *part, int64_t nparts, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_l2_final, dim3(1), dim3(256), 0, s, nparts, part, out);
    return hipGetLastError();
}

// Launches of several steps: small blocks of at most 512 nodes, one a thread, or, in
// FP32, large ones that fill a third of a CU's LDS.
struct LbmBlock {
    int tx, cap;
};
constexpr LbmBlock kLbmSmall{32, 512}, kLbmLarge{64, 1456};

// Time of a launch of `steps` steps, us, from its shape: a fixed part, and a part per
// node that the busiest CU computes (whole blocks, the nodes around them with
// them), fitted to lattices of 256 to 4,194,304 nodes, square and thin; most lie within
// 10 %. A block of steps that its lattice does not fill, or a last CU round that
// is nearly empty, can cost more than the passes over memory that it saves, so
// neither the size alone nor the number of steps decides. us a step, single
// steps, 2, 3 and 4 in a launch:
//   FP64 2048x65 4.5, 3.9 3.2 3.5; 512^2 6.6, 4.9 4.6 4.5; 2048^2 115, 64 50 49
//   FP32 2048x65 3.5, small blocks 3.1 2.6 3.0, large 4.0 3.4 2.9
//   FP32 512^2 4.2, small 4.0 3.8 4.0, large 4.0 3.4 4.0
//   FP32 1024^2 10.9, small 9.5 9.4 11.3, large 10.0 8.4 8.2; 2048^2 49, large 36 29 27
double lbm_launch_us(int nx, int ny, int precision, int steps, const LbmBlock &b) {
    const double n = (double)nx * ny;
    const bool f64 = precision == MLBM_FP64;
    if (steps == 1)   // + populations that the caches no longer hold, + workgroups of short rows
        return 2.4 + (f64 ? 16e-6 * n + 11e-6 * std::max(0.0, n - 3e5)
                          : 8e-6 * n + 6e-6 * std::max(0.0, n - 2.1e6)) +
               450e-6 * ((double)ny * ((nx + 255) / 256) - n / 256);
    const int r = steps - 1, w = b.tx + 2 * r, h = b.cap / w, ty = h - 2 * r;
    const int64_t blocks = (int64_t)((nx + b.tx - 1) / b.tx) * ((ny + ty - 1) / ty);
    const double nodes = (double)((blocks + 255) / 256) * w * h;   // of the busiest CU
    constexpr double fixed64[3] = {1.9, 3.0, 3.4}, each64[3] = {4.8e-3, 4.8e-3, 5.3e-3};
    constexpr double far64[3] = {10e-6, 7e-6, 0.0};   // a node that the caches do not hold
    constexpr double fixedS[3] = {2.5, 3.5, 3.4}, eachS[3] = {3.6e-3, 3.9e-3, 4.9e-3};
    constexpr double fixedL[3] = {3.0, 5.1, 5.2}, eachL[3] = {3.4e-3, 3.5e-3, 3.9e-3};
    const int k = steps - 2;
    if (f64) return fixed64[k] + each64[k] * nodes + far64[k] * std::max(0.0, n - 1.2e6);
    return b.tx == kLbmSmall.tx ? fixedS[k] + eachS[k] * nodes : fixedL[k] + eachL[k] * nodes;
}

bool lbm_large(int nx, int ny, int precision, int steps) {
    return precision != MLBM_FP64 && lbm_launch_us(nx, ny, precision, steps, kLbmLarge) <
                                         lbm_launch_us(nx, ny, precision, steps, kLbmSmall);
}

// A number of launches that is even where the number of steps is leaves the result
// in the buffer that single steps leave it in: launches of two and four steps come
// in pairs, those of one and three alone. The cheapest groups for n_steps: the
// cheapest one a step, and the best mix for what is left. Without a graph a launch
// of a few microseconds waits for the host (185x331, 16 steps with initial state and
// moments: 62 us with four launches, 66 with six that take less time themselves). A
// single step between others finds some of its populations in other XCDs' caches (1.15: with 1, mixes
// with single steps that measured 4 % slower were taken, 1115x1352 FP32 18 steps 284
// us for 271), and on flat lattices (fewer rows of blocks than XCDs) most of them,
// and leaves its own there, about 22 ns per 1,000 nodes in FP32 (16384x17, three
// steps and one: 15 us expected, 21).
LbmSteps lbm_steps(int nx, int ny, int precision, int32_t n_steps, bool captured) {
    const double host_us = captured ? 0.0 : 2.0;
    double us[5], cost[kLbmGroups];
    for (int k = 1; k < 5; ++k)
        us[k] = host_us +
                lbm_launch_us(nx, ny, precision, k, lbm_large(nx, ny, precision, k) ? kLbmLarge : kLbmSmall);
    // (FP64: four steps lose to three where rows of blocks do not start on whole lines,
    // 1986x897 26 us a step for 24, and win little elsewhere)
    if (precision == MLBM_FP64 && (int64_t)nx * ny > 300000) us[4] *= 1.06;
    auto steps = [](int u) { return kLbmGroup[u][0] + kLbmGroup[u][1]; };
    int bulk = 0;
    for (int u = 0; u < kLbmGroups; ++u) {
        cost[u] = us[kLbmGroup[u][0]] + (kLbmGroup[u][1] ? us[kLbmGroup[u][1]] : 0.0);
        if (u == 0) cost[u] *= 1.15;
        if (u == 0 && ny < 112) cost[u] += (precision == MLBM_FP64 ? 44e-6 : 22e-6) * std::min(3e5, (double)nx * ny);
        if (cost[u] / steps(u) < cost[bulk] / steps(bulk)) bulk = u;
    }
    constexpr int REST = 24;
    LbmSteps out{};
    if (n_steps >= REST) out.count[bulk] = (n_steps - REST) / steps(bulk) + 1;
    int left = n_steps - out.count[bulk] * steps(bulk);   // < REST
    double best[REST] = {};
    int last[REST] = {};
    for (int t = 1; t <= left; ++t) {
        best[t] = 1e300;
        for (int u = 0; u < kLbmGroups; ++u)
            if (steps(u) <= t && best[t - steps(u)] + cost[u] < best[t]) {
                best[t] = best[t - steps(u)] + cost[u];
                last[t] = u;
            }
    }
    const double total = best[left] + out.count[bulk] * cost[bulk];
    for (; left > 0; left -= steps(last[left])) ++out.count[last[left]];
    if (n_steps * us[1] <= total) out = LbmSteps{{n_steps}};
    return out;
}

template <class T, int TX, int CAP, int NTH>
void launch_lbm_fused(int nx, int ny, double rtau, double rho0, int steps, const void *g, void *go,
                      hipStream_t s) {
    if (steps == 2) launch_lbm_steps<T, TX, CAP, NTH, 2>(nx, ny, rtau, rho0, g, go, s);
    else if (steps == 3) launch_lbm_steps<T, TX, CAP, NTH, 3>(nx, ny, rtau, rho0, g, go, s);
    else launch_lbm_steps<T, TX, CAP, NTH, 4>(nx, ny, rtau, rho0, g, go, s);
}

hipError_t launch_lbm_step(int nx, int ny, int precision, double tau, double rho0, int steps,
                           const void *g, void *go, hipStream_t s) {
    const double rtau = 1.0 / tau;
    if (steps == 1) {
        const int64_t nblocks = (int64_t)ny * ((nx + 255) / 256);
        if (precision == MLBM_FP64)
            hipLaunchKernelGGL(k_lbm_step<double>, dim3(xcd_grid(nblocks)), dim3(256), 0, s, nx, ny,
                               nblocks, (const double *)g, (double *)go, rtau, rho0);
        else
            hipLaunchKernelGGL(k_lbm_step<float>, dim3(xcd_grid(nblocks)), dim3(256), 0, s, nx, ny,
                               nblocks, (const float *)g, (float *)go, rtau, rho0);
        return hipGetLastError();
    }
    if (precision == MLBM_FP64)
        launch_lbm_fused<double, kLbmSmall.tx, kLbmSmall.cap, 512>(nx, ny, rtau, rho0, steps, g, go, s);
    else if (lbm_large(nx, ny, precision, steps))
        launch_lbm_fused<float, kLbmLarge.tx, kLbmLarge.cap, 512>(nx, ny, rtau, rho0, steps, g, go, s);
    else
        launch_lbm_fused<float, kLbmSmall.tx, kLbmSmall.cap, 512>(nx, ny, rtau, rho0, steps, g, go, s);
    return hipGetLastError();
}

hipError_t launch_lbm_init(int n, int precision, double rho0, const double *rho, const double *ux,
                           const double *uy, void *g, hipStream_t s) {
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_init<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const int32_t *)nullptr, rho, ux, uy, (const uint8_t *)nullptr,
                           (const double *)nullptr, rho0, rho0, 0, 0, 0, (double *)g);
    else
        hipLaunchKernelGGL(k_init<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const int32_t *)nullptr, rho, ux, uy, (const uint8_t *)nullptr,
                           (const double *)nullptr, rho0, rho0, 0, 1, 0, (float *)g);
    return hipGetLastError();
}

hipError_t launch_lbm_moments(int n, int precision, double rho0, const void *g, double *rho,
                              double *ux, double *uy, hipStream_t s) {
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_moments<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const int32_t *)nullptr, (const double *)g, (const float *)nullptr,
                           (const double *)nullptr, (const uint8_t *)nullptr, rho0, 0, rho, ux,
                           uy, (int32_t *)nullptr, 0);
    else
        hipLaunchKernelGGL(k_moments<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           (const int32_t *)nullptr, (const float *)g, (const float *)nullptr,
                           (const double *)nullptr, (const uint8_t *)nullptr, rho0, 1, rho, ux,
                           uy, (int32_t *)nullptr, 0);
    return hipGetLastError();
}

}  // namespace mlbm
