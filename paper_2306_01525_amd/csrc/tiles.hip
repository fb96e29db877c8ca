// Tile-local gather tables for the LDS-staged step kernel.
//
// The step kernel processes tiles of kTile consecutive nodes (Hilbert order,
// so a tile is a compact patch). For tile t it needs the post-collision
// populations of every stencil member of every owner used by the tile's
// departure points. This kernel (one workgroup per tile) computes
//   O_t: the sorted set of owners {owner_k(p) : p in tile, k = 1..8}
//        (the tile's own nodes in own-stencil mode),
//   H_t: the sorted set of stencil members {nbr[j][o] : o in O_t, j < K},
// and stores, with indices local to the tile,
//   ownerL[k][p]   = position of owner_k(p) in O_t (16 bit, paper mode),
//   nbrL[t][o][w]  = positions of nbr[j][O_t[o]] in H_t for j = 3w, 3w+1, 3w+2,
//                    packed as three 10-bit fields of one word (|H_t| <= 1024),
//   hlist[t][h]    = global index of H_t[h],
//   tdesc[t]       = (|O_t|, |H_t|), |H_t| = 0 marks a tile that does not fit
//                    the caps and is stepped with global gathers instead.
// Both sets are collected and numbered in LDS (IndexSet), one after the other
// in the same memory; ownerL is written between them. The stencil rows are read
// with consecutive lanes on consecutive owners, which are consecutive nodes as
// a rule, kLoads entries of a thread in flight at a time.
#include "index_set.h"

namespace mlbm {
namespace {

constexpr int kOCand = 8 * kTile;   // owner candidates per tile
constexpr int kThreads = 1024;
constexpr int kLoads = 6;
static_assert(kOCand <= IndexSet::kWords, "every owner candidate can be a word of its own");

// Bound by its chain of passes on small clouds and by LDS operations on large
// ones. With the sets sorted by bitonic networks and the rows read member by
// member, 10,201 nodes (40 tiles, K = 25) took 57 us and 262,144 (1,024 tiles,
// K = 30) 170 us; now 16 and 54.
__global__ __launch_bounds__(kThreads) void k_tiles(int n, int K, int mode,
                                                    const int32_t *__restrict__ nbr,
                                                    const int32_t *__restrict__ owner, int ocap,
                                                    int hcap, int32_t *__restrict__ tdesc,
                                                    uint16_t *__restrict__ ownerL,
                                                    uint32_t *__restrict__ nbrL,
                                                    int32_t *__restrict__ hlist,
                                                    int32_t *__restrict__ stats) {
    __shared__ IndexSet set;
    __shared__ int32_t oset[kOCand];
    const int64_t ntiles = ((int64_t)n + kTile - 1) / kTile, tt = xcd_tile(ntiles);
    if (tt >= ntiles) return;   // uniform
    const int t = (int)tt;
    const int base = t * kTile;
    const int cnt = min(kTile, n - base);
    const int tid = threadIdx.x;

    // ---- O_t --------------------------------------------------------------
    int no = cnt;
    set.clear();
    __syncthreads();
    if (mode == MLBM_STENCIL_OWN) {
        for (int i = tid; i < cnt; i += kThreads) oset[i] = base + i;
    } else {
        constexpr int kOwn = kOCand / kThreads;   // candidates per thread
        const int l = tid & (kTile - 1);
        int32_t q[kOwn];
#pragma unroll
        for (int c = 0; c < kOwn; ++c) {
            const int64_t k = tid / kTile + c * (kThreads / kTile);
            q[c] = l < cnt ? owner[k * n + base + l] : 0;
        }
#pragma unroll
        for (int c = 0; c < kOwn; ++c)
            if (l < cnt) set.add(q[c]);
        __syncthreads();
        set.count();
        set.order(oset);
        no = set.members;
        __syncthreads();
        if (no <= ocap) {
#pragma unroll
            for (int c = 0; c < kOwn; ++c) {
                const int64_t k = tid / kTile + c * (kThreads / kTile);
                if (l < cnt) ownerL[k * n + base + l] = (uint16_t)set.find(q[c]);
            }
        }
        __syncthreads();
        set.clear();
    }
    __syncthreads();

    // ---- H_t --------------------------------------------------------------
    bool fits = no <= ocap;   // uniform
    if (fits) {
        const int total = no * K;
        for (int e0 = tid; e0 < total; e0 += kLoads * kThreads) {
            int32_t q[kLoads];
#pragma unroll
            for (int c = 0; c < kLoads; ++c) {
                const int e = min(e0 + c * kThreads, total - 1);
                const int j = e / no;
                q[c] = nbr[(int64_t)j * n + oset[e - j * no]];
            }
#pragma unroll
            for (int c = 0; c < kLoads; ++c)
                if (e0 + c * kThreads < total) set.add(q[c]);
        }
    }
    __syncthreads();
    set.count();
    const int nh = set.members;
    fits = fits && !set.over && nh <= hcap;
    if (fits) {
        set.order(hlist + (int64_t)t * hcap);
        __syncthreads();
        const int Kw = (K + 2) / 3;
        uint32_t *nl = nbrL + (int64_t)t * ocap * Kw;
        for (int e = tid; e < no * Kw; e += kThreads) {
            const int w = e / no, o = e - w * no;
            int32_t q[3];
#pragma unroll
            for (int sft = 0; sft < 3; ++sft)
                q[sft] = nbr[(int64_t)min(3 * w + sft, K - 1) * n + oset[o]];
            uint32_t word = 0;
#pragma unroll
            for (int sft = 0; sft < 3; ++sft)
                if (3 * w + sft < K) word |= (uint32_t)set.find(q[sft]) << (10 * sft);
            nl[(int64_t)o * Kw + w] = word;
        }
    }
    if (tid == 0) {
        tdesc[2 * t] = no;
        tdesc[2 * t + 1] = fits ? nh : 0;
        if (fits) {
            // LDS bytes of this tile in the step kernel: 8 directions x nh
            // populations (float) + no x ceil(K/3) index words
            atomicMax(&stats[0], 8 * nh * 4 + no * ((K + 2) / 3) * 4);
            atomicMax(&stats[4], nh);
        } else {
            atomicAdd(&stats[1], 1);
        }
    }
}

}  // namespace

hipError_t launch_tiles(const CloudPlan &cp, int32_t *stats, hipStream_t s) {
    const int ntiles = (cp.n + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_tiles, dim3(xcd_grid(ntiles)), dim3(kThreads), 0, s, cp.n, cp.K, cp.prm.stencil_mode,
                       cp.nbr, cp.owner, cp.ocap, cp.hcap, cp.tdesc, cp.ownerL, cp.nbrL,
                       cp.hlist, stats);
    return hipGetLastError();
}

}  // namespace mlbm
