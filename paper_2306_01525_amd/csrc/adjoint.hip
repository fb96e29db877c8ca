// Discrete adjoint of the MLBM time loop on gfx950 (periodic, no walls, no
// force). The forward step is f^{n+1} = S(C(f^n)): C the BGK collision
// (eqs. LBM_collision, feq), S the semi-Lagrangian streaming through the
// shape vectors (Sec. 2.3). Its adjoint is lam^n = C'(f^n)^T S^T lam^{n+1}.
//
// S^T is applied as a gather, not a scatter: for every direction k and source
// node m, the list of (arriving node i, weight) pairs whose stencil reads m is
// stored as a CSR row sorted by i. Each lane owns one source node and sums its
// row in that fixed order, so the adjoint needs no atomics and is
// deterministic. The weights are the ones the forward step uses (FP32 after
// the partition-of-unity correction, or FP64).
#include <climits>

#include "index_set.h"

namespace mlbm {
namespace {

__device__ __forceinline__ int stencil_owner(const int32_t *owner, int mode, int k, int n,
                                             int i) {
    return mode == MLBM_STENCIL_OWN ? i : owner[(int64_t)(k - 1) * n + i];
}

// Row lengths and fill of the transposed operator. Entries (arriving node i,
// direction k, stencil slot j) are gathered by row (k, source node m) in an
// LDS hash table per tile of arriving nodes, so that a tile adds to a row, or
// claims a run of it, with a single atomic. Keys that find no slot within
// kTrProbe probes (an unusually wide tile) fall back to one atomic per entry;
// k_tr_finish orders every row afterwards.
constexpr int kTrHash = 4096;    // counts: keys of four directions
constexpr int kTrHashF = 1024;   // fill: keys of one direction
constexpr int kTrProbe = 32;
constexpr int kTrCs = 4;         // threads a node in the counts
constexpr uint32_t kTrEmpty = 0xFFFFFFFFu;

template <int HS = kTrHash>
__device__ __forceinline__ int tr_slot(uint32_t *hkey, uint32_t key, bool insert) {
    static_assert((HS & (HS - 1)) == 0, "power of two");
    const uint32_t h = (key * 2654435761u) >> (32 - __builtin_ctz(HS));
    for (int p = 0; p < kTrProbe; ++p) {
        const int sl = (int)((h + p) & (HS - 1));
        const uint32_t cur = hkey[sl];
        if (cur == key) return sl;
        if (cur == kTrEmpty) {
            if (!insert) return -1;
            const uint32_t prev = atomicCAS(&hkey[sl], kTrEmpty, key);
            if (prev == kTrEmpty || prev == key) return sl;
        }
    }
    return -1;
}

// Counts of one thread's entries, stencil slots j0, j0 + step, ... of node i, per
// key in hcnt; entries without a slot add to cnt_direct[row] directly.
__device__ __forceinline__ void tr_count_node(int n, int K, int mode, int h, int i, int j0, int step,
                                              const int32_t *nbr, const int32_t *owner,
                                              uint32_t *hkey, int32_t *hcnt,
                                              int32_t *cnt_direct) {
    if (i >= n) return;
    int s[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s[kk] = stencil_owner(owner, mode, 4 * h + kk + 1, n, i);
#pragma unroll 2
    for (int j = j0; j < K; j += step) {
        int m[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) m[kk] = nbr[(int64_t)j * n + s[kk]];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int sl = tr_slot(hkey, (uint32_t)(kk * n + m[kk]), true);
            if (sl >= 0)
                atomicAdd(&hcnt[sl], 1);
            else
                atomicAdd(&cnt_direct[(int64_t)(4 * h + kk) * n + m[kk]], 1);
        }
    }
}

__device__ __forceinline__ void tr_hash_clear(uint32_t *hkey, int32_t *hcnt) {
    for (int t = threadIdx.x; t < kTrHash; t += blockDim.x) {
        hkey[t] = kTrEmpty;
        hcnt[t] = 0;
    }
}

__device__ __forceinline__ int64_t tr_key_row(uint32_t key, int n, int h) {
    const int kk = (int)(key / (uint32_t)n), m = (int)(key - (uint32_t)kk * n);
    return (int64_t)(4 * h + kk) * n + m;
}

// Counts: a workgroup per tile of 256 arriving nodes and half of the
// directions (1-4 or 5-8), keys (k - 1 - 4 h) n + m. Four threads a node, on
// alternate stencil slots: the entries of a thread wait for memory and for the
// hash table one after another (K 30: 10,201 nodes, one thread a node, 78 us, now
// 23; 262,144 nodes 312 and 216).
__global__ __launch_bounds__(kTrCs * 256) void k_tr_count(int n, int K, int mode,
                                                  const int32_t *__restrict__ nbr,
                                                  const int32_t *__restrict__ owner,
                                                  int32_t *__restrict__ cnt) {
    __shared__ uint32_t hkey[kTrHash];
    __shared__ int32_t hcnt[kTrHash];
    const int64_t nt = ((int64_t)n + 255) / 256, t = xcd_tile(nt);
    if (t >= nt) return;   // uniform
    const int h = blockIdx.y, i = (int)(t * 256) + (int)(threadIdx.x & 255);
    tr_hash_clear(hkey, hcnt);
    __syncthreads();
    tr_count_node(n, K, mode, h, i, threadIdx.x >> 8, kTrCs, nbr, owner, hkey, hcnt, cnt);
    __syncthreads();
    for (int t = threadIdx.x; t < kTrHash; t += blockDim.x)
        if (hkey[t] != kTrEmpty) atomicAdd(&cnt[tr_key_row(hkey[t], n, h)], hcnt[t]);
}

// Fill: a workgroup of kTrJs TT threads takes a tile of TT arriving nodes
// (kTrJs threads a node, each on every kTrJs-th stencil slot: the LDS the
// tile needs leaves room for few workgroups, so each brings many wavefronts)
// and a half of the directions, one direction after another. For each it counts the
// tile's entries per row, claims one run of each row, gathers the entries in
// LDS run by run with their places, and then writes the runs out with
// consecutive lanes on consecutive places. The LDS holds TT K entries (the
// host picks TT so that they fit).
constexpr int kTrJs = 4;
template <class T, int TT>
__global__ __launch_bounds__(kTrJs * TT) void k_tr_fill(int n, int K, int mode,
                                                const int32_t *__restrict__ nbr,
                                                const int32_t *__restrict__ owner,
                                                const float *__restrict__ W32,
                                                const double *__restrict__ W64,
                                                const int32_t *__restrict__ ptr,
                                                int32_t *__restrict__ cur,
                                                int32_t *__restrict__ col, T *__restrict__ val) {
    extern __shared__ __align__(16) unsigned char s_stage[];
    __shared__ uint32_t hkey[kTrHashF];
    __shared__ int32_t hcnt[kTrHashF];
    __shared__ int32_t hbase[kTrHashF];
    __shared__ int32_t hloc[kTrHashF];
    constexpr int NT = kTrJs * TT;
    __shared__ int32_t s_part[NT];
    constexpr int SPT = kTrHashF / NT;   // hash slots per thread in the scan
    static_assert(kTrHashF % NT == 0, "whole slots per thread");
    const int64_t nt = ((int64_t)n + TT - 1) / TT, t = xcd_tile(nt);
    if (t >= nt) return;   // uniform
    const int h = blockIdx.y, tid = threadIdx.x;
    const int i = (int)(t * TT) + tid % TT, j0 = tid / TT;
    const size_t words = ((size_t)TT * K * sizeof(int32_t) + 15) & ~size_t(15);
    int32_t *scol = reinterpret_cast<int32_t *>(s_stage);
    int32_t *spos = reinterpret_cast<int32_t *>(s_stage + words);
    T *sval = reinterpret_cast<T *>(s_stage + 2 * words);
    for (int kk = 0; kk < 4; ++kk) {
        const int k = 4 * h + kk + 1;
        for (int q = tid; q < kTrHashF; q += NT) {
            hkey[q] = kTrEmpty;
            hcnt[q] = 0;
        }
        __syncthreads();
        const int s = i < n ? stencil_owner(owner, mode, k, n, i) : 0;
        if (i < n) {
            for (int j = j0; j < K; j += kTrJs) {
                const int sl = tr_slot<kTrHashF>(hkey, (uint32_t)nbr[(int64_t)j * n + s], true);
                if (sl >= 0) atomicAdd(&hcnt[sl], 1);
            }
        }
        __syncthreads();
        // local run starts in slot order (exclusive scan), the rows' runs
        int mine = 0;
#pragma unroll
        for (int q = 0; q < SPT; ++q) mine += hcnt[tid * SPT + q];
        s_part[tid] = mine;
        __syncthreads();
        for (int w = 1; w < NT; w <<= 1) {
            const int add = tid >= w ? s_part[tid - w] : 0;
            __syncthreads();
            s_part[tid] += add;
            __syncthreads();
        }
        int run = s_part[tid] - mine;
        const int total = s_part[NT - 1];
#pragma unroll
        for (int q = 0; q < SPT; ++q) {
            const int sl = tid * SPT + q;
            const int c = hcnt[sl];
            hloc[sl] = run;
            run += c;
            if (c > 0) {
                const int64_t row = (int64_t)(k - 1) * n + hkey[sl];
                hbase[sl] = ptr[row] + atomicAdd(&cur[row], c);
            }
            hcnt[sl] = 0;
        }
        __syncthreads();
        if (i < n) {
            for (int j = j0; j < K; j += kTrJs) {
                const int m = nbr[(int64_t)j * n + s];
                const int sl = tr_slot<kTrHashF>(hkey, (uint32_t)m, false);
                const T w = W64 ? (T)W64[w64_at(k, j, n, i)]
                                : (T)W32[(((int64_t)j * 2 + ((k - 1) >> 2)) * n + i) * 4 +
                                         ((k - 1) & 3)];
                if (sl >= 0) {
                    const int r = atomicAdd(&hcnt[sl], 1), q = hloc[sl] + r;
                    scol[q] = i;
                    spos[q] = hbase[sl] + r;
                    sval[q] = w;
                } else {   // no slot: a place of its own
                    const int64_t row = (int64_t)(k - 1) * n + m;
                    const int pos = ptr[row] + atomicAdd(&cur[row], 1);
                    col[pos] = i;
                    val[pos] = w;
                }
            }
        }
        __syncthreads();
        for (int q = tid; q < total; q += NT) {
            const int pos = spos[q];
            col[pos] = scol[q];
            val[pos] = sval[q];
        }
        __syncthreads();
    }
}

__global__ void k_set_i32(int32_t *p, int32_t v) { *p = v; }

// Row heads of the transposed operator, compacted per group of 64 nodes (one
// wavefront, consecutive internal indices). Node m's head length is
//   hd(m) = max over its eight rows of min(row length, lw),
// and slot e of a group holds, in node order, one unit for each node of the
// group with hd > e: the eight rows' entry e (directions 1-4 and 5-8 as two
// 16-byte FP32 vectors, as the forward weights; zero weight and column m past
// a row's end). The group's slots follow one another from unit g * 64 * lw.
// A wavefront walking slots in order finds its units with a ballot: the
// active lanes of slot e are consecutive units, so every load is coalesced,
// and the lines fetched hold only nodes that use them. The 10-bit local
// columns of the inverse halo are compacted the same way over triples of
// slots (a node takes part in triple w when 3w < hd), from unit g * 64 * lw3.
// Number of lanes below this one whose bit is set in the wavefront mask.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Entry k (0..7) of unit r of a block of c units whose first unit is u0. A
// block is stored as two halves, entries 0-3 of its c units and then entries
// 4-7, so that a wavefront reads each half as one contiguous run.
__device__ __forceinline__ int64_t unit_entry(int64_t u0, int c, int r, int k) {
    return u0 * 8 + (int64_t)((k >> 2) * c + r) * 4 + (k & 3);
}

constexpr int kEllMaxLw = kMaxK + 4;
constexpr int kFinRows = 16;    // nodes of a workgroup of k_tr_finish
constexpr int kFinLen = 64;     // row entries ranked in LDS; longer rows: sort_long_row
constexpr int kFinPitch = 68;   // their stride (16-byte aligned, rows on other banks)

// Sorts a row by column (no two equal), one wavefront, in place: blocks of 64
// entries are ranked and merged into the sorted part before them, whose entries
// move up by the count of smaller columns in the block, from the end, 64 at a time
// (an entry moves by at most 64 places, so what a turn overwrites has been read).
// blk: 64 words of LDS. Clouds of a few dense clusters, whose edge nodes own most of
// the departure points, have rows of hundreds to thousands of entries: 20,000 nodes
// in eight clusters, rows of up to 2,305, the whole pass 1.9 ms; 1,250 with an
// insertion sort by one lane a row, which k_tr_finish takes sixteen of in turn.
template <class T>
__device__ void sort_long_row(int lane, int len, int32_t *col, T *val, int32_t *blk) {
    for (int done = 0; done < len; done += 64) {
        const bool in = lane < len - done;
        const int32_t c = in ? col[done + lane] : INT_MAX;
        const T v = in ? val[done + lane] : (T)0;
        int rank = 0, lo = 0;
        for (int j = 0; j < 64; ++j) rank += __builtin_amdgcn_readlane(c, j) < c ? 1 : 0;
        if (!in) rank = lane;   // the pads, behind all others
        blk[rank] = c;
        wave_lds_sync();
        if (in) {   // smaller entries of the sorted part
            int hi = done;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (col[mid] < c) lo = mid + 1;
                else hi = mid;
            }
        }
        for (int t = done - 64; t >= 0; t -= 64) {   // (done is a multiple of 64)
            const int32_t e = col[t + lane];
            const T ev = val[t + lane];
            int up = 0, end = 64;
            while (up < end) {
                const int mid = (up + end) >> 1;
                if (blk[mid] < e) up = mid + 1;
                else end = mid;
            }
            if (up > 0) {
                col[t + lane + up] = e;
                val[t + lane + up] = ev;
            }
            if (__ballot(up > 0) == 0) break;   // nothing below moves either
        }
        if (in) {
            col[lo + rank] = c;
            val[lo + rank] = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // read by other lanes next
        wave_lds_sync();
    }
}

// Last pass over the transposed operator: sorts each CSR row by arriving node and
// writes the compacted heads. A workgroup takes 16 nodes of a group and half of
// the directions, one direction a wavefront. Sixteen lanes hold a row; an arriving
// node appears at most once in it (the stencils that the search finds repeat no
// member), so an entry's place is the count of smaller columns, taken from the row
// in LDS four columns a read. SORTED rows come in order, and may hold an arriving
// node more than once (imported stencils may repeat a member): their entries keep
// their places. The sorted heads stay
// in LDS, from where all lanes gather the units, padded with (m, 0) past a row's
// end, as two 16-byte vectors each; consecutive lanes hold consecutive units.
// Four rows a wavefront are ranked while the next four are on their way (without
// that 581 us for the 493 below).
// Sort (by lane exchanges) and heads (each lane walking its own rows in memory) as
// two passes, and now, us, degree 4, K 30: 10,201 nodes FP32 24 + 82, 22; 90,000
// FP64 193 + 432, 243; 262,144 FP32 528 + 592, 493 (1.6 GB, 3.2 TB/s).
template <class T, bool SORTED>
__global__ __launch_bounds__(256) void k_tr_finish(int n, int lw, const int32_t *__restrict__ ptr,
                                                   int32_t *col, T *val, int32_t *__restrict__ ecol,
                                                   T *__restrict__ eval) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint64_t s_mask[kEllMaxLw];   // nodes of the group with a unit in slot e
    __shared__ int s_off[kEllMaxLw];         // units of earlier slots
    __shared__ int s_hd[64];                 // head lengths of the group
    __shared__ int s_row[4][kFinRows + 1];   // row bounds
    typedef T T4 __attribute__((ext_vector_type(4)));
    constexpr int NR = kFinRows, PARTS = 64 / NR, NJ = kFinLen / 16;
    const int S = lw | 1;
    const int64_t parts = ((int64_t)n + 63) / 64 * PARTS, part = xcd_tile(parts);
    if (part >= parts) return;   // uniform
    const int64_t g = part / PARTS;
    const int m0 = (int)(g * 64), r0 = m0 + (int)(part % PARTS) * NR, h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t *unsorted = reinterpret_cast<int32_t *>(smem);               // [4][4][kFinPitch]
    T *hval = reinterpret_cast<T *>(unsorted + 16 * kFinPitch);          // [4][NR][S]
    int32_t *hcol = reinterpret_cast<int32_t *>(hval + 4 * NR * S);      // [4][NR][S]
    if (wv == 0) {
        int hd = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (m0 + lane < n) {
                const int64_t row = (int64_t)k * n + m0 + lane;
                hd = max(hd, min(ptr[row + 1] - ptr[row], lw));
            }
        s_hd[lane] = hd;
        int off = 0;
        for (int e = 0; e < lw; ++e) {
            const uint64_t mask = __ballot(e < hd);
            if (lane == 0) {
                s_mask[e] = mask;
                s_off[e] = off;
            }
            off += __popcll(mask);
        }
    }
    const int64_t krow = (int64_t)(4 * h + wv) * n;
    if (lane <= NR) s_row[wv][lane] = ptr[krow + min(r0 + lane, n)];
    wave_lds_sync();
    int32_t *uc = unsorted + wv * 4 * kFinPitch, *hc = hcol + wv * NR * S;
    T *hv = hval + wv * NR * S;
    const int sub = lane >> 4, p16 = lane & 15;
    // entries of four rows: this lane's, and the longest row of the wavefront's
    auto fetch = [&](int r, int32_t (&c)[NJ], T (&v)[NJ], int &longest) {
        const int b = s_row[wv][r], all = s_row[wv][r + 1] - b, len = all <= kFinLen ? all : 0;
        longest = max(len, __shfl_xor(len, 16));
        longest = __builtin_amdgcn_readfirstlane(max(longest, __shfl_xor(longest, 32)));
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const bool in = 16 * j + p16 < len;
            c[j] = in ? col[b + 16 * j + p16] : INT_MAX;
            v[j] = in ? val[b + 16 * j + p16] : (T)0;
        }
    };
    int32_t c[NJ], cn[NJ] = {};
    T v[NJ], vn[NJ] = {};
    int longest, ln = 0;
    fetch(sub, c, v, longest);
#pragma unroll
    for (int r4 = 0; r4 < NR; r4 += 4) {
        const int r = r4 + sub, b = s_row[wv][r], all = s_row[wv][r + 1] - b;
        const int len = all <= kFinLen ? all : 0;
        if (r4 + 4 < NR) fetch(r + 4, cn, vn, ln);   // in flight under this turn
        int rank[NJ] = {};
        if constexpr (SORTED) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) rank[j] = 16 * j + p16;
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (16 * j < longest) uc[sub * kFinPitch + 16 * j + p16] = c[j];
            wave_lds_sync();
            const int4 *row = reinterpret_cast<const int4 *>(uc + sub * kFinPitch);
            for (int t = 0; 4 * t < longest; ++t) {   // (filled with INT_MAX to a multiple of 16)
                const int4 x = row[t];
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    if (16 * j < longest)
                        rank[j] += (x.x < c[j] ? 1 : 0) + (x.y < c[j] ? 1 : 0) +
                                   (x.z < c[j] ? 1 : 0) + (x.w < c[j] ? 1 : 0);
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (16 * j + p16 < len) {
                if (!SORTED) {
                    col[b + rank[j]] = c[j];
                    val[b + rank[j]] = v[j];
                }
                if (rank[j] < lw) {
                    hc[r * S + rank[j]] = c[j];
                    hv[r * S + rank[j]] = v[j];
                }
            }
        wave_lds_sync();   // the next rows take the place of these
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            c[j] = cn[j];
            v[j] = vn[j];
        }
        longest = ln;
    }
    // rows longer than that: clouds of uneven spacing
    const int mine = s_row[wv][p16 + 1] - s_row[wv][p16];
    if (__ballot(mine > kFinLen) != 0) {
        for (int r = 0; r < NR; ++r) {
            const int b = s_row[wv][r], all = s_row[wv][r + 1] - b;
            if (all <= kFinLen) continue;   // uniform
            if (!SORTED) sort_long_row(lane, all, col + b, val + b, uc);
            for (int e = lane; e < lw; e += 64) {
                hc[r * S + e] = col[b + e];
                hv[r * S + e] = val[b + e];
            }
        }
    }
    __syncthreads();
    const int l = tid % NR, m = r0 + l, bit = m - m0;
    const int hd = s_hd[bit];
    for (int e = tid / NR; e < hd; e += 256 / NR) {
        const uint64_t mask = s_mask[e];
        const int64_t at = unit_entry(g * 64 * lw + s_off[e], __popcll(mask),
                                      __popcll(mask & ((uint64_t(1) << bit) - 1)), 4 * h);
        int cc[4];
        T4 w;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool in = e < s_row[k][l + 1] - s_row[k][l];
            cc[k] = in ? hcol[(k * NR + l) * S + e] : m;
            w[k] = in ? hval[(k * NR + l) * S + e] : (T)0;
        }
        *reinterpret_cast<int4 *>(ecol + at) = make_int4(cc[0], cc[1], cc[2], cc[3]);
        *reinterpret_cast<T4 *>(eval + at) = w;
    }
}

// Workgroup sum of one double per lane (NT lanes), in a fixed order, into
// part[at], or added to it.
template <int NT = 256>
__device__ __forceinline__ void block_sum_to(double v, double *part, int64_t at, bool add = false) {
    __shared__ double sh[NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = add ? part[at] : 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) a += sh[w];
        part[at] = a;
    }
}

__global__ __launch_bounds__(256) void k_sum_final(int64_t nparts, const double *__restrict__ part,
                                                   double *__restrict__ out, int accumulate) {
    __shared__ double sh[256];
    double a = 0.0;
    for (int64_t b = threadIdx.x; b < nparts; b += 256) a += part[b];
    sh[threadIdx.x] = a;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = accumulate ? *out + sh[0] : sh[0];
}

template <class T>
__device__ __forceinline__ void moments_of(const T *f, int n, int p, int dev, double rho0,
                                           T (&fk)[kQ], T &rho, T &ux, T &uy, T &drho) {
    T r = 0, jx = 0, jy = 0;
#pragma unroll
    for (int k = 0; k < kQ; ++k) {
        fk[k] = f[(int64_t)k * n + p];
        r += fk[k];
        jx += fk[k] * (T)lat_ex(k);
        jy += fk[k] * (T)lat_ey(k);
    }
    rho = dev ? (T)rho0 + r : r;
    drho = dev ? r : r - (T)rho0;
    ux = jx / rho;
    uy = jy / rho;
}

// Inverse halo of a tile of source nodes: every arriving node that the head
// (first lw entries) of the transposed rows of the tile's nodes reads, sorted
// (IndexSet), capped at cap. The slot-major columns of those rows are rewritten
// as positions in that set, three 10-bit fields per word: word w of row k of node
// m (compacted like the heads, over triples of slots) holds slots 3w, 3w+1, 3w+2;
// fields past the end of the row are 0. Bound by its chains of waits: with one
// entry at a time a thread and the columns left to a quarter of the wavefronts
// 10,201 nodes (K 30) took 103 us and 262,144 320, now 55 and 268.
__global__ __launch_bounds__(1024) void k_adj_tiles(int n, int lw, int hcap, int cap,
                                                    const int32_t *__restrict__ ptr,
                                                    const int32_t *__restrict__ col,
                                                    const int32_t *__restrict__ ecol,
                                                    int32_t *__restrict__ tdescT,
                                                    int32_t *__restrict__ ilist,
                                                    uint32_t *__restrict__ elocal,
                                                    int32_t *__restrict__ stats) {
    __shared__ IndexSet set;
    const int t = blockIdx.x, tid = threadIdx.x;
    const int base = t * kTile, cnt = min(kTile, n - base);
    const int lw3 = (lw + 2) / 3;
    set.clear();
    __syncthreads();
    // sixteen lanes a row, kRows rows of theirs in flight
    constexpr int kRows = 4, kTeams = 1024 / 16;
    const int p16 = tid & 15;
    for (int w0 = tid >> 4; w0 < 8 * kTile; w0 += kRows * kTeams) {
        int b[kRows], len[kRows];
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int w = w0 + i * kTeams, l = w & (kTile - 1);   // row w / kTile of node l
            b[i] = len[i] = 0;
            if (l < cnt) {
                const int64_t row = (int64_t)(w / kTile) * n + base + l;
                b[i] = ptr[row];
                len[i] = min(ptr[row + 1] - b[i], lw);
            }
        }
        int q[kRows][kEllMaxLw / 16 + 1];
#pragma unroll
        for (int i = 0; i < kRows; ++i)
#pragma unroll
            for (int j = 0; j < kEllMaxLw / 16 + 1; ++j)
                if (16 * j + p16 < len[i]) q[i][j] = col[b[i] + 16 * j + p16];
#pragma unroll
        for (int i = 0; i < kRows; ++i)
#pragma unroll
            for (int j = 0; j < kEllMaxLw / 16 + 1; ++j)
                if (16 * j + p16 < len[i]) set.add(q[i][j]);
    }
    __syncthreads();
    set.count();
    const int ni = set.members;
    const bool fits = !set.over && ni <= cap && cap <= hcap && cap <= 1024;
    if (fits) {
        set.order(ilist + (int64_t)t * hcap);
        __syncthreads();
        // local columns: the columns come from the compacted heads, slot by slot
        // (contiguous over the lanes; the rows themselves would be read with a
        // stride across the lanes, triple after triple). Four wavefronts a group
        // of 64 nodes, one lane a node, each on every fourth triple; the ballots
        // of the others only move its offsets.
        typedef int32_t I4 __attribute__((ext_vector_type(4)));
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        const int wv = tid >> 6, turn = wv >> 2;
        const int m = base + (wv & 3) * 64 + (tid & 63);
        int len[8], hd = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            len[k] = 0;
            if (m < n) {
                const int64_t row = (int64_t)k * n + m;
                len[k] = ptr[row + 1] - ptr[row];
                hd = max(hd, min(len[k], lw));
            }
        }
        const int64_t g0 = (int64_t)(m >> 6) * 64 * lw3;   // words of the group
        const int64_t gv = (int64_t)(m >> 6) * 64 * lw;    // heads of the group
        int64_t off = 0, voff = 0;
        for (int w = 0; w < lw3; ++w) {
            const bool on = 3 * w < hd;
            const uint64_t mask = __ballot(on);
            if (mask == 0) break;
            I4 ca[3], cb[3];
#pragma unroll
            for (int sft = 0; sft < 3; ++sft) {
                const bool ons = 3 * w + sft < hd;
                const uint64_t ms = __ballot(ons);
                const int cs = __popcll(ms);
                if (ons && (w & 3) == turn) {
                    const int32_t *u = ecol + unit_entry(gv + voff, cs, lanes_below(ms), 0);
                    ca[sft] = *reinterpret_cast<const I4 *>(u);
                    cb[sft] = *reinterpret_cast<const I4 *>(u + 4 * cs);
                }
                voff += cs;
            }
            if (on && (w & 3) == turn) {
                U4 wa = (U4)0, wb = (U4)0;
#pragma unroll
                for (int sft = 0; sft < 3; ++sft) {
                    const int sl = 3 * w + sft;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (sl < min(len[k], lw)) wa[k] |= (uint32_t)set.find(ca[sft][k]) << (10 * sft);
                        if (sl < min(len[k + 4], lw))
                            wb[k] |= (uint32_t)set.find(cb[sft][k]) << (10 * sft);
                    }
                }
                const int r = lanes_below(mask), c = __popcll(mask);
                *reinterpret_cast<U4 *>(elocal + unit_entry(g0 + off, c, r, 0)) = wa;
                *reinterpret_cast<U4 *>(elocal + unit_entry(g0 + off, c, r, 4)) = wb;
            }
            off += __popcll(mask);
        }
    }
    if (tid == 0) {
        tdescT[t] = fits ? ni : 0;
        if (fits) atomicMax(&stats[0], ni);
        else atomicAdd(&stats[1], 1);
    }
}

// lam_n = C'(f^n)^T (S^T lam_next); part[block] = sum of (S^T lam).(dC/dtau).
//   d feq_a / d rho = w_a [1 - 4.5 (e_a.u)^2 + 1.5 u^2]
//   d feq_a / d j   = w_a [3 e_a + 9 (e_a.u) e_a - 3 u]
//   C_a = f_a - (f_a - feq_a)/tau, so
//   lam_b = (1 - 1/tau) lg_b + (1/tau) (A + B . e_b),
//   A = sum_a lg_a d feq_a / d rho, B = sum_a lg_a d feq_a / d j,
//   d C_a / d tau = (f_a - feq_a) / tau^2.
// One workgroup per tile of source nodes. Tiles with an inverse halo stage
// lam_next of that halo in LDS and read the row heads through local indices;
// other tiles (and the rare row tails beyond lw entries) read global memory.
// Every row is summed in its sorted order, so both paths give identical sums.
// Two wavefronts per group of 64 source nodes (512 threads per tile):
// wavefront 2g + h walks group g's units for directions 1-4 (h = 0) or 5-8
// (h = 1) and loads only its half of each unit (each half is one contiguous
// run per slot block), which doubles the wavefronts that keep loads in flight.
// Both take the same ballots (over the longest of the node's eight rows),
// exchange their four row sums through LDS and finish the node together:
// h = 0 reads f^n, passes its moments over and stores lambda_0..4 and the
// tau partial, h = 1 stores lambda_5..8.
//
// GR groups make a workgroup: four (a whole tile) where the tiles fill the
// chip, two or one where they do not (adj_groups), each with the halo of its tile.
// FP32 pairs and FP64 single groups take a chunk of C = 4 triples at a time, asking
// for the first one's weights before they wait for the halo; the others go triple
// by triple and let their many wavefronts overlap (FP64 pairs with chunks of four
// measured 5 to 10 % slower, FP32 ones without 5 to 25 %). FP32 pairs and whole
// tiles fetch UN = 4 halo nodes a lane at a time, which costs registers that FP64
// pays for. What is left of a small step is its chain of dependent trips (row
// bounds, units, halo, moments).
// A large step is bound by the traffic of the heads: 262,144 nodes FP32 read
// about 0.42 GB in 66 us, 6.3 TB/s.
template <class T, int GR>
__global__ __launch_bounds__(128 * GR) void k_adj_step(
    int n, const T *__restrict__ fn, const T *__restrict__ lam_next, T *__restrict__ lam_n,
    const int32_t *__restrict__ ptr, const int32_t *__restrict__ col, const T *__restrict__ val,
    int lw, const int32_t *__restrict__ ecol, const T *__restrict__ eval,
    const int32_t *__restrict__ tdescT, const int32_t *__restrict__ ilist,
    const uint32_t *__restrict__ elocal, int hcap, double rtau, double rho0, int dev,
    double *__restrict__ part, int add, int32_t *err) {
    constexpr int NTH = 128 * GR, PER = kTile / 64 / GR;   // workgroups per tile
    constexpr int C = GR < 4 && (GR == 1 || sizeof(T) == 4) ? 4 : 1;
    constexpr int UN = GR == 4 || sizeof(T) == 4 ? 4 : 1;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ T s_x[GR][2][4][64];   // row sums exchanged between the halves
    __shared__ T s_m[GR][4][64];      // moments of f^n, from half 0 to half 1
    __shared__ int s_hd[GR][2][64];   // head length over each half's rows
    typedef T T4 __attribute__((ext_vector_type(4)));
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));
    typedef int32_t I4 __attribute__((ext_vector_type(4)));
    const int64_t nwg = ((int64_t)n + 64 * GR - 1) / (64 * GR);
    const int64_t wg = xcd_tile(nwg);
    if (wg >= nwg) return;
    const int t = (int)(wg / PER), tid = threadIdx.x;
    const int wv = tid >> 6, lane = tid & 63;
    const int hv = wv & 1, gq = wv >> 1;    // direction half, group within the workgroup
    const int m = (int)(wg * GR + gq) * 64 + lane;
    const int ni = tdescT ? tdescT[t] : 0;
    T *L = reinterpret_cast<T *>(smem);   // [8][ni]

    T acc[4] = {0, 0, 0, 0};   // rows 4 hv + i
    // each half reads its own four row lengths; the head length over all
    // eight is exchanged across the staging barrier
    int hmax = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (m < n) {
            const int64_t row = (int64_t)(4 * hv + i) * n + m;
            hmax = max(hmax, min(ptr[row + 1] - ptr[row], lw));
        }
    }
    s_hd[gq][hv][lane] = hmax;
    // The heads are compacted per group of 64 nodes: slot e holds one unit
    // for each node with hmax > e (ballot and masked bit count give a lane's
    // unit), slots past a row's end hold weight 0, and a triple of slots is
    // loaded together, non-temporal (the heads are streamed once per step and
    // need not displace the lambda rows from L2); fetching one triple ahead
    // measured slower. A lane past its head (or past the last node) reads its
    // group's first unit (a line the group fetches anyway; one shared address
    // for all such lanes would be a hot spot) and adds nothing: its weights
    // are zeroed and its local columns point at position 0.
    const T4 *ev = reinterpret_cast<const T4 *>(eval);
    const U4 *elw = reinterpret_cast<const U4 *>(elocal);
    const int lw3 = (lw + 2) / 3;
    const int64_t grp = min(m, n - 1) >> 6;   // lanes past the last node: its group
    const int64_t gv = grp * 64 * lw, gw = grp * 64 * lw3;
    int64_t voff = 0, woff = 0;
    // the words and weights of triples w .. w + C - 1, this lane's or zero
    U4 wd[C];
    T4 v[C][3];
    auto triples = [&](int w) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const bool onw = 3 * (w + c) < hmax;
            const uint64_t mw = __ballot(onw);
            const int cw = __popcll(mw);
            const int64_t aw = onw ? 2 * (gw + woff) + lanes_below(mw) + hv * cw : 2 * gw;
            wd[c] = __builtin_nontemporal_load(elw + aw);
            wd[c] = onw ? wd[c] : (U4)0;
            woff += cw;
#pragma unroll
            for (int sft = 0; sft < 3; ++sft) {
                const bool on = 3 * (w + c) + sft < hmax;
                const uint64_t me = __ballot(on);
                const int ce = __popcll(me);
                const int64_t a = on ? 2 * (gv + voff) + lanes_below(me) + hv * ce : 2 * gv;
                const T4 va = __builtin_nontemporal_load(ev + a);
                v[c][sft] = on ? va : (T4)0;
                voff += ce;
            }
        }
    };
    if (C > 1 && ni > 0) {
        __syncthreads();
        hmax = max(hmax, s_hd[gq][1 - hv][lane]);
        triples(0);
    }
    if (ni > 0) {
        const int32_t *il = ilist + (int64_t)t * hcap;
#pragma unroll UN
        for (int h = tid; h < ni; h += NTH) {
            int q = il[h];
            if ((unsigned)q >= (unsigned)n) {   // a bad table must not fault
                q = 0;
                report_index(err);
            }
#pragma unroll
            for (int k = 1; k < kQ; ++k) L[(k - 1) * ni + h] = lam_next[(int64_t)k * n + q];
        }
    }
    __syncthreads();
    hmax = max(hmax, s_hd[gq][1 - hv][lane]);
    int wmax = hmax;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wmax = max(wmax, __shfl_xor(wmax, off));
    const int ntrip = (wmax + 2) / 3;
    if (ni > 0) {
        const T *Lh = L + 4 * hv * ni;
        for (int w = 0; w < ntrip; w += C) {
            if (C == 1 || w > 0) triples(w);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (w + c >= ntrip) break;
#pragma unroll
                for (int sft = 0; sft < 3; ++sft) {
                    const int sh = 10 * sft;
                    acc[0] += v[c][sft].x * Lh[0 * ni + ((wd[c].x >> sh) & 1023u)];
                    acc[1] += v[c][sft].y * Lh[1 * ni + ((wd[c].y >> sh) & 1023u)];
                    acc[2] += v[c][sft].z * Lh[2 * ni + ((wd[c].z >> sh) & 1023u)];
                    acc[3] += v[c][sft].w * Lh[3 * ni + ((wd[c].w >> sh) & 1023u)];
                }
            }
        }
    }
    if (m < n) {
        if (ni == 0) {
            const I4 *ec = reinterpret_cast<const I4 *>(ecol);
            const T *lk = lam_next + (int64_t)(1 + 4 * hv) * n;
            for (int e = 0; e < lw; ++e) {
                const bool on = e < hmax;
                const uint64_t me = __ballot(on);
                if (me == 0) break;
                const int ce = __popcll(me);
                const int64_t a = on ? 2 * (gv + voff) + lanes_below(me) + hv * ce : 2 * gv;
                const T4 va = on ? ev[a] : (T4)0;
                const I4 ca = ec[a];
                acc[0] += va.x * lk[0 * (int64_t)n + ca.x];
                acc[1] += va.y * lk[1 * (int64_t)n + ca.y];
                acc[2] += va.z * lk[2 * (int64_t)n + ca.z];
                acc[3] += va.w * lk[3 * (int64_t)n + ca.w];
                voff += ce;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 4 * hv + i;
            const T *lk = lam_next + (int64_t)(k + 1) * n;
            const int64_t row = (int64_t)k * n + m;
            const int b0 = ptr[row], b1 = ptr[row + 1];
            for (int e = b0 + lw; e < b1; ++e) acc[i] += val[e] * lk[col[e]];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) s_x[gq][hv][i][lane] = acc[i];
    T fk[kQ], rho = 0, ux = 0, uy = 0, drho = 0;
    if (hv == 0 && m < n) {
        moments_of<T>(fn, n, m, dev, rho0, fk, rho, ux, uy, drho);
        s_m[gq][0][lane] = rho;
        s_m[gq][1][lane] = ux;
        s_m[gq][2][lane] = uy;
        s_m[gq][3][lane] = drho;
    }
    __syncthreads();
    double dt = 0.0;
    if (m < n) {
        T lg[kQ];
        lg[0] = lam_next[m];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lg[1 + i] = hv ? s_x[gq][0][i][lane] : acc[i];
            lg[5 + i] = hv ? acc[i] : s_x[gq][1][i][lane];
        }
        if (hv) {
            rho = s_m[gq][0][lane];
            ux = s_m[gq][1][lane];
            uy = s_m[gq][2][lane];
            drho = s_m[gq][3][lane];
        }
        const T uu = ux * ux + uy * uy;
        T A = 0, Bx = 0, By = 0;
        double dtl = 0.0;
#pragma unroll
        for (int a = 0; a < kQ; ++a) {
            const T ex = (T)lat_ex(a), ey = (T)lat_ey(a);
            const T eu = ex * ux + ey * uy;
            const T wl = lat_wmul(a, lg[a]);
            A += wl * ((T)1 - (T)4.5 * eu * eu + (T)1.5 * uu);
            Bx += wl * ((T)3 * ex + (T)9 * eu * ex - (T)3 * ux);
            By += wl * ((T)3 * ey + (T)9 * eu * ey - (T)3 * uy);
            if (hv == 0) {   // the tau partial, from the half that holds f^n
                const T poly = (T)3 * eu + (T)4.5 * eu * eu - (T)1.5 * uu;
                const T fneq = dev ? fk[a] - lat_wmul(a, drho + rho * poly)
                                   : fk[a] - lat_wmul(a, rho * ((T)1 + poly));
                dtl += (double)lg[a] * (double)fneq;
            }
        }
        dt = hv ? 0.0 : dtl * rtau * rtau;
        const T rt = (T)rtau;
        const int b0 = hv ? 5 : 0, b1 = hv ? kQ : 5;
#pragma unroll
        for (int b = 0; b < kQ; ++b)
            if (b >= b0 && b < b1)
                lam_n[(int64_t)b * n + m] =
                    ((T)1 - rt) * lg[b] + rt * (A + Bx * (T)lat_ex(b) + By * (T)lat_ey(b));
    }
    block_sum_to<NTH>(dt, part, wg, add != 0);
}

// dJ/df_b for J = 1/2 sum |u - u*|^2: (r . (e_b - u)) / rho, r = u - u*.
template <class T>
__global__ __launch_bounds__(256) void k_loss_seed(int n, const int32_t *__restrict__ perm,
                                                   const T *__restrict__ fT,
                                                   const double *__restrict__ uxt,
                                                   const double *__restrict__ uyt,
                                                   T *__restrict__ lam, double rho0, int dev,
                                                   double *__restrict__ part) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    double jl = 0.0;
    if (p < n) {
        T fk[kQ], rho, ux, uy, drho;
        moments_of<T>(fT, n, p, dev, rho0, fk, rho, ux, uy, drho);
        const int u = perm[p];
        const double rx = (double)ux - uxt[u], ry = (double)uy - uyt[u];
        jl = 0.5 * (rx * rx + ry * ry);
#pragma unroll
        for (int b = 0; b < kQ; ++b)
            lam[(int64_t)b * n + p] =
                (T)((rx * ((double)lat_ex(b) - (double)ux) + ry * ((double)lat_ey(b) - (double)uy)) /
                    (double)rho);
    }
    block_sum_to(jl, part, blockIdx.x);
}

// dJ/du0 = sum_k lam_k d feq_k(rho0, u0) / d u0.
template <class T>
__global__ void k_init_adjoint(int n, const int32_t *__restrict__ perm,
                               const double *__restrict__ u0x, const double *__restrict__ u0y,
                               const T *__restrict__ lam, double rho0, double *__restrict__ gx,
                               double *__restrict__ gy) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int u = perm[p];
    const double ux = u0x ? u0x[u] : 0.0, uy = u0y ? u0y[u] : 0.0;
    double sx = 0.0, sy = 0.0;
    for (int k = 0; k < kQ; ++k) {
        const double l = (double)lam[(int64_t)k * n + p];
        const double eu = lat_ex(k) * ux + lat_ey(k) * uy;
        sx += l * lat_w(k) * rho0 * (3.0 * lat_ex(k) + 9.0 * eu * lat_ex(k) - 3.0 * ux);
        sy += l * lat_w(k) * rho0 * (3.0 * lat_ey(k) + 9.0 * eu * lat_ey(k) - 3.0 * uy);
    }
    gx[u] = sx;
    gy[u] = sy;
}

}  // namespace

size_t transpose_temp_bytes(int n, int K) {
    (void)K;
    const size_t rows = (size_t)8 * n;
    return ((rows * sizeof(int32_t) + 255) & ~size_t(255)) + scan_temp_bytes((int)rows) + 256;
}

hipError_t launch_transpose(const CloudPlan &cp, int precision, void *tmp, size_t tmp_bytes,
                            hipStream_t s) {
    const int n = cp.n, K = cp.K, mode = cp.prm.stencil_mode;
    const int64_t rows = (int64_t)8 * n;
    int32_t *cnt = (int32_t *)tmp;
    const size_t cnt_bytes = ((size_t)rows * sizeof(int32_t) + 255) & ~size_t(255);
    void *scan_tmp = (char *)tmp + cnt_bytes;
    const size_t scan_bytes = tmp_bytes - cnt_bytes;
    hipError_t e = launch_fill_i32(cnt, 0, rows, s);
    if (e != hipSuccess) return e;
    if (n >= (1 << 29)) return hipErrorInvalidValue;   // hash keys 4 n + m in 32 bits
    // tiles of 256 arriving nodes (neighbouring tiles on one XCD, whose L2
    // then merges the runs they write into shared rows) x half of the directions
    const dim3 egrid(xcd_grid(blocks_for(n, 256)), 2);
    hipLaunchKernelGGL(k_tr_count, egrid, dim3(kTrCs * 256), 0, s, n, K, mode, cp.nbr, cp.owner, cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = exclusive_scan(scan_tmp, scan_bytes, cnt, cp.tr_ptr, (int)rows, s)) != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, s, cp.tr_ptr + rows,
                       (int32_t)(rows * K));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_fill_i32(cnt, 0, rows, s)) != hipSuccess) return e;
    // staging of the fill: TT K entries of a tile (column, place, weight),
    // 128 nodes a tile while they take at most 46 KiB (with the hash table,
    // under 64 KiB), else 64
    const size_t esz = precision == MLBM_FP64 ? sizeof(double) : sizeof(float);
    auto stage_bytes = [&](int tt) {
        return 2 * (((size_t)tt * K * 4 + 15) & ~size_t(15)) + (size_t)tt * K * esz;
    };
    const bool wide = stage_bytes(128) <= 46 * 1024;
    const unsigned lds = (unsigned)stage_bytes(wide ? 128 : 64);
    const dim3 fgrid(xcd_grid(blocks_for(n, wide ? 128 : 64)), 2);
    if (precision == MLBM_FP64) {
        if (wide)
            hipLaunchKernelGGL((k_tr_fill<double, 128>), fgrid, dim3(kTrJs * 128), lds, s, n, K, mode,
                               cp.nbr, cp.owner, (const float *)nullptr, cp.W64, cp.tr_ptr, cnt,
                               cp.tr_col, (double *)cp.tr_val);
        else
            hipLaunchKernelGGL((k_tr_fill<double, 64>), fgrid, dim3(kTrJs * 64), lds, s, n, K, mode,
                               cp.nbr, cp.owner, (const float *)nullptr, cp.W64, cp.tr_ptr, cnt,
                               cp.tr_col, (double *)cp.tr_val);
    } else {
        if (wide)
            hipLaunchKernelGGL((k_tr_fill<float, 128>), fgrid, dim3(kTrJs * 128), lds, s, n, K, mode,
                               cp.nbr, cp.owner, cp.W32, (const double *)nullptr, cp.tr_ptr, cnt,
                               cp.tr_col, (float *)cp.tr_val);
        else
            hipLaunchKernelGGL((k_tr_fill<float, 64>), fgrid, dim3(kTrJs * 64), lds, s, n, K, mode,
                               cp.nbr, cp.owner, cp.W32, (const double *)nullptr, cp.tr_ptr, cnt,
                               cp.tr_col, (float *)cp.tr_val);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_tr_finish(cp, precision, false, s);
}

hipError_t launch_tr_finish(const CloudPlan &cp, int precision, bool sorted, hipStream_t s) {
    if (cp.tr_lw > kEllMaxLw) return hipErrorInvalidValue;
    const size_t esz = precision == MLBM_FP64 ? sizeof(double) : sizeof(float);
    const unsigned lds = (unsigned)(16 * kFinPitch * 4 + 4 * kFinRows * (cp.tr_lw | 1) * (4 + esz));
    const dim3 grid(xcd_grid(head_nodes(cp.n) / kFinRows), 2), block(256);
    auto k64 = sorted ? k_tr_finish<double, true> : k_tr_finish<double, false>;
    auto k32 = sorted ? k_tr_finish<float, true> : k_tr_finish<float, false>;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k64, grid, block, lds, s, cp.n, cp.tr_lw, cp.tr_ptr, cp.tr_col,
                           (double *)cp.tr_val, cp.ell_col, (double *)cp.ell_val);
    else
        hipLaunchKernelGGL(k32, grid, block, lds, s, cp.n, cp.tr_lw, cp.tr_ptr, cp.tr_col,
                           (float *)cp.tr_val, cp.ell_col, (float *)cp.ell_val);
    return hipGetLastError();
}

hipError_t launch_loss_seed(const CloudPlan &cp, int precision, const void *fT,
                            const double *uxt, const double *uyt, void *lam, double *J,
                            double *part, hipStream_t s) {
    const int n = cp.n;
    const int64_t nb = blocks_for(n, 256);
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_loss_seed<double>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const double *)fT, uxt, uyt, (double *)lam, cp.prm.rho0, 0, part);
    else
        hipLaunchKernelGGL(k_loss_seed<float>, dim3(nb), dim3(256), 0, s, n, cp.perm,
                           (const float *)fT, uxt, uyt, (float *)lam, cp.prm.rho0, 1, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s, nb, (const double *)part, J, 0);
    return hipGetLastError();
}

// Groups per workgroup of the reversed step. us a step of mlbm_steps_adjoint, one /
// two / four groups (the form of the precision; FP32 takes no single groups):
//   nodes    FP32 K 6     K 12         K 30         FP64 K 6            K 12                K 30
//   1,600    7.4 / 7.1    8.7 / 8.4    10.5 / 12.0  8.1 / 7.4 / 8.1     9.6 / 8.9 / 9.9     12 / 14 / 17
//   16,384   8.0 / 9.0    9.4 / 10.7   12.9 / 16.8  9.3 / 10.0 / 11.8   11.3 / 12.4 / 15.3  16 / 19 / 27
//   32,761   8.5 / 9.4    10.1 / 11.2  14.6 / 17.4  11.6 / 10.5 / 12.4  15.0 / 13.1 / 16.4  22 / 21 / 29
//   40,000   9.7 / 9.5    12.1 / 11.5  16.9 / 17.8  13.1 / 12.5 / 12.5  17.5 / 16.7 / 16.7  27 / 29 / 29
//   48,841   9.9 / 9.7    12.7 / 11.8  17.8 / 18.6  13.6 / 12.9 / 12.8  18.1 / 17.1 / 17.1  29 / 31 / 31
//   65,536   10.6 / 10.2  14.0 / 12.6  20.7 / 21.0  16.0 / 13.8 / 13.7  22 / 19 / 18        48 / 33 / 33
// FP64 K 48 at 40,000 nodes 50 / 42 / 42.
static int adj_groups(const CloudPlan &cp, int precision) {
    const int n = cp.n, K = cp.K;
    if (precision != MLBM_FP64) return n <= (K < 24 ? 36864 : 49152) ? 2 : 4;
    if (n <= 20480) return 1;
    if (n <= 36864) return 2;
    return n <= 49152 && K >= 18 && K <= 40 ? 1 : 4;
}

int64_t adjoint_parts(const CloudPlan &cp, int precision) {
    return blocks_for(cp.n, 64 * adj_groups(cp, precision));
}

template <class T, int GR>
static void launch_adj(const CloudPlan &cp, int dev, const void *fn, const void *lam_next,
                       void *lam_n, double *part, bool add, hipStream_t s) {
    const unsigned lds = cp.adj_ni ? (unsigned)(8 * cp.adj_ni * sizeof(T)) : 0;
    hipLaunchKernelGGL((k_adj_step<T, GR>), dim3(xcd_grid(blocks_for(cp.n, 64 * GR))), dim3(128 * GR), lds,
                       s, cp.n, (const T *)fn, (const T *)lam_next, (T *)lam_n, cp.tr_ptr, cp.tr_col,
                       (const T *)cp.tr_val, cp.tr_lw, cp.ell_col, (const T *)cp.ell_val,
                       cp.adj_ni ? cp.tdescT : nullptr, cp.ilist, cp.elocal, cp.hcap,
                       1.0 / cp.prm.tau, cp.prm.rho0, dev, part, add ? 1 : 0, cp.err);
}

hipError_t launch_step_adjoint(const CloudPlan &cp, int precision, const void *fn,
                               const void *lam_next, void *lam_n, double *part, bool add,
                               hipStream_t s) {
    const int groups = adj_groups(cp, precision);
    if (precision == MLBM_FP64)
        groups == 1 ? launch_adj<double, 1>(cp, 0, fn, lam_next, lam_n, part, add, s)
        : groups == 2 ? launch_adj<double, 2>(cp, 0, fn, lam_next, lam_n, part, add, s)
                      : launch_adj<double, 4>(cp, 0, fn, lam_next, lam_n, part, add, s);
    else
        groups == 2 ? launch_adj<float, 2>(cp, 1, fn, lam_next, lam_n, part, add, s)
                    : launch_adj<float, 4>(cp, 1, fn, lam_next, lam_n, part, add, s);
    return hipGetLastError();
}

hipError_t launch_adjoint_tau(const CloudPlan &cp, int precision, const double *part, double *dtau,
                              hipStream_t s) {
    hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(256), 0, s,
                       adjoint_parts(cp, precision), part, dtau, 1);
    return hipGetLastError();
}

hipError_t launch_init_adjoint(const CloudPlan &cp, int precision, const double *u0x,
                               const double *u0y, const void *lam0, double *gx, double *gy,
                               hipStream_t s) {
    const int n = cp.n;
    if (precision == MLBM_FP64)
        hipLaunchKernelGGL(k_init_adjoint<double>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, u0x, u0y, (const double *)lam0, cp.prm.rho0, gx, gy);
    else
        hipLaunchKernelGGL(k_init_adjoint<float>, dim3(blocks_for(n, 256)), dim3(256), 0, s, n,
                           cp.perm, u0x, u0y, (const float *)lam0, cp.prm.rho0, gx, gy);
    return hipGetLastError();
}

hipError_t launch_adj_tiles(const CloudPlan &cp, int32_t *stats, hipStream_t s) {
    const int ntiles = (cp.n + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_adj_tiles, dim3(ntiles), dim3(1024), 0, s, cp.n, cp.tr_lw, cp.hcap,
                       cp.adj_cap, cp.tr_ptr, cp.tr_col, cp.ell_col, cp.tdescT, cp.ilist,
                       cp.elocal, stats);
    return hipGetLastError();
}

}  // namespace mlbm
