// A workgroup's set of node indices in LDS, with the position of each in the
// sorted set: the gather tables of the step and of its adjoint renumber the
// nodes that a tile reads.
//
// The set is a hash table of 32-node words (key = index / 32, a mask of the
// members), since nodes in Hilbert order come in runs: a tile's 500 to 1,000
// members fill some 100 to 200 words. The members before a word are the sum of
// the mask counts of all smaller keys, counted over all words by eight lanes a
// word, so nothing is sorted: a set of w words costs w^2 / blockDim reads a
// thread (about 20; 1,000 if no two members share a word), where a bitonic
// network over the members took 55 to 66 passes with a barrier each. A look-up
// is one probe as a rule, where a binary search took ten dependent reads.
#pragma once

#include "common.h"

namespace mlbm {

struct IndexSet {
    static constexpr int kSlots = 4096;    // hash table (power of two)
    static constexpr int kWords = 2048;    // words kept; more of them: over is set
    static constexpr uint32_t kNone = 0xFFFFFFFFu;

    uint32_t key[kSlots], mask[kSlots];
    uint32_t packed[kWords];               // key and member count of word i
    uint16_t first[kSlots];                // members before the word
    uint16_t slot[kWords];
    int words, members, over;

    // All threads; a barrier has to follow before the first add.
    __device__ void clear() {
        for (int i = threadIdx.x; i < kSlots; i += blockDim.x) {
            key[i] = kNone;
            mask[i] = 0;
        }
        if (threadIdx.x == 0) words = members = over = 0;
    }

    __device__ static uint32_t home(uint32_t k) { return (k * 2654435761u) >> 20; }   // 12 bits

    __device__ static uint32_t peek(const uint32_t *p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    __device__ void add(int32_t q) {
        const uint32_t k = (uint32_t)q >> 5, bit = 1u << (q & 31);
        uint32_t h = home(k);
        for (int probe = 0; probe < kSlots; ++probe) {
            uint32_t cur = peek(&key[h]);
            if (cur == kNone) {
                cur = atomicCAS(&key[h], kNone, k);
                if (cur == kNone) {
                    const int i = atomicAdd(&words, 1);
                    if (i < kWords) slot[i] = (uint16_t)h;
                    else over = 1;
                    cur = k;
                }
            }
            if (cur == k) {
                if (!(peek(&mask[h]) & bit)) atomicOr(&mask[h], bit);
                return;
            }
            h = (h + 1) & (kSlots - 1);
        }
        over = 1;
    }

    // All threads, after a barrier behind the last add; the count of members
    // holds for all threads after it returns (it ends with a barrier).
    __device__ void count() {
        const int nw = min(words, kWords);
        for (int i = threadIdx.x; i < nw; i += blockDim.x) {
            const int c = __popc(mask[slot[i]]);
            packed[i] = (key[slot[i]] << 6) | (uint32_t)c;
            atomicAdd(&members, c);
        }
        __syncthreads();
    }

    // All threads, after count() and with over unset: the members in order to
    // out, and their positions for find() (a barrier has to follow).
    __device__ void order(int32_t *out) {
        const int nw = words, l = threadIdx.x & 7;
        for (int i = threadIdx.x >> 3; i < nw; i += blockDim.x >> 3) {
            const uint32_t lim = packed[i] & ~63u;
            int before = 0;
            for (int j = l; j < nw; j += 8) {
                const uint32_t p = packed[j];
                before += p < lim ? (int)(p & 63u) : 0;
            }
#pragma unroll
            for (int off = 4; off > 0; off >>= 1) before += __shfl_xor(before, off, 8);
            const int h = slot[i];
            if (l == 0) first[h] = (uint16_t)before;
            const uint32_t mk = mask[h];
            const int32_t q0 = (int32_t)(key[h] << 5);
#pragma unroll
            for (int b = 0; b < 4; ++b) {   // lane l writes members 4 l .. 4 l + 3 of the word
                const int at = 4 * l + b;
                if (mk >> at & 1u) out[before + __popc(mk & ((1u << at) - 1u))] = q0 + at;
            }
        }
    }

    // Position of member q, after order() and a barrier.
    __device__ int find(int32_t q) const {
        const uint32_t k = (uint32_t)q >> 5;
        uint32_t h = home(k);
        for (int probe = 0; probe < kSlots && key[h] != k; ++probe) h = (h + 1) & (kSlots - 1);
        return first[h] + __popc(mask[h] & ((1u << (q & 31)) - 1u));
    }
};

}  // namespace mlbm
