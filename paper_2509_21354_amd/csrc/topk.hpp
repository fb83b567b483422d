// The best k of n scores of one sequence, exactly: score descending, NaN as minus infinity, ties to the lower index.
//
// NW waves hold the scores as integer keys that order like them, KPL per lane (wave w has candidates 64 KPL w .. in runs of
// 64, see index(), so that ballots run in index order).  NW = 1: each wave of the workgroup by itself, without barriers.  The key of the k-th best is found bit by
// bit from the top: a trial value, the number of keys at or above it (ballots and bit counts, no shuffles), keep the bit
// if they are at least k.  The search ends early when they are exactly k.  32 n / 64 comparisons at most, where ranking
// by counting takes n^2 / 64.
#pragma once
#include "common.hpp"

namespace kvev {

// the key of a score: unsigned order = float order, -0 as +0, NaN as minus infinity; never 0, which pads
__device__ __forceinline__ uint32_t topk_key(float u)
{
    const uint32_t f = __float_as_uint((u != u ? -INFINITY : u) + 0.f);
    return f & 0x80000000u ? ~f : f | 0x80000000u;
}

template <int KPL, int NW> struct TopK {
    struct Lds { int cnt[2][NW], part[NW]; };

    // candidate of key[i]
    static __device__ __forceinline__ int index(int i)
    {
        return ((NW > 1 ? (int)(threadIdx.x >> 6) * KPL : 0) + i) * 64 + (int)(threadIdx.x & 63);
    }

    // sum over the workgroup of a wave-uniform count (phase: alternates between calls)
    static __device__ __forceinline__ int total(int c, Lds &lds, int &phase)
    {
        if constexpr (NW == 1) return c;
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) lds.cnt[phase][wave] = c;
        __syncthreads();
        int t = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += lds.cnt[phase][w];
        phase ^= 1;
        return t;
    }

    // For each flag of this lane: how many flags precede it in index order; returns the number of all flags.
    static __device__ __forceinline__ int before(const bool (&flag)[KPL], int (&pos)[KPL], Lds &lds)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const unsigned long long below = (1ull << lane) - 1ull;
        int count = 0;
#pragma unroll
        for (int i = 0; i < KPL; ++i) {
            const unsigned long long mask = __ballot(flag[i]);
            pos[i] = count + __popcll(mask & below);
            count += __popcll(mask);
        }
        if constexpr (NW == 1) return count;
        __syncthreads();             // (whoever still reads the counts of the call before)
        if (lane == 0) lds.part[wave] = count;
        __syncthreads();
        int base = 0, all = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int c = lds.part[w];
            base += w < wave ? c : 0;
            all += c;
        }
#pragma unroll
        for (int i = 0; i < KPL; ++i) pos[i] += base;
        return all;
    }

    // keep[i]: key[i] is among the best k (of n; padding keys are 0)
    static __device__ __forceinline__ void best(const uint32_t (&key)[KPL], int n, int k, bool (&keep)[KPL], Lds &lds)
    {
        if (k >= n || k <= 0) {
#pragma unroll
            for (int i = 0; i < KPL; ++i) keep[i] = k > 0 && key[i] != 0;
            return;
        }
        int phase = 0;
        auto at_least = [&](uint32_t t) __attribute__((always_inline)) {
            int c = 0;
#pragma unroll
            for (int i = 0; i < KPL; ++i) c += __popcll(__ballot(key[i] >= t));
            return total(c, lds, phase);
        };
        uint32_t t = 0;
        bool exact = false;
        for (int bit = 31; bit >= 0 && !exact; --bit) {
            const uint32_t trial = t | 1u << bit;
            const int c = at_least(trial);
            if (c >= k) { t = trial; exact = c == k; }
        }
#pragma unroll
        for (int i = 0; i < KPL; ++i) keep[i] = key[i] >= t;
        if (exact) return;
        // more than k keys at or above the k-th best key: of those equal to it, the first ones in index order
        const int need = k - (t == 0xffffffffu ? 0 : at_least(t + 1));
        bool tie[KPL];
        int rank[KPL];
#pragma unroll
        for (int i = 0; i < KPL; ++i) tie[i] = key[i] == t;
        before(tie, rank, lds);
#pragma unroll
        for (int i = 0; i < KPL; ++i) keep[i] = key[i] > t || (tie[i] && rank[i] < need);
    }
};

}  // namespace kvev
