// Device helper of the per-cluster row passes (proxy.hip, codec.hip).  Internal
// to the library.
#pragma once

#include "common.hpp"

namespace ps {
namespace {

constexpr int kListChunk = 512;   // listed rows a wave looks through at a time

// The entries p = list[0..n) (n <= kListChunk) with 0 <= p < seq and
// labels[p] == k, in list order, into rows[]; returns how many.  CLAMP: entries
// outside [0, seq) are taken as the nearest position instead of skipped.  One
// wave per workgroup; the entries are visible to all its lanes on return.
template <bool CLAMP = false>
__device__ __forceinline__ int list_members(const int32_t* list, int n, const int32_t* labels, int seq, int k,
                                            int32_t* rows) {
    const int lane = threadIdx.x & (kWave - 1);
    int m = 0;
    for (int i0 = 0; i0 < n; i0 += kWave) {
        int p = i0 + lane < n ? list[i0 + lane] : -1;
        if (CLAMP && i0 + lane < n) p = min(max(p, 0), seq - 1);
        const bool in = p >= 0 && p < seq && labels[p] == k;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
        if (in) rows[m + __builtin_popcountll(mask & ((1ull << lane) - 1))] = p;
        m += __builtin_popcountll(mask);
    }
    __syncthreads();
    return m;
}

}  // namespace
}  // namespace ps
