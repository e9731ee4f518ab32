// The order of lists of log scores, in a form that the host can run too: the rank of an entry is the number of entries that beat it.
#pragma once
#include <hip/hip_runtime.h>

// How many of v[from .. to) beat entry i, whose value is `mine`: larger value, or equal value and earlier place.  A NaN beats
// nothing and nothing beats it: for lists in which it marks a place without an entry.
template <int UNROLL>
__host__ __device__ __forceinline__ int rank_beaten(const double *v, int from, int to, double mine, int i) {
    int rank = 0;
#pragma unroll UNROLL
    for (int j = from; j < to; ++j) {
        const double o = v[j];
        rank += (o > mine) || (o == mine && j < i);
    }
    return rank;
}

// In a list all of whose entries take a place, whatever their values, NaN comes behind every number and by place among themselves,
// so that the ranks are a permutation: scores come from the caller's encoder frames, which nobody checks, and who reads an entry by
// its rank finds one at every rank below the list's length.  The rank, from the count above: (behind the count, not in
// it: a list without a NaN pays one comparison an entry)
__host__ __device__ __forceinline__ int rank_placed(const double *v, int n, double mine, int i, int beaten) {
    if (__builtin_expect(mine != mine, 0)) {
        beaten = 0;
#pragma unroll 1
        for (int j = 0; j < n; ++j) beaten += v[j] == v[j] || j < i;
    }
    return beaten;
}
template <int UNROLL>
__host__ __device__ __forceinline__ int rank_in_list(const double *v, int n, int i) {
    const double mine = v[i];
    return rank_placed(v, n, mine, i, rank_beaten<UNROLL>(v, 0, n, mine, i));
}
