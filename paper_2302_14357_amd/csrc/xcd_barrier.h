// What a workgroup reads from the word of its XCD's barrier (xcd_device.h), in a form that the host can run too.
#pragma once
#include "tbs_internal.h"

#define XR_NOT_YET (-2)

// word: arrivals (low half) and the sum of `live` (high half) since the launch began; due: the arrivals that end this barrier;
// seen: the sum up to the last barrier that ended a round.  live: this barrier ends a round.
// Only there may the high half be read.  At the barrier ahead of it a workgroup that is slow to look may find the others through
// it, through their step of the round and counted into the next one: their `live` is in the word by then.  At the barrier that ends
// a round all of that round's `live` is there, and none of the next round's can be: there are barriers in between, and no one passes
// those without this workgroup.
__host__ __device__ inline int xcd_barrier_read(u64 word, unsigned due, unsigned seen, bool live) {
    if ((int)((unsigned)word - due) < 0) return XR_NOT_YET;
    return live ? (int)((unsigned)(word >> 32) - seen) : 0;
}
