// Who computes which work item of a grouped GEMM, and how a workgroup waits for items of others: without anything of the device, for the
// kernels and for a model of them on the host.
#pragma once

#include <stdint.h>

namespace moe {
namespace gg {

constexpr int kXcds = 8;

// Whether a workgroup's first item is its own by its number, which saves it the first claim.  Not in the first GEMM of a linked launch,
// for whose tiles others wait: the item of a workgroup that is not resident would be in nobody's hands, and the workgroups that wait
// for it may hold the CU that it needs.  There an item belongs to nobody until a running workgroup has claimed it.
constexpr bool owns_first(bool linked, int mats) { return !(linked && mats == 2); }

// Every XCD has a list of items, numbered from 0 (its whole tiles, then the pieces of its leftover tiles), and a counter of what has been
// claimed of it, zero at the start.  With OWN_FIRST the counter stands for the items behind the first `members`.
template <bool OWN_FIRST>
struct HandOut {
    int members;             // workgroups of an XCD
    int n_whole;             // whole tiles of an XCD
    int left, chunk, parts;  // leftover tiles of all, those of an XCD at most, pieces of each

    __host__ __device__ __attribute__((always_inline)) int left_of(int xcd) const {
        const int end = (xcd + 1) * chunk < left ? (xcd + 1) * chunk : left;
        return end > xcd * chunk ? end - xcd * chunk : 0;
    }
    __host__ __device__ __attribute__((always_inline)) int items(int xcd) const { return n_whole + left_of(xcd) * parts; }
    __host__ __device__ __attribute__((always_inline)) int reserved() const { return OWN_FIRST ? members : 0; }
    // The item that workgroup `member` has without a claim (-1: none).
    __host__ __device__ __attribute__((always_inline)) int first(int member, int xcd) const {
        return OWN_FIRST && member < items(xcd) ? member : -1;
    }
    // The item that claim number n of an XCD's counter stands for (-1: its list is at its end).
    __host__ __device__ __attribute__((always_inline)) int claimed(int n, int xcd) const {
        return reserved() + n < items(xcd) ? reserved() + n : -1;
    }
    // What an XCD's counter, standing at `count`, has still to hand out (0 or less: nothing).
    __host__ __device__ __attribute__((always_inline)) int open(int xcd, int count) const { return items(xcd) - reserved() - count; }
    // Whether the counters have anything to hand out (the first XCD's list is the longest).
    __host__ __device__ __attribute__((always_inline)) bool any() const { return items(0) > reserved(); }
};

// Waits until the expert of this rank is ready, in all wavefronts of a workgroup alike; false: the wait ran out.  Every wavefront multiplies
// the rows that each of them loads, so there is one answer for all: the first wavefront looks (`ready`: ranks that are) and shares what it
// has seen.  A workgroup that gave up once looks once from then on.
template <class Wavefront>
__host__ __device__ __attribute__((always_inline)) inline bool await_rank(int rank, uint64_t& ready, int& spin_limit, Wavefront& wavefront) {
    if ((ready >> rank & 1) != 0) return true;
    if (wavefront.is_first()) {
        for (int n = 0; (ready >> rank & 1) == 0; ++n) {
            if (n >= spin_limit) {
                wavefront.report();
                break;
            }
            if (n > 0) wavefront.pause();
            ready = wavefront.look();
        }
    }
    ready = wavefront.share(ready);
    if ((ready >> rank & 1) != 0) return true;
    if (spin_limit > 1) spin_limit = 1;
    return false;
}

}  // namespace gg
}  // namespace moe
