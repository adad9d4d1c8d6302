// Expert activation counts and the token -> expert permutation.
//
// The counts are the per-sequence "activity level" of each expert that DAOP's
// sequence-specific allocation consumes (Sec. IV-B, Algorithm 1: tokens
// assigned to each expert).  The permutation groups the (token, j) selections
// by expert so that each expert processes all of its tokens together
// (Algorithm 1's parallel local expert execution).
//
// Everything is integer work and fully deterministic: each workgroup of the
// routing kernel leaves a histogram of its 16 tokens; here every workgroup
// re-derives, from those histograms, the expert totals and the number of
// selections that precede its own tokens, then ranks its own selections in
// token order.  The resulting order inside an expert is by (token, j).
#include "moe_internal.h"

namespace moe {
namespace {

__global__ __launch_bounds__(64) void hist_from_idx_kernel(const int32_t* __restrict__ idx, int tokens, int k,
                                                           int E, int32_t* __restrict__ hist) {
    __shared__ int h[64];
    const int tid = threadIdx.x;
    h[tid] = 0;
    __syncthreads();
    const int a0 = blockIdx.x * kRouteTokensPerBlock * k;
    const int a1 = min(tokens * k, a0 + kRouteTokensPerBlock * k);
    for (int a = a0 + tid; a < a1; a += 64) {
        const int e = min(max(idx[a], 0), E - 1);
        atomicAdd(&h[e], 1);
    }
    __syncthreads();
    if (tid < E) hist[(size_t)blockIdx.x * E + tid] = h[tid];
}

// Inclusive sum over the lanes of a wavefront.
__device__ inline int lane_prefix(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Ranks the n_local selections (at most 128, one per thread of the first two wavefronts; expert `e` in thread tid)
// among those of the same expert: slot = base[e] + selections of e before it.  A wavefront finds the lanes of the same
// expert from six ballots, one per bit of the expert's number (a loop over the selections before a thread's own cost
// up to 96 LDS reads in a row; with it and a running sum over 64 experts 1003 tokens took 11.7 us, now 8.1); the second wavefront starts from the first
// one's counts.  Call with all threads of the workgroup; `first_half` is scratch, `base` has been written and synchronised.
__device__ inline void rank_selections(int n_local, int e, int a0, const int* base, int* first_half,
                                       int32_t* __restrict__ row_of_slot, int32_t* __restrict__ slot_of) {
    const int tid = threadIdx.x, lane = tid & 63;
    const bool on = tid < n_local;
    uint64_t same = __ballot(on);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const bool bit = ((e >> b) & 1) != 0;
        const uint64_t m = __ballot(bit);
        same &= bit ? m : ~m;
    }
    const int before = __popcll(same & ((1ull << lane) - 1ull));
    if (on && tid < 64 && before == 0) first_half[e] = __popcll(same);  // an expert's first selection leaves the count
    __syncthreads();
    if (on) {
        const int slot = base[e] + before + (tid >= 64 ? first_half[e] : 0);
        slot_of[a0 + tid] = slot;
        row_of_slot[slot] = a0 + tid;
    }
}

// grid = max(1, n_blocks) workgroups of 256 threads.
__global__ __launch_bounds__(256) void finalize_kernel(const int32_t* __restrict__ hist, int n_blocks, int E,
                                                       int k, int tokens, const int32_t* __restrict__ idx,
                                                       int32_t* __restrict__ counts, int accumulate,
                                                       int32_t* __restrict__ offs,
                                                       int32_t* __restrict__ row_of_slot,
                                                       int32_t* __restrict__ slot_of, int32_t* __restrict__ sync) {
    __shared__ int total[64];
    __shared__ int before[64];
    __shared__ int base[64];
    __shared__ int first_half[64];
    const int tid = threadIdx.x;
    const int blk = blockIdx.x;
    static_assert(kRouteTokensPerBlock * 8 <= 128, "two wavefronts rank a block's selections");
    const int a0 = blk * kRouteTokensPerBlock * k;
    const int n_local = min(tokens * k, a0 + kRouteTokensPerBlock * k) - a0;
    // requested before the histograms, used after them
    const int my_e = row_of_slot != nullptr && tid < n_local ? min(max(idx[a0 + tid], 0), E - 1) : 0;
    if (tid < 64) {
        first_half[tid] = 0;
        total[tid] = 0;
        before[tid] = 0;
    }
    __syncthreads();
    // Coalesced sweep over all block histograms (integer sums, so the order is immaterial).  When E
    // divides the workgroup size a thread always meets the same expert and sums in registers.
    const int n_cells = n_blocks * E;
    const int my_first = blk * E;
    if (256 % E == 0) {
        int tot = 0, bef = 0;
#pragma unroll 4
        for (int i = tid; i < n_cells; i += 256) {
            const int v = hist[i];
            tot += v;
            bef += i < my_first ? v : 0;
        }
        if (tot != 0) atomicAdd(&total[tid % E], tot);
        if (bef != 0) atomicAdd(&before[tid % E], bef);
    } else {
        for (int i = tid; i < n_cells; i += 256) {
            const int v = hist[i];
            if (v != 0) {
                atomicAdd(&total[i % E], v);
                if (i < my_first) atomicAdd(&before[i % E], v);
            }
        }
    }
    __syncthreads();
    if (tid < 64) {  // (lanes of experts that do not exist hold zero)
        const int mine = total[tid], end = lane_prefix(mine);
        base[tid] = end - mine + before[tid];
        if (blk == 0 && offs != nullptr && tid < E) {
            offs[tid] = end - mine;
            if (tid == E - 1) offs[E] = end;
        }
    }
    if (blk == 0 && counts != nullptr && tid < E) counts[tid] = (accumulate ? counts[tid] : 0) + total[tid];
    if (blk == 0 && sync != nullptr)
        for (int i = tid; i < kSyncInts; i += 256) sync[i] = 0;
    if (row_of_slot == nullptr) return;
    __syncthreads();
    rank_selections(n_local, my_e, a0, base, first_half, row_of_slot, slot_of);
}

// ---- long calls: the fused kernel above sweeps all block histograms in every workgroup, which is
// quadratic in the number of blocks.  Beyond kFusedBlocks blocks one workgroup turns the histograms
// into per-block exclusive prefixes in place (and writes counts / offs), then one workgroup per
// block ranks its selections from its own row.
constexpr int kFusedBlocks = 1024;

// 1024 threads = 16 block ranges x 64 expert lanes.
__global__ __launch_bounds__(1024) void scan_blocks_kernel(int32_t* __restrict__ hist, int n_blocks, int E,
                                                           int32_t* __restrict__ counts, int accumulate,
                                                           int32_t* __restrict__ offs, int32_t* __restrict__ sync) {
    __shared__ int part[16][64];
    __shared__ int total[64];
    const int tid = threadIdx.x, e = tid & 63, g = tid >> 6;
    const int per = (n_blocks + 15) / 16;
    const int b0 = g * per, b1 = min(n_blocks, b0 + per);
    int sum = 0;
    if (e < E)
        for (int b = b0; b < b1; ++b) sum += hist[(size_t)b * E + e];
    part[g][e] = sum;
    __syncthreads();
    if (g == 0) {
        int run = 0;
        for (int i = 0; i < 16; ++i) {
            const int v = part[i][e];
            part[i][e] = run;
            run += v;
        }
        total[e] = run;
    }
    __syncthreads();
    if (e < E) {
        int run = part[g][e];
        for (int b = b0; b < b1; ++b) {
            const int v = hist[(size_t)b * E + e];
            hist[(size_t)b * E + e] = run;
            run += v;
        }
    }
    if (tid == 0 && offs != nullptr) {
        int run = 0;
        for (int i = 0; i < E; ++i) {
            offs[i] = run;
            run += total[i];
        }
        offs[E] = run;
    }
    if (tid < E && counts != nullptr) counts[tid] = (accumulate ? counts[tid] : 0) + total[tid];
    if (sync != nullptr)
        for (int i = tid; i < kSyncInts; i += 1024) sync[i] = 0;
}

// prefix: the histograms after scan_blocks_kernel; offs from the same kernel.
__global__ __launch_bounds__(256) void rank_kernel(const int32_t* __restrict__ prefix, const int32_t* __restrict__ offs,
                                                   int E, int k, int tokens, const int32_t* __restrict__ idx,
                                                   int32_t* __restrict__ row_of_slot, int32_t* __restrict__ slot_of) {
    __shared__ int base[64];
    __shared__ int first_half[64];
    const int tid = threadIdx.x, blk = blockIdx.x;
    if (tid < E) base[tid] = offs[tid] + prefix[(size_t)blk * E + tid];
    if (tid < 64) first_half[tid] = 0;
    const int a0 = blk * kRouteTokensPerBlock * k;
    const int n_local = min(tokens * k, a0 + kRouteTokensPerBlock * k) - a0;
    const int my_e = tid < n_local ? min(max(idx[a0 + tid], 0), E - 1) : 0;
    __syncthreads();
    rank_selections(n_local, my_e, a0, base, first_half, row_of_slot, slot_of);
}

}  // namespace

hipError_t launch_hist_from_idx(const moe_shape_t& s, int tokens, const int32_t* idx, int32_t* hist,
                                hipStream_t stream) {
    const int nb = route_blocks(tokens);
    if (nb > 0) hist_from_idx_kernel<<<nb, 64, 0, stream>>>(idx, tokens, s.top_k, s.n_experts, hist);
    return hipGetLastError();
}

hipError_t launch_finalize(const moe_shape_t& s, int tokens, int32_t* hist, const int32_t* idx,
                           int32_t* counts, int accumulate, int32_t* offs, int32_t* row_of_slot,
                           int32_t* slot_of, int32_t* sync, hipStream_t stream) {
    const int nb = route_blocks(tokens);
    if (row_of_slot != nullptr && nb > kFusedBlocks) {
        scan_blocks_kernel<<<1, 1024, 0, stream>>>(hist, nb, s.n_experts, counts, accumulate, offs, sync);
        rank_kernel<<<nb, 256, 0, stream>>>(hist, offs, s.n_experts, s.top_k, tokens, idx, row_of_slot, slot_of);
        return hipGetLastError();
    }
    const int grid = (row_of_slot != nullptr && nb > 0) ? nb : 1;
    finalize_kernel<<<grid, 256, 0, stream>>>(hist, nb, s.n_experts, s.top_k, tokens, idx, counts, accumulate,
                                              offs, row_of_slot, slot_of, sync);
    return hipGetLastError();
}

}  // namespace moe
