// Device code of the gating function shared by the routing kernels and the
// fused decode kernel (DAOP paper Sec. II-A "MoE Structure": gate logits,
// softmax over all experts, top-k with renormalised weights; the same
// computation with the next layer's gate gives the prediction of Sec. III
// observation 3 / Sec. IV-C).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

// Eight consecutive elements as loaded (16 or 32 bytes), converted to fp32 only when they are used,
// so that a group of loads can be issued back to back before the first conversion.
template <typename scalar_t>
struct Raw8;
template <>
struct Raw8<float> {
    float4 a, b;
    __device__ inline void load(const float* p) {
        a = *reinterpret_cast<const float4*>(p);
        b = *reinterpret_cast<const float4*>(p + 4);
    }
    __device__ inline void get(float (&v)[8]) const {
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
};
template <>
struct Raw8<uint16_t> {
    uint4 q;
    __device__ inline void load(const uint16_t* p) { q = *reinterpret_cast<const uint4*>(p); }
    __device__ inline void get(float (&v)[8]) const {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};

// Reductions over the 64 lanes, the result in every lane.  Within a row of 16 lanes the partners
// come through the data-parallel-primitive path (exchange with the neighbour, the neighbouring
// pair, the mirrored half row and the mirrored row: four register-to-register moves), the four row
// results are then read out as scalars.  An LDS-routed shuffle per step would cost about a hundred
// cycles each, and the softmax and top-k chain some twenty of these reductions one after another.
// Every lane performs the same operations on the same values in the same order, so all lanes hold
// bit-identical results (the additions of wave_sum are: pairs, quads, half rows, rows, then the
// four rows in ascending order).
template <int CTRL>
__device__ inline float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ inline float lane_value(float v, int lane) {  // lane is a compile-time constant at every use
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
constexpr int kDppSwapNeighbours = 0xB1;   // quad_perm [1, 0, 3, 2]
constexpr int kDppSwapPairs = 0x4E;        // quad_perm [2, 3, 0, 1]
constexpr int kDppHalfRowMirror = 0x141;   // lane i of each 8 <- lane 7 - i
constexpr int kDppRowMirror = 0x140;       // lane i of each 16 <- lane 15 - i

__device__ inline float wave_max(float v) {
    v = fmaxf(v, dpp_move<kDppSwapNeighbours>(v));
    v = fmaxf(v, dpp_move<kDppSwapPairs>(v));
    v = fmaxf(v, dpp_move<kDppHalfRowMirror>(v));
    v = fmaxf(v, dpp_move<kDppRowMirror>(v));
    const float r0 = lane_value(v, 0), r1 = lane_value(v, 16), r2 = lane_value(v, 32), r3 = lane_value(v, 48);
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

__device__ inline float wave_sum(float v) {
    v += dpp_move<kDppSwapNeighbours>(v);
    v += dpp_move<kDppSwapPairs>(v);
    v += dpp_move<kDppHalfRowMirror>(v);
    v += dpp_move<kDppRowMirror>(v);
    const float r0 = lane_value(v, 0), r1 = lane_value(v, 16), r2 = lane_value(v, 32), r3 = lane_value(v, 48);
    return ((r0 + r1) + r2) + r3;
}

// Softmax over the E logits held one per lane (z of lane e is expert e's logit, -inf beyond E),
// then k passes of arg-max across the lanes, the lowest lane among equals winning.  Every lane
// takes part; on return lane j < k holds selection j (expert and renormalised weight), in
// descending probability.
//
// With `degrade` (graceful degradation, Sec. IV-C "Accuracy Stabilization" / "Graceful
// Degradation"; `resident` = this lane's expert is in the GPU expert cache): if no selected expert
// is resident, the last selection (the lowest probability) is replaced by the most probable
// resident expert, if there is one; it cannot outrank the k - 1 selections that stay, so the
// order is preserved.
__device__ inline void select_topk_lanes(float z, int lane, int E, int k, int& my_sel, float& my_w,
                                         bool degrade = false, bool resident = false) {
    const float zmax = wave_max(z);
    float p = lane < E ? expf(z - zmax) : 0.f;
    p = p / wave_sum(p);
    bool taken = lane >= E;
    float my_p = 0.f, wsum = 0.f;
    my_sel = 0;
    for (int j = 0; j < k; ++j) {
        const float cand = taken ? -1.f : p;
        float best = wave_max(cand);
        uint64_t m = __ballot(!taken && cand == best);
        if (m == 0) {  // only with non-finite inputs: still select a valid, distinct expert
            m = __ballot(!taken);
            best = 0.f;
        }
        const int sel = __ffsll((long long)m) - 1;
        if (lane == sel) taken = true;
        if (lane == j) {
            my_sel = sel;
            my_p = best;
        }
        wsum += best;
    }
    if (degrade) {
        const bool selected = taken && lane < E;
        if (__ballot(selected && resident) == 0) {
            const bool cand = !taken && resident;
            const float best = wave_max(cand ? p : -1.f);
            const uint64_t m = __ballot(cand && p == best);
            if (m != 0) {
                if (lane == k - 1) {
                    my_sel = __ffsll((long long)m) - 1;
                    my_p = best;
                }
                wsum = 0.f;
                for (int j = 0; j < k; ++j) wsum += __shfl(my_p, j, 64);
            }
        }
    }
    my_w = my_p / wsum;
}

// ---- routing of a decode-size call (at most 16 tokens) by one workgroup of 8 wavefronts ----

constexpr int kSmallRouteThreads = 512;
constexpr int kSmallRouteMaxTokens = 16;

struct RouteSmem {
    int idx[kSmallRouteMaxTokens * 8];
    float w[kSmallRouteMaxTokens * 8];
};
// Floats of LDS scratch route_tokens_wg needs: [wavefront][token][expert] partial logits (bf16: the same as MFMA results).
constexpr int kRoutePartFloats = 8 * kSmallRouteMaxTokens * 64;

// Sums acc[0..8) over the 64 lanes with a halving exchange: after the three exchange steps each
// lane carries one of the 8 values (which one is given by lane bits 5, 4, 3), after three more
// butterfly steps lanes with (lane & 7) == 0 hold the full sum of value
// 4 * bit5 + 2 * bit4 + bit3.  10 shuffles instead of 48, in a fixed order.
__device__ inline float reduce8_scatter(const float (&acc)[8], int lane) {
    const bool b5 = (lane & 32) != 0, b4 = (lane & 16) != 0, b3 = (lane & 8) != 0;
    float v4[4], v2[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float keep = b5 ? acc[4 + i] : acc[i];
        const float give = b5 ? acc[i] : acc[4 + i];
        v4[i] = keep + __shfl_xor(give, 32, 64);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = b4 ? v4[2 + i] : v4[i];
        const float give = b4 ? v4[i] : v4[2 + i];
        v2[i] = keep + __shfl_xor(give, 16, 64);
    }
    const float keep = b3 ? v2[1] : v2[0];
    const float give = b3 ? v2[0] : v2[1];
    float v = keep + __shfl_xor(give, 8, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 1, 64);
    return v;
}

// bf16 logits on the matrix cores: the tokens are the 16 rows of an MFMA, 16 experts its columns, and the 8 wavefronts split the hidden
// dimension in interleaved units of 64 elements.  All loads of up to 8 units are requested before the first one is used, so 16 experts cost
// one memory round trip whatever the number of tokens.  A load covers 8 rows x 128 bytes, consecutive lanes on consecutive addresses,
// and each wavefront turns its units in 4 KB of LDS of its own (see route_mfma_kernel).  The loads go through buffer descriptors that end
// with the operands: rows and units that do not exist read as zeros and cost nothing in the vector cache.  Eight sums, added in a tree, keep
// the MFMAs apart and the result as close to the exact one as the sums of vector lanes.
// Layer calls of a few tokens, vector lanes two tokens and eight experts a round trip / so: Mixtral shape, 16 tokens 416 / 404 us, 8 tokens
// 405 / 401; Phi shape, 8 tokens 128 / 119; 64 experts of hidden 2048, ffn 1408, 3 tokens 85 / 69, 12 tokens 241 / 187.
typedef __attribute__((ext_vector_type(8))) __bf16 route_bf16x8;
typedef __attribute__((ext_vector_type(4))) float route_f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t route_u32x4;

// (beyond, 32-bit offsets do not reach 64 rows)
constexpr int kRouteMfmaMaxHidden = 1 << 24;
__host__ __device__ inline bool route_on_mfma(int H) { return H <= kRouteMfmaMaxHidden; }
// One or two tokens and up to eight experts are a single pass on the vector lanes, which is faster.
__host__ __device__ inline bool decode_routes_on_mfma(int T, int H, int E) { return (T > 2 || E > 8) && route_on_mfma(H); }
constexpr int kRouteTurnBytes = 8 * 4096;

__device__ inline void route_wave_order() {  // a wavefront's LDS accesses stay in order (for the compiler; the hardware keeps it)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Units u0, u0 + 8, ... (UNITS of them).  xoff / woff: byte offset of this lane's piece of the first 8 rows in unit 0.
template <int UNITS>
__device__ __attribute__((always_inline)) inline void logits_chunk(__amdgpu_buffer_rsrc_t x, __amdgpu_buffer_rsrc_t w, uint32_t xoff, uint32_t woff,
                                                                   uint32_t rows8, int u0, int n_units, unsigned char* mine, route_f32x4 (&acc)[8]) {
    const int lane = threadIdx.x & 63, row = lane >> 3, piece = lane & 7;
    route_u32x4 v[UNITS][4];  // x rows 0 to 7, 8 to 15, w rows 0 to 7, 8 to 15
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
        const int u = u0 + 8 * i;
        const uint32_t at = (uint32_t)u * 128u;
        const bool on = u < n_units;
        v[i][2] = __builtin_amdgcn_raw_buffer_load_b128(w, on ? woff + at : ~15u, 0, 0);
        v[i][3] = __builtin_amdgcn_raw_buffer_load_b128(w, on ? woff + rows8 + at : ~15u, 0, 0);
        v[i][0] = __builtin_amdgcn_raw_buffer_load_b128(x, on ? xoff + at : ~15u, 0, 0);
        v[i][1] = __builtin_amdgcn_raw_buffer_load_b128(x, on ? xoff + rows8 + at : ~15u, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // piece p of row r stands at position p ^ (r / 2 % 8) of its 128 bytes
    const int put_lo = row * 128 + ((piece ^ (row >> 1)) << 4), put_hi = (row + 8) * 128 + ((piece ^ (4 + (row >> 1))) << 4);
    const int get = (lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) << 4);
#pragma unroll
    for (int i = 0; i < UNITS; ++i) {
        *reinterpret_cast<route_u32x4*>(mine + put_lo) = v[i][0];
        *reinterpret_cast<route_u32x4*>(mine + put_hi) = v[i][1];
        *reinterpret_cast<route_u32x4*>(mine + 2048 + put_lo) = v[i][2];
        *reinterpret_cast<route_u32x4*>(mine + 2048 + put_hi) = v[i][3];
        route_wave_order();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const route_u32x4 a = *reinterpret_cast<const route_u32x4*>(mine + (get ^ (h * 64)));
            const route_u32x4 b = *reinterpret_cast<const route_u32x4*>(mine + 2048 + (get ^ (h * 64)));
            route_f32x4& sum = acc[(2 * i + h) & 7];
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(route_bf16x8, a), __builtin_bit_cast(route_bf16x8, b), sum, 0, 0, 0);
        }
        route_wave_order();
    }
}

// part[(wave * blocks + b) * 256 + 4 * lane + r]: expert 16 b + lane % 16, token 4 * (lane / 16) + r.
__device__ __attribute__((always_inline)) inline void partial_logits_mfma(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg, int T, int H,
                                                                          int E, float* part, unsigned char* turn) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t row_bytes = (uint32_t)H * 2u, off = (uint32_t)(lane >> 3) * row_bytes + (uint32_t)(lane & 7) * 16u;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x), 0, (int)((uint32_t)T * row_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(wg), 0, (int)((uint32_t)E * row_bytes), 0x00020000);
    const int n_units = H / 64, blocks = (E + 15) / 16;
    for (int b = 0; b < blocks; ++b) {
        route_f32x4 acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = route_f32x4{0.f, 0.f, 0.f, 0.f};
        for (int u0 = wave; u0 < n_units; u0 += 64) {
            const uint32_t woff = off + (uint32_t)b * 16u * row_bytes;
            if (n_units - u0 > 32) logits_chunk<8>(xr, wr, off, woff, 8u * row_bytes, u0, n_units, turn + wave * 4096, acc);
            else logits_chunk<4>(xr, wr, off, woff, 8u * row_bytes, u0, n_units, turn + wave * 4096, acc);
        }
        route_f32x4 sum;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            sum[r] = ((acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r])) + ((acc[4][r] + acc[5][r]) + (acc[6][r] + acc[7][r]));
        *reinterpret_cast<route_f32x4*>(part + (size_t)(wave * blocks + b) * 256 + lane * 4) = sum;
    }
}

// Routes tokens 0..T (T <= 16) against one gate; every thread of the 512-thread workgroup calls
// it.  On return (after a workgroup barrier) sm.idx[t*k + j] / sm.w[t*k + j] hold expert and
// renormalised weight of selection j of token t, in descending probability, ties to the lower
// index.  The arithmetic depends only on (T, H, E, k), never on the workgroup, so any number of
// workgroups computing the same call agree bit for bit.  `part` is kRoutePartFloats of LDS.
// `turn` (kRouteTurnBytes of LDS): bf16 on the matrix cores; null: on the vector lanes.  With `on_gpu` (uint8 [E]) the selection
// is degraded gracefully, see select_topk_lanes.
//
// With `turn`: partial_logits_mfma().  Else the 8 wavefronts split the hidden dimension in interleaved 512-element chunks, so the
// gate and x are read once per workgroup whatever T is; a wavefront walks the tokens two at a time over
// its chunks (the gate pieces of later tokens come from the vector cache).  Per-wavefront partial
// logits are summed through LDS in a fixed order; the softmax and the k arg-max passes run
// across the lanes of one wavefront, lane e holding expert e.
template <typename scalar_t>
__device__ __attribute__((always_inline)) inline void route_tokens_wg(const scalar_t* __restrict__ x, const scalar_t* __restrict__ wg,
                                       const float* __restrict__ bias, int T, int H, int E, int k, RouteSmem& sm,
                                       float* part, unsigned char* turn, const uint8_t* __restrict__ on_gpu = nullptr) {
    const bool on_mfma = turn != nullptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // requested first so that it arrives together with the gate rows
    const float my_bias = (bias != nullptr && lane < E) ? bias[lane] : 0.f;
    const bool resident = on_gpu != nullptr && lane < E && on_gpu[lane] != 0;
    if constexpr (sizeof(scalar_t) == 2)
        if (on_mfma) partial_logits_mfma(x, wg, T, H, E, part, turn);
    if (!on_mfma) {
        const int n_blocks = (E + 7) / 8;
        const int esub = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
        for (int t = 0; t < T; t += 2) {
            const bool two = t + 1 < T;
            const scalar_t* x0 = x + (size_t)t * H;
            const scalar_t* x1 = x + (size_t)(two ? t + 1 : t) * H;
            for (int eb = 0; eb < n_blocks; ++eb) {
                const int ne = min(8, E - eb * 8);
                const scalar_t* wrow = wg + (size_t)eb * 8 * H;
                float acc0[8], acc1[8];
    #pragma unroll
                for (int r = 0; r < 8; ++r) acc0[r] = acc1[r] = 0.f;
                for (int h = (wave * 64 + lane) * 8; h < H; h += 8 * 512) {
                    // All loads of the step first, unconditionally (rows past the last expert re-read it;
                    // their sums are never looked at), and nothing else scheduled between them: a load
                    // under a branch, or one the scheduler leaves next to its use, costs a memory round
                    // trip of its own, ten in a row instead of one.
                    Raw8<scalar_t> xr0, xr1, wr[8];
                    xr0.load(x0 + h);
                    xr1.load(x1 + h);
    #pragma unroll
                    for (int r = 0; r < 8; ++r) wr[r].load(wrow + (size_t)min(r, ne - 1) * H + h);
                    __builtin_amdgcn_sched_barrier(0);
                    float xv0[8], xv1[8];
                    xr0.get(xv0);
                    xr1.get(xv1);
    #pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        float wv[8];
                        wr[r].get(wv);
    #pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            acc0[r] = fmaf(xv0[i], wv[i], acc0[r]);
                            acc1[r] = fmaf(xv1[i], wv[i], acc1[r]);
                        }
                    }
                }
                const float v0 = reduce8_scatter(acc0, lane);
                const float v1 = reduce8_scatter(acc1, lane);
                if ((lane & 7) == 0) {
                    part[(wave * T + t) * 64 + eb * 8 + esub] = v0;
                    if (two) part[(wave * T + t + 1) * 64 + eb * 8 + esub] = v1;
                }
            }
        }
    }
    __syncthreads();
    for (int t = wave; t < T; t += 8) {
        float z = -INFINITY;
        if (lane < E) {
            if (on_mfma) {
                const int blocks = (E + 15) / 16;
                float v[8];
#pragma unroll
                for (int w = 0; w < 8; ++w) v[w] = part[(w * blocks + (lane >> 4)) * 256 + ((t >> 2) * 16 + (lane & 15)) * 4 + (t & 3)];
                z = (((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]))) + my_bias;
            } else {
                float s = 0.f;
                for (int w = 0; w < 8; ++w) s += part[(w * T + t) * 64 + lane];
                z = s + my_bias;
            }
        }
        int my_sel;
        float my_w;
        select_topk_lanes(z, lane, E, k, my_sel, my_w, on_gpu != nullptr, resident);
        if (lane < k) {
            sm.idx[t * k + lane] = my_sel;
            sm.w[t * k + lane] = my_w;
        }
    }
    __syncthreads();
}

}  // namespace moe
