// Gating function, softmax, top-k selection and selection histograms
// (DAOP paper Sec. II-A "MoE Structure"; activity counts of Sec. IV-B /
// Algorithm 1; next-layer prediction of Sec. III observation 3 / Sec. IV-C,
// which is the same computation with the next layer's gate on the same x).
//
// Prefill-size calls: a 16-token x 16-expert MFMA tile per workgroup and gate with the hidden dimension split
// over 16 wavefronts (route_mfma_kernel).
//
// Decode-size calls (at most 16 tokens) are a chain of memory latencies rather
// than a stream: one workgroup routes the whole call with the hidden dimension
// split over its wavefronts (route_device.h) and writes the counts itself.
#include <type_traits>

#include "moe_internal.h"
#include "route_device.h"

namespace moe {
namespace {

struct RouteParams {
    const void* x;
    int tokens, hidden, n_experts, top_k, n_gates;
    GateArgs gate[2];
    int32_t* counts;       // decode-size calls only
    int32_t* counts_next;  // decode-size calls only
    int accumulate;
};

// The gate GEMM on the matrix cores.  One workgroup of 16 wavefronts owns 16 tokens: they
// are the 16 rows of an MFMA whose 16 columns are a block of 16 experts, and the wavefronts split the hidden
// dimension in contiguous runs of 64-byte steps, 16 bytes a lane: one v_mfma_f32_16x16x32_bf16, or for fp32 storage
// four v_mfma_f32_16x16x4_f32, element q of every lane's four going to the q-th (the same K elements in both operands).
// The wavefronts' partial 16 x 16 tiles are summed through LDS in a fixed order; then wavefront i takes token i with
// expert e on lane e for the softmax and the top-k.
//
// At these sizes (a gate of 64 to 512 KB, 16 tokens a workgroup) the kernel is a chain of latencies, so every load of
// up to kChunk steps is requested before the first one is used, and unconditionally: rows that do not exist re-read one that
// does (a load under a branch waits for its own memory round trip).  There is a version for every number of steps, so that a
// wavefront of a short hidden dimension asks for no step twice (all eight always, one gate, 8 experts: hidden 512 11.7 -> 6.9 us,
// 2048 11.7 -> 9.1) and addresses are constants from the row's start (with an address a step, 64 experts spilled registers:
// hidden 2048, 1003 tokens 19.3 -> 16.2 us; fp32 with 64 experts has registers for one step only, hidden 1024 21.0 -> 17.0).
// The two gates of a call go to different workgroups (x comes from the L2 the second time) while those fit the chip at one a CU, and
// are done one after the other by the same workgroup beyond that (4096 tokens: 23 us so, 27 us in two rounds).
// Measured, both gates: 1003 tokens, 64 experts, hidden 2048: 28 -> 17 us; 32 and 77 tokens, 8 experts, hidden 4096:
// 17 -> 12 us; fp32, 512 tokens, 64 experts, hidden 1024: 208 -> 20 us (a wavefront per token read the whole gate).
// NBG = number of 16-expert blocks.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// acc[q] += a . b over a step.  fp32 storage keeps the four element positions apart until the end, and adds partial sums in
// a tree: one running sum was 1.2 to 1.6 times as far from the 64-bit gate weights as lanes with 8-element sums of
// their own had been (1.77e-7 against 1.13e-7 at a hidden dimension of 1024), this is no further than those.
__device__ inline void mfma_step(u32x4 a, u32x4 b, f32x4 (&acc)[1]) {
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc[0], 0, 0, 0);
}
__device__ inline void mfma_step(u32x4 a, u32x4 b, f32x4 (&acc)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[q]), __uint_as_float(b[q]), acc[q], 0, 0, 0);
}
__device__ inline f32x4 total_of(const f32x4 (&acc)[1]) { return acc[0]; }
__device__ inline f32x4 total_of(const f32x4 (&acc)[4]) {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
    return r;
}
// f(n) with n, at most N, as a constant.
template <int N, class F>
__device__ inline void for_count(int n, F f) {
    if (n == N) f(std::integral_constant<int, N>{});
    else if constexpr (N > 1) for_count<N - 1>(n, f);
}

template <typename scalar_t, int NBG>
__global__ __launch_bounds__(1024) void route_mfma_kernel(RouteParams p) {
    constexpr bool kF32 = sizeof(scalar_t) == 4;
    constexpr int kSums = kF32 ? 4 : 1;
    constexpr int kChunk = NBG == 1 ? 8 : NBG == 4 && kF32 ? 1 : 4;  // steps whose operands are in registers at a time
    constexpr int kStep = 64 / (int)sizeof(scalar_t), kLane = 16 / (int)sizeof(scalar_t);
    __shared__ int hist[2][64];
    __shared__ f32x4 part[16][NBG][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 128) hist[tid >> 6][tid & 63] = 0;
    const int H = p.hidden, E = p.n_experts, T = p.tokens;
    const int t0 = blockIdx.x * kRouteTokensPerBlock;
    const int row = lane & 15, kq = lane >> 4;
    const scalar_t* xrow = static_cast<const scalar_t*>(p.x) + (size_t)min(t0 + row, T - 1) * H + kq * kLane;
    const int k_steps = H / kStep;
    const int per = (k_steps + 15) / 16;
    const int s_begin = wave * per;
    const int s_end = min(k_steps, s_begin + per);

    const int t = t0 + wave;  // the token this wavefront selects for
    const int g_begin = gridDim.y > 1 ? blockIdx.y : 0, g_end = gridDim.y > 1 ? blockIdx.y + 1 : p.n_gates;
    for (int g = g_begin; g < g_end; ++g) {
        const GateArgs gate = p.gate[g];
        const float my_bias = gate.bias != nullptr && lane < E ? gate.bias[lane] : 0.f;
        const scalar_t* wrow[NBG];  // columns past the last expert compute a logit that nobody reads
#pragma unroll
        for (int nb = 0; nb < NBG; ++nb) wrow[nb] = static_cast<const scalar_t*>(gate.w) + (size_t)min(nb * 16 + row, E - 1) * H + kq * kLane;

        f32x4 acc[NBG][kSums];
#pragma unroll
        for (int nb = 0; nb < NBG; ++nb)
#pragma unroll
            for (int q = 0; q < kSums; ++q) acc[nb][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto steps = [&](auto n_c, int s0) {
            constexpr int N = decltype(n_c)::value;
            u32x4 xa[N], wb[NBG][N];
            const scalar_t* xs = xrow + (size_t)s0 * kStep;
#pragma unroll
            for (int i = 0; i < N; ++i) xa[i] = *reinterpret_cast<const u32x4*>(xs + i * kStep);
#pragma unroll
            for (int nb = 0; nb < NBG; ++nb) {
                const scalar_t* ws = wrow[nb] + (size_t)s0 * kStep;
#pragma unroll
                for (int i = 0; i < N; ++i) wb[nb][i] = *reinterpret_cast<const u32x4*>(ws + i * kStep);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int nb = 0; nb < NBG; ++nb) mfma_step(xa[i], wb[nb][i], acc[nb]);
        };
        for (int s0 = s_begin; s0 < s_end; s0 += kChunk) {
            for_count<kChunk>(min(kChunk, s_end - s0), [&](auto n) { steps(n, s0); });
        }

        // MFMA result: lane holds column (expert in block) lane & 15 and rows (tokens) 4 * (lane / 16) + r.
        if (g > g_begin) __syncthreads();  // the previous gate's partial tiles have been read
#pragma unroll
        for (int nb = 0; nb < NBG; ++nb) part[wave][nb][lane] = total_of(acc[nb]);
        __syncthreads();
        if (t < T) {
            float z = -INFINITY;
            if (lane < E) {
                const int nb = lane >> 4, src = (wave >> 2) * 16 + (lane & 15), r = wave & 3;
                float v[16];
#pragma unroll
                for (int w = 0; w < 16; ++w) v[w] = part[w][nb][src][r];
                if constexpr (kF32) {
#pragma unroll
                    for (int d = 8; d > 0; d /= 2)
#pragma unroll
                        for (int w = 0; w < d; ++w) v[w] += v[w + d];
                } else {
#pragma unroll
                    for (int w = 1; w < 16; ++w) v[0] += v[w];
                }
                z = v[0] + my_bias;
            }
            int my_sel;
            float my_w;
            select_topk_lanes(z, lane, E, p.top_k, my_sel, my_w);
            if (lane < p.top_k) {
                gate.idx[(size_t)t * p.top_k + lane] = my_sel;
                if (gate.wts != nullptr) gate.wts[(size_t)t * p.top_k + lane] = my_w;
                atomicAdd(&hist[g][my_sel], 1);
            }
        }
    }
    __syncthreads();
    if (tid < E)
        for (int g = g_begin; g < g_end; ++g)
            if (p.gate[g].hist != nullptr) p.gate[g].hist[(size_t)blockIdx.x * E + tid] = hist[g][tid];
}

// One workgroup routes a decode-size call against up to two gates and writes indices, weights
// and counts.
template <typename scalar_t>
__global__ __launch_bounds__(kSmallRouteThreads) void route_small_kernel(RouteParams p) {
    __shared__ RouteSmem sm;
    __shared__ float part[kRoutePartFloats];
    const int tid = threadIdx.x;
    const int E = p.n_experts, A = p.tokens * p.top_k;
    int old_count = 0;  // requested before the gate rows so that its latency is hidden
    if (tid < E && p.accumulate && p.counts != nullptr) old_count = p.counts[tid];
    for (int g = 0; g < p.n_gates; ++g) {
        route_tokens_wg<scalar_t>(static_cast<const scalar_t*>(p.x), static_cast<const scalar_t*>(p.gate[g].w),
                                  p.gate[g].bias, p.tokens, p.hidden, E, p.top_k, sm, part,
                                  sizeof(scalar_t) == 2 && route_on_mfma(p.tokens, p.hidden));
        if (tid < A) {
            p.gate[g].idx[tid] = sm.idx[tid];
            if (p.gate[g].wts != nullptr) p.gate[g].wts[tid] = sm.w[tid];
        }
        int32_t* counts = g == 0 ? p.counts : p.counts_next;
        if (tid < E && counts != nullptr) {
            int c = 0;
            for (int a = 0; a < A; ++a) c += sm.idx[a] == tid;
            counts[tid] = (g == 0 ? old_count : 0) + c;
        }
        __syncthreads();  // sm is reused by the next gate
    }
}

template <typename scalar_t>
void launch_mfma(const RouteParams& p, hipStream_t stream) {
    const int blocks = route_blocks(p.tokens);
    const dim3 grid(blocks, blocks * p.n_gates <= compute_units() ? p.n_gates : 1);
    if (p.n_experts <= 16) route_mfma_kernel<scalar_t, 1><<<grid, 1024, 0, stream>>>(p);
    else if (p.n_experts <= 32) route_mfma_kernel<scalar_t, 2><<<grid, 1024, 0, stream>>>(p);
    else route_mfma_kernel<scalar_t, 4><<<grid, 1024, 0, stream>>>(p);
}

RouteParams make_params(const moe_shape_t& s, int tokens, const void* x, const GateArgs* gates, int n_gates) {
    RouteParams p{};
    p.x = x;
    p.tokens = tokens;
    p.hidden = s.hidden;
    p.n_experts = s.n_experts;
    p.top_k = s.top_k;
    p.n_gates = n_gates;
    for (int g = 0; g < n_gates; ++g) p.gate[g] = gates[g];
    return p;
}

}  // namespace

hipError_t launch_route(const moe_shape_t& s, int tokens, const void* x, const GateArgs* gates, int n_gates,
                        hipStream_t stream) {
    RouteParams p = make_params(s, tokens, x, gates, n_gates);
    if (s.dtype == MOE_F32) launch_mfma<float>(p, stream);
    else launch_mfma<uint16_t>(p, stream);
    return hipGetLastError();
}

hipError_t launch_route_small(const moe_shape_t& s, int tokens, const void* x, const GateArgs* gates,
                              int n_gates, int32_t* counts, int accumulate, int32_t* counts_next,
                              hipStream_t stream) {
    RouteParams p = make_params(s, tokens, x, gates, n_gates);
    p.counts = counts;
    p.counts_next = counts_next;
    p.accumulate = accumulate;
    if (s.dtype == MOE_F32) route_small_kernel<float><<<1, kSmallRouteThreads, 0, stream>>>(p);
    else route_small_kernel<uint16_t><<<1, kSmallRouteThreads, 0, stream>>>(p);
    return hipGetLastError();
}

}  // namespace moe
