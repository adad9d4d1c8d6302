// Gating function, softmax, top-k selection and selection histograms
// (DAOP paper Sec. II-A "MoE Structure"; activity counts of Sec. IV-B /
// Algorithm 1; next-layer prediction of Sec. III observation 3 / Sec. IV-C,
// which is the same computation with the next layer's gate on the same x).
//
// Prefill-size calls: a 16-token x 16-expert MFMA tile per workgroup and gate with the hidden dimension split
// over its wavefronts (route_mfma_kernel).
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
    int accumulate;
    RouteFinish finish;    // words == null: left to other kernels
};

// The gate GEMM on the matrix cores.  One workgroup owns 16 tokens: they
// are the 16 rows of an MFMA whose 16 columns are a block of 16 experts, and the wavefronts split the hidden
// dimension in contiguous runs of 128-byte units, two MFMA steps each, 16 bytes a lane: one v_mfma_f32_16x16x32_bf16, or for fp32 storage
// four v_mfma_f32_16x16x4_f32, element q of every lane's four going to the q-th (the same K elements in both operands).
// A load instruction covers 8 rows x 128 bytes, consecutive lanes on consecutive addresses, and each wavefront turns its units in 4 KB of
// LDS of its own: in the layout that the MFMA wants, every quad of lanes is on four rows, which costs the address path 64 cycles an
// instruction instead of 16 (kernel, 2048 tokens of hidden 4096, 16 experts 11.4 -> 6.8 us; 77 tokens 9.6 -> 7.6; 1003 tokens of hidden
// 2048, 64 experts 14.4 -> 11.4).
// The wavefronts' partial 16 x 16 tiles are summed through LDS in a fixed order; then each token is one wavefront's, with
// expert e on lane e for the softmax and the top-k.
//
// At these sizes (a gate of 64 to 512 KB, 16 tokens a workgroup) the kernel is a chain of latencies, so every load of
// up to kChunk units is requested before the first one is used, and unconditionally: rows that do not exist re-read one that
// does (a load under a branch waits for its own memory round trip).  There is a version for every number of units, so that a
// wavefront of a short hidden dimension asks for no unit twice, and addresses are constants from the row's start (with an address a
// step, 64 experts spilled registers; fp32 with 64 experts has registers for one unit only).
// The two gates of a call go to different workgroups (x comes from the L2 the second time) while those fit the chip at one a CU, and
// are done one after the other by the same workgroup beyond that (whole layer of hidden 4096, ffn 64, 8 experts, 4096 tokens 116.6 us so,
// 117.7 with different workgroups; hidden 2048, 64 experts, 2500 tokens 83.8 / 84.8).
// NBG = number of 16-expert blocks.  SHARERS: where more than 32 experts meet a hidden dimension of at most four units, a wavefront makes one
// unit for NBG / SHARERS of the blocks.  (A wavefront's chain of blocks, each through LDS and in fp32 eight MFMAs a step, is what such a
// call waits for while other wavefronts have no unit.  moe_route, 64 experts top-6, 200 tokens, a unit a wavefront / shared: fp32, hidden 64
// 9.0 / 8.4 us, 128 top-4, 100 tokens 8.0 / 7.9; bf16, hidden 64 8.3 / 8.1, 192 top-4, 100 tokens 7.3 / 7.2; with 17 to 32 experts a chain is two
// blocks, and sharing is no faster: fp32, hidden 64 7.1 / 7.1, bf16, hidden 256 7.0 / 7.1.)
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// acc += a . b over step h of a unit.  fp32 storage keeps the four element positions of the two steps apart until the end, and adds partial
// sums in a tree: one running sum was 1.2 to 1.6 times as far from the 64-bit gate weights as lanes with 8-element sums of
// their own had been (1.77e-7 against 1.13e-7 at a hidden dimension of 1024), this is no further than those.
__device__ inline void mfma_step(u32x4 a, u32x4 b, int, f32x4 (&acc)[1]) {
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc[0], 0, 0, 0);
}
__device__ inline void mfma_step(u32x4 a, u32x4 b, int h, f32x4 (&acc)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc[h * 4 + q] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[q]), __uint_as_float(b[q]), acc[h * 4 + q], 0, 0, 0);
}
__device__ inline f32x4 total_of(const f32x4 (&acc)[1]) { return acc[0]; }
__device__ inline f32x4 total_of(const f32x4 (&acc)[8]) {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r[i] = ((acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i])) + ((acc[4][i] + acc[5][i]) + (acc[6][i] + acc[7][i]));
    return r;
}
// f(n) with n, at most N, as a constant.
template <int N, class F>
__device__ inline void for_count(int n, F f) {
    if (n == N) f(std::integral_constant<int, N>{});
    else if constexpr (N > 1) for_count<N - 1>(n, f);
}

// Orders a wavefront's own LDS traffic (which the hardware does by itself; this is for the compiler).
__device__ inline void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Wavefronts: 16, or 8 for more than 16 experts, which then have registers for four units (two in fp32 with 64 experts).
template <int NBG>
constexpr int kRouteWaves = NBG == 1 ? 16 : 8;

// ---- Counts and permutation by the workgroup that ends last, instead of another launch.
// Every workgroup of the first gate stores its histogram in `words`, a tag with each count, and then looks whether all workgroups' words are
// there.  A store is acknowledged before its workgroup looks, so the last one to store finds them all, and nobody waits for
// anybody.  If several do, the one that takes the first word away goes on.  It leaves all words cleared, so that no word of a call is
// ever there before that call has stored it; other contents of the memory equal a tag of 56 bits only by accident.
//
// The workgroup's 2 us for the counts are less than a launch of 2 us and the gap before it, and less for the host (moe_route and
// moe_predict_next, 2048 tokens, 16 experts 23.6 -> 19.5 us).  The permutation is one pass of 16 wavefronts up to 1024
// selections: fp32, hidden 256, 64 tokens 25.9 -> 23.0 us, 500 tokens 37.1 -> 36.7; bf16, 1024 by 1024, 500 tokens 53.5 -> 53.0, Mixtral shape
// 512 tokens 606.7 -> 604.1.  More passes, or 8 wavefronts of more than 16 experts, are no faster than workgroups that share it:
// 2048 selections 773.6 -> 778.1, 64 experts, 1800 selections 251.8 -> 254.2, fp32 179.2 -> 182.3.
//
// Every workgroup reads all words, so the time grows with their number and with that of the workgroups.  Up to 3072 words and 256 workgroups
// (what the chip holds at one a CU) a call that waits for the host gains up to 3 us and one that does not is as fast as with another launch;
// beyond, it loses.  moe_route in us, another launch / so, replayed from a graph and called in a row: 8 experts, hidden 4096, 2048 tokens 9.6 / 9.7 and 12.5 / 9.7,
// 4096 tokens 12.5 / 12.8 and 12.6 / 12.6, 8192 tokens 21.7 / 23.9, 16384 tokens 38.2 / 49.8; 16 experts, 3000 tokens 11.9 / 11.4 and 12.0 / 11.2, 4096 tokens
// 13.6 / 14.0 and 13.6 / 13.7; 32 experts, hidden 2048, 1500 tokens 10.8 / 11.0 and 12.0 / 11.0, 2048 tokens 10.8 / 12.1; 64 experts, 500 tokens 12.1 / 12.3 and
// 12.8 / 12.5, 1000 tokens 13.0 / 13.8, 2048 tokens 14.3 / 17.4; fp32, 8 experts, hidden 1024, 4096 tokens 9.9 / 10.3 and 11.8 / 10.1, 8192 tokens 16.7 / 20.2.
constexpr uint64_t kWordTag = 0x9E3779B97F4A7Cull << 8;
constexpr int kFinishMaxWords = 3072, kFinishMaxBlocks = 256, kFinishMaxSelections = 1024, kFinishMaxExperts = 16;

template <int WAVES>
__device__ inline void finish_routing(const RouteFinish& f, const int32_t* idx, int n_blocks, int E, int A, const int* hist) {
    __shared__ int total[64], base[64], count[WAVES][64];
    __shared__ int won;
    constexpr int kThreads = WAVES * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 64) total[tid] = 0;
    if (tid < E)
        __hip_atomic_store(&f.words[(size_t)blockIdx.x * E + tid], kWordTag | (uint64_t)hist[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int n = n_blocks * E;
    bool all = true;
    for (int i = tid; i < n; i += kThreads) {
        const uint64_t w = __hip_atomic_load(&f.words[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        all &= (w & ~(uint64_t)255) == kWordTag;
        if ((w & 255) != 0) atomicAdd(&total[i % E], (int)(w & 255));  // (of no use unless all words are there)
    }
    if (!__syncthreads_and(all)) return;
    if (tid == 0) won = (__hip_atomic_exchange(&f.words[0], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~(uint64_t)255) == kWordTag;
    __syncthreads();
    if (!won) return;
    for (int i = tid; i < n; i += kThreads) f.words[i] = 0;
    if (f.counts != nullptr && tid < E) f.counts[tid] = (f.accumulate ? f.counts[tid] : 0) + total[tid];
    if (WAVES != 16 || f.row_of_slot == nullptr) return;  // (route_finishes())
    static_assert(kFinishMaxSelections <= 1024 && kFinishMaxExperts <= 16, "a thread a selection, four bits an expert");
    for (int i = tid; i < kSyncInts; i += kThreads) f.sync[i] = 0;
    if (tid < 64) {
        const int mine = tid < E ? total[tid] : 0;
        int end = mine;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
            const int u = __shfl_up(end, d, 64);
            if (lane >= d) end += u;
        }
        base[tid] = end - mine;
        if (tid < E) f.offs[tid] = end - mine;
        if (tid == E - 1) f.offs[E] = end;
    }
    // A thread a selection: slot = base of the expert + those of the same expert before it, in the wavefront from four ballots (one
    // per bit of the expert's number), in the wavefronts before it from their counts.
    const bool on = tid < A;
    const int e = on ? __hip_atomic_load(&idx[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    uint64_t same = __ballot(on);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const bool bit = ((e >> b) & 1) != 0;
        const uint64_t m = __ballot(bit);
        same &= bit ? m : ~m;
    }
    const int before = __popcll(same & ((1ull << lane) - 1ull));
    count[wave][lane] = 0;
    wave_order();
    if (on && before == 0) count[wave][e] = __popcll(same);
    __syncthreads();
    if (on) {
        int slot = base[e] + before;
        for (int w = 0; w < wave; ++w) slot += count[w][e];
        f.slot_of[tid] = slot;
        f.row_of_slot[slot] = tid;
    }
}

// Adds the products of N units with NB blocks of experts, requested together.  x, w: lane l's piece of rows l / 8 (lo) and 8 + l / 8 (hi) of
// the first unit, piece l % 8, which goes to position (l % 8) ^ (row / 2 % 8) of the row in `mine` (4 KB); operands: row l % 16, piece l / 16
// (+ 4 for the second step).
template <int N, typename scalar_t, int NB, int SUMS>
__device__ __attribute__((always_inline)) inline void add_units(const scalar_t* x_lo, const scalar_t* x_hi, const scalar_t* const (&w_lo)[NB],
                                                                const scalar_t* const (&w_hi)[NB], size_t off, unsigned char* mine,
                                                                f32x4 (&acc)[NB][SUMS]) {
    constexpr int kUnit = 128 / (int)sizeof(scalar_t);
    const int lane = threadIdx.x & 63, row = lane >> 3, piece = lane & 7;
    const int put_lo = row * 128 + ((piece ^ (row >> 1)) << 4), put_hi = (row + 8) * 128 + ((piece ^ (4 + (row >> 1))) << 4);
    const int get = (lane & 15) * 128 + (((lane >> 4) ^ ((lane >> 1) & 7)) << 4);  // (second step: ^ 64)
    u32x4 xl[N], xh[N], wl[NB][N], wh[NB][N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        xl[i] = *reinterpret_cast<const u32x4*>(x_lo + off + i * kUnit);
        xh[i] = *reinterpret_cast<const u32x4*>(x_hi + off + i * kUnit);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            wl[nb][i] = *reinterpret_cast<const u32x4*>(w_lo[nb] + off + i * kUnit);
            wh[nb][i] = *reinterpret_cast<const u32x4*>(w_hi[nb] + off + i * kUnit);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        *reinterpret_cast<u32x4*>(mine + put_lo) = xl[i];
        *reinterpret_cast<u32x4*>(mine + put_hi) = xh[i];
        u32x4 xa[2];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            *reinterpret_cast<u32x4*>(mine + 2048 + put_lo) = wl[nb][i];
            *reinterpret_cast<u32x4*>(mine + 2048 + put_hi) = wh[nb][i];
            wave_order();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (nb == 0) xa[h] = *reinterpret_cast<const u32x4*>(mine + (get ^ (h * 64)));
                mfma_step(xa[h], *reinterpret_cast<const u32x4*>(mine + 2048 + (get ^ (h * 64))), h, acc[nb]);
            }
            wave_order();
        }
    }
}

template <typename scalar_t, int NBG, int SHARERS>
__global__ __launch_bounds__(kRouteWaves<NBG> * 64) void route_mfma_kernel(RouteParams p) {
    constexpr bool kF32 = sizeof(scalar_t) == 4;
    constexpr int kSums = kF32 ? 8 : 1, kWaves = kRouteWaves<NBG>;
    constexpr int kChunk = !kF32 || NBG == 2 ? 4 : NBG == 1 ? 2 : 1;  // units whose operands are in registers at a time
    constexpr int kUnit = 128 / (int)sizeof(scalar_t), kLane = 16 / (int)sizeof(scalar_t);
    __shared__ __attribute__((aligned(256))) unsigned char turn[kWaves][4096];  // per wavefront a unit of 16 tokens and of 16 experts
    __shared__ int hist[2][64];
    __shared__ f32x4 part[kWaves][NBG][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 128) hist[tid >> 6][tid & 63] = 0;
    const int H = p.hidden, E = p.n_experts, T = p.tokens;
    const int t0 = blockIdx.x * kRouteTokensPerBlock;
    const int row = lane >> 3, piece = lane & 7;  // see add_units()
    const scalar_t* x_lo = static_cast<const scalar_t*>(p.x) + (size_t)min(t0 + row, T - 1) * H + piece * kLane;
    const scalar_t* x_hi = static_cast<const scalar_t*>(p.x) + (size_t)min(t0 + row + 8, T - 1) * H + piece * kLane;
    unsigned char* mine = turn[wave];
    const int n_units = H / kUnit;
    // This wavefront's units and blocks of experts, and the partial tile that they go to.
    const int per = SHARERS > 1 ? 1 : (n_units + kWaves - 1) / kWaves;
    const int slot = wave / SHARERS, slots = SHARERS > 1 ? n_units : kWaves;
    const int u_begin = slot * per, u_end = min(n_units, u_begin + per);
    constexpr int NB = NBG / SHARERS, kChunkUnits = SHARERS > 1 ? 1 : kChunk;
    const int first = wave % SHARERS * NB;

    const int g_begin = gridDim.y > 1 ? blockIdx.y : 0, g_end = gridDim.y > 1 ? blockIdx.y + 1 : p.n_gates;
    for (int g = g_begin; g < g_end; ++g) {
        const GateArgs gate = p.gate[g];
        const float my_bias = gate.bias != nullptr && lane < E ? gate.bias[lane] : 0.f;
        // rows 16 nb + lane / 8 and 8 further on; columns past the last expert compute a logit that nobody reads
        const scalar_t *w_lo[NB], *w_hi[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            w_lo[nb] = static_cast<const scalar_t*>(gate.w) + (size_t)min((first + nb) * 16 + row, E - 1) * H + piece * kLane;
            w_hi[nb] = static_cast<const scalar_t*>(gate.w) + (size_t)min((first + nb) * 16 + row + 8, E - 1) * H + piece * kLane;
        }
        f32x4 acc[NB][kSums];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q = 0; q < kSums; ++q) acc[nb][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int u0 = u_begin; u0 < u_end; u0 += kChunkUnits)
            for_count<kChunkUnits>(min(kChunkUnits, u_end - u0), [&](auto n) {
                add_units<decltype(n)::value>(x_lo, x_hi, w_lo, w_hi, (size_t)u0 * kUnit, mine, acc);
            });

        // MFMA result: lane holds column (expert in block) lane & 15 and rows (tokens) 4 * (lane / 16) + r.
        if (g > g_begin) __syncthreads();  // the previous gate's partial tiles have been read
        if (SHARERS == 1 || slot < slots) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) part[slot][first + nb][lane] = total_of(acc[nb]);
        }
        __syncthreads();
        for (int i = wave; i < kRouteTokensPerBlock && t0 + i < T; i += kWaves) {  // token t0 + i, by one wavefront
            const int t = t0 + i;
            float z = -INFINITY;
            if (lane < E) {
                const int nb = lane >> 4, src = (i >> 2) * 16 + (lane & 15), r = i & 3;
                float v[kWaves];
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v[w] = SHARERS == 1 || w < slots ? part[w][nb][src][r] : 0.f;
                if constexpr (kF32) {
#pragma unroll
                    for (int d = kWaves / 2; d > 0; d /= 2)
#pragma unroll
                        for (int w = 0; w < d; ++w) v[w] += v[w + d];
                } else {
#pragma unroll
                    for (int w = 1; w < kWaves; ++w) v[0] += v[w];
                }
                z = v[0] + my_bias;
            }
            int my_sel;
            float my_w;
            select_topk_lanes(z, lane, E, p.top_k, my_sel, my_w);
            if (lane < p.top_k) {
                if (p.finish.words != nullptr && g == 0)  // (read by another workgroup of this launch)
                    __hip_atomic_store(&gate.idx[(size_t)t * p.top_k + lane], my_sel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else
                    gate.idx[(size_t)t * p.top_k + lane] = my_sel;
                if (gate.wts != nullptr) gate.wts[(size_t)t * p.top_k + lane] = my_w;
                atomicAdd(&hist[g][my_sel], 1);
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (p.finish.words != nullptr && g_begin == 0) finish_routing<kWaves>(p.finish, p.gate[0].idx, gridDim.x, E, T * p.top_k, hist[0]);
    if (tid < E)
        for (int g = g_begin; g < g_end; ++g)
            if (p.gate[g].hist != nullptr) p.gate[g].hist[(size_t)blockIdx.x * E + tid] = hist[g][tid];
}

// One workgroup routes a decode-size call against up to two gates and writes indices, weights
// and the first gate's counts.
template <typename scalar_t, bool MFMA>
__global__ __launch_bounds__(kSmallRouteThreads) void route_small_kernel(RouteParams p) {
    __shared__ RouteSmem sm;
    __shared__ float part[kRoutePartFloats];
    __shared__ __attribute__((aligned(256))) unsigned char turn[MFMA ? kRouteTurnBytes : 16];
    const int tid = threadIdx.x;
    const int E = p.n_experts, A = p.tokens * p.top_k;
    int old_count = 0;  // requested before the gate rows so that its latency is hidden
    if (tid < E && p.accumulate && p.counts != nullptr) old_count = p.counts[tid];
    for (int g = 0; g < p.n_gates; ++g) {
        route_tokens_wg<scalar_t>(static_cast<const scalar_t*>(p.x), static_cast<const scalar_t*>(p.gate[g].w),
                                  p.gate[g].bias, p.tokens, p.hidden, E, p.top_k, sm, part, MFMA ? turn : nullptr);
        if (tid < A) {
            p.gate[g].idx[tid] = sm.idx[tid];
            if (p.gate[g].wts != nullptr) p.gate[g].wts[tid] = sm.w[tid];
        }
        if (g == 0 && tid < E && p.counts != nullptr) {
            int c = 0;
            for (int a = 0; a < A; ++a) c += sm.idx[a] == tid;
            p.counts[tid] = old_count + c;
        }
        __syncthreads();  // sm is reused by the next gate
    }
}

template <typename scalar_t>
void launch_mfma(const RouteParams& p, hipStream_t stream) {
    const int blocks = route_blocks(p.tokens);
    const dim3 grid(blocks, blocks * p.n_gates <= compute_units() ? p.n_gates : 1);
    auto launch = [&](auto nbg, auto sharers) {
        constexpr int kBlocks = decltype(nbg)::value;
        route_mfma_kernel<scalar_t, kBlocks, decltype(sharers)::value><<<grid, kRouteWaves<kBlocks> * 64, 0, stream>>>(p);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    const int units = p.hidden / (128 / (int)sizeof(scalar_t));
    if (p.n_experts <= 16) launch(One{}, One{});
    else if (p.n_experts <= 32) launch(Two{}, One{});
    else if (units <= 2) launch(Four{}, Four{});
    else if (units <= 4) launch(Four{}, Two{});
    else launch(Four{}, One{});
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

bool route_finishes(const moe_shape_t& s, int tokens, bool permute) {
    return route_blocks(tokens) <= kFinishMaxBlocks && (int64_t)route_blocks(tokens) * s.n_experts <= kFinishMaxWords &&
           (!permute || ((int64_t)tokens * s.top_k <= kFinishMaxSelections && s.n_experts <= kFinishMaxExperts));
}

hipError_t launch_route(const moe_shape_t& s, int tokens, const void* x, const GateArgs* gates, int n_gates,
                        const RouteFinish* finish, hipStream_t stream) {
    RouteParams p = make_params(s, tokens, x, gates, n_gates);
    if (finish != nullptr) p.finish = *finish;
    if (s.dtype == MOE_F32) launch_mfma<float>(p, stream);
    else launch_mfma<uint16_t>(p, stream);
    return hipGetLastError();
}

hipError_t launch_route_small(const moe_shape_t& s, int tokens, const void* x, const GateArgs* gates,
                              int n_gates, int32_t* counts, int accumulate, hipStream_t stream) {
    RouteParams p = make_params(s, tokens, x, gates, n_gates);
    p.counts = counts;
    p.accumulate = accumulate;
    if (s.dtype == MOE_F32) route_small_kernel<float, false><<<1, kSmallRouteThreads, 0, stream>>>(p);
    else if (decode_routes_on_mfma(tokens, s.hidden, s.n_experts)) route_small_kernel<uint16_t, true><<<1, kSmallRouteThreads, 0, stream>>>(p);
    else route_small_kernel<uint16_t, false><<<1, kSmallRouteThreads, 0, stream>>>(p);
    return hipGetLastError();
}

}  // namespace moe
