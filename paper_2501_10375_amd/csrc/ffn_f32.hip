// Grouped SwiGLU expert FFN and weighted combine for fp32 storage
// (expert execution of DAOP Sec. II-A / Algorithm 1's local expert execution,
// with the Mixtral expert  y = W2 ( silu(W1 x) * (W3 x) )  the paper builds on).
//
// This is the exact-arithmetic configuration: fp32 in, fp32 accumulation, nothing narrowed.  Rows of a
// unit are gathered through the permutation and never span two experts.
//
// The sizes of this configuration are mostly small (hidden and ffn of a few hundred to a few thousand), so a call
// lasts as long as its chain of memory latencies, not as its arithmetic.  The two GEMMs are therefore
// organised to have few dependent steps (gemm_f32), with a second kernel for calls that have enough work for
// every CU (gemm_f32_alone):
//   * v_mfma_f32_16x16x4_f32: its operands are one float per lane, row lane % 16 and K element lane / 16.
//     Which four of sixteen K elements an MFMA multiplies is free as long as both operands agree, so a lane
//     loads four consecutive floats of its row (16 bytes) and feeds them to four MFMAs.  That is the layout
//     the rows have in memory: no LDS staging and no barrier in the loop.
//   * the four wavefronts of a workgroup split K; their partial sums meet in LDS once, in wavefront order.
//   * a workgroup makes 16 features of up to 16 * NC slots; NC grows with the call (see pick_groups()), so
//     that a small call is spread over the chip and a large one re-reads its operands less often.
//   * each wavefront has kAhead K steps of loads in flight.
// Measured against the LDS-tiled FMA kernels these replaced (64 x 64 outputs, K in steps of 16 between two
// barriers), first and second GEMM:
//   64 tokens, hidden 256, ffn 512, 8 experts top-2:        33 + 34 -> 9 + 7 us
//   100 tokens, hidden 512, ffn 1024, 8 experts top-2:      64 + 65 -> 21 + 13 us
//   512 tokens, hidden 1024, ffn 2048, 4 experts top-4:    262 + 185 -> 227 + 131 us, alone 154 + 93
//   2048 tokens, hidden and ffn 4096, 8 experts top-2:     3544 + 1951 -> 4119 + 1987 us, alone 2367 + 1524 (116 and 90 TFLOP/s)
// and half as far from a 64-bit layer (y: 6.0e-7 -> 3.1e-7, 1.2e-6 -> 6.0e-7 at the first and the third), because a
// running sum is a quarter as long.
#include <type_traits>

#include "moe_internal.h"

namespace moe {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 4;
constexpr int kRows = 16;    // rows of an MFMA operand
constexpr int kStepK = 16;   // K elements of a step: 16 bytes a lane
constexpr int kAhead = 4;    // steps in flight
constexpr int kPair = 2;     // steps requested together: 128 bytes of a row, a whole cache line

// Unit u of the call: up to `unit_rows` slots of one expert.  Lane e looks after expert e; every wavefront finds
// the same answer.  False if there is no such unit.
__device__ inline bool find_unit(const int32_t* __restrict__ offs, int E, int unit_rows, int u, int& e, int& slot0, int& rows) {
    const int lane = threadIdx.x & 63;
    const int first = lane < E ? offs[lane] : 0;
    const int count = lane < E ? offs[lane + 1] - first : 0;
    const int units = (count + unit_rows - 1) / unit_rows;
    int end = units;  // inclusive sum
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int v = __shfl_up(end, d, 64);
        if (lane >= d) end += v;
    }
    const uint64_t mine = __ballot(u >= end - units && u < end);
    if (mine == 0) return false;
    const int r = __ffsll((long long)mine) - 1;
    const int local = (u - __builtin_amdgcn_readlane(end - units, r)) * unit_rows;
    e = r;
    slot0 = __builtin_amdgcn_readlane(first, r) + local;
    rows = min(unit_rows, __builtin_amdgcn_readlane(count, r) - local);
    return true;
}

// Work of this workgroup.  Workgroups go to the XCDs in turn, blockIdx.x % 8; the units are cut into 8 contiguous
// chunks, and one XCD takes a chunk at one feature tile, so that units of one expert read their weight rows through the
// same L2.  Which chunk it takes moves on with the feature tile: the last ones may hold fewer units.
__device__ inline bool my_work(int tiles, int& tile, int& unit) {
    tile = blockIdx.z * gridDim.y + blockIdx.y;
    unit = (int)((blockIdx.x + blockIdx.y) & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    return tile < tiles;
}

// acc[m][c] += (16 weight rows m) . (16 rows of column group c) over `steps` K steps; w[m] and x[c] are this lane's
// first 16 bytes (row lane % 16, K element 4 * (lane / 16)).  after(i) is called behind K step i.
template <int NM, int NC, class F>
__device__ inline void dot_rows(const float* const (&w)[NM], const float* const (&x)[NC], int steps, f32x4 (&acc)[NM][NC], F after) {
    f32x4 wf[kAhead][NM], xf[kAhead][NC];
    auto load = [&](int i, int s) {
        const size_t off = (size_t)min(s, steps - 1) * kStepK;  // requests past the end re-read the last step (never used)
#pragma unroll
        for (int m = 0; m < NM; ++m) wf[i][m] = *reinterpret_cast<const f32x4*>(w[m] + off);
#pragma unroll
        for (int c = 0; c < NC; ++c) xf[i][c] = *reinterpret_cast<const f32x4*>(x[c] + off);
    };
    auto multiply = [&](int i, int s) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int m = 0; m < NM; ++m)
                    acc[m][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[i][m][q], xf[i][c][q], acc[m][c], 0, 0, 0);
        after(s);
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load(i, i);
    int s = 0;
    for (; s + kAhead < steps; s += kAhead) {
#pragma unroll
        for (int i = 0; i < kAhead; i += kPair) {
#pragma unroll
            for (int j = i; j < i + kPair; ++j) multiply(j, s + j);
#pragma unroll
            for (int j = i; j < i + kPair; ++j) load(j, s + kAhead + j);
        }
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
        if (s + i < steps) multiply(i, s + i);
}

// A workgroup makes FR * 16 features.
// NM = 2 (gemm1): dst[slot, f] = silu(x_row . wa[e, f]) * (x_row . wb[e, f]), x_row gathered through row_of_slot;
// NM = 1 (gemm2): dst[slot, n] = src[slot] . wa[e, n].
template <int NM, int FR, int NC_MAX>
__global__ __launch_bounds__(kWaves * 64) void gemm_f32(const float* __restrict__ src, const float* __restrict__ wa,
                                                        const float* __restrict__ wb, const int32_t* __restrict__ offs,
                                                        const int32_t* __restrict__ row_of_slot, int E, int k, int N, int K,
                                                        float* __restrict__ dst,
                                                        const float* __restrict__ x_stale,
                                                        const uint8_t* __restrict__ stale) {
    __shared__ f32x4 part[kWaves][NM * FR][NC_MAX][64];
    int tile, unit, e, slot0, rows;
    if (!my_work(N / (FR * kRows), tile, unit)) return;
    if (!find_unit(offs, E, NC_MAX * kRows, unit, e, slot0, rows)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = lane & 15, kq = lane >> 4;
    const int n0 = tile * FR * kRows;
    const int steps = K / kStepK / kWaves;  // K is a multiple of 64: the wavefronts take equal contiguous runs
    const size_t at = (size_t)wave * steps * kStepK + kq * 4;
    const float* w[NM * FR];
#pragma unroll
    for (int m = 0; m < NM * FR; ++m) w[m] = (m < FR ? wa : wb) + ((size_t)e * N + n0 + (m % FR) * kRows + row) * K + at;
    // the unit's column groups, as many as it has
    auto run = [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        const float* x[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int slot = slot0 + min(c * kRows + row, rows - 1);  // rows past the end re-read a valid row; never stored
            if constexpr (NM == 2) {
                const int assignment = row_of_slot[slot];  // t * k + j
                // a pre-calculated selection reads the earlier hidden state of its token
                x[c] = ((stale != nullptr && stale[assignment] != 0) ? x_stale : src) + (size_t)(assignment / k) * K + at;
            } else {
                x[c] = src + (size_t)slot * K + at;
            }
        }
        f32x4 acc[NM * FR][NC];
#pragma unroll
        for (int m = 0; m < NM * FR; ++m)
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[m][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        dot_rows<NM * FR, NC>(w, x, steps, acc, [](int) {});
#pragma unroll
        for (int m = 0; m < NM * FR; ++m)
#pragma unroll
            for (int c = 0; c < NC; ++c) part[wave][m][c][lane] = acc[m][c];
    };
    const int groups = (rows + kRows - 1) / kRows;
    if constexpr (NC_MAX >= 4) {
        if (groups == 4) run(std::integral_constant<int, 4>{});
        if (groups == 3) run(std::integral_constant<int, 3>{});
    }
    if constexpr (NC_MAX >= 2) {
        if (groups == 2) run(std::integral_constant<int, 2>{});
    }
    if (groups == 1) run(std::integral_constant<int, 1>{});
    __syncthreads();
    // MFMA result: lane holds column (slot) lane % 16 and rows (features) 4 * (lane / 16) .. + 3.  A wavefront sums one
    // 16 x 16 result at a time.
    for (int item = wave; item < groups * FR; item += kWaves) {
        const int c = item / FR, f = item % FR;
        const int slot = c * kRows + row;
        if (slot >= rows) continue;
        f32x4 sum[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            sum[m] = part[0][m * FR + f][c][lane];
#pragma unroll
            for (int v = 1; v < kWaves; ++v) {
                const f32x4 o = part[v][m * FR + f][c][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[m][i] += o[i];
            }
        }
        f32x4 o = sum[0];
        if constexpr (NM == 2) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = sum[0][i] / (1.f + expf(-sum[0][i])) * sum[1][i];
        }
        *reinterpret_cast<f32x4*>(dst + (size_t)(slot0 + slot) * N + n0 + f * kRows + kq * 4) = o;
    }
}

// The same sums for calls with work for every CU (see launch_gemm_f32()): a wavefront makes its FR * 16 features of up to NC_MAX * 16
// slots alone, so that nothing goes through LDS, and a workgroup makes four times the features per slot row that it reads, which
// is what long calls are bound by.  It adds up the four quarters of K one after the other, as the kernel above does from four
// wavefronts: the results are the same bits.  WGS: workgroups a CU that the registers must allow.
template <int NM, int FR, int NC_MAX, int WGS>
__global__ __launch_bounds__(kWaves * 64, WGS) void gemm_f32_alone(const float* __restrict__ src, const float* __restrict__ wa,
                                                              const float* __restrict__ wb, const int32_t* __restrict__ offs,
                                                              const int32_t* __restrict__ row_of_slot, int E, int k, int N, int K,
                                                              float* __restrict__ dst,
                                                              const float* __restrict__ x_stale,
                                                              const uint8_t* __restrict__ stale) {
    int tile, unit, e, slot0, rows;
    constexpr int kTile = kWaves * FR * kRows;
    if (!my_work((N + kTile - 1) / kTile, tile, unit)) return;
    if (!find_unit(offs, E, NC_MAX * kRows, unit, e, slot0, rows)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row = lane & 15, kq = lane >> 4;
    const int n0 = (tile * kWaves + wave) * FR * kRows;
    if (n0 >= N) return;  // (N is a multiple of 64: a wavefront has all of its features or none)
    const float* w[NM * FR];
#pragma unroll
    for (int m = 0; m < NM * FR; ++m) w[m] = (m < FR ? wa : wb) + ((size_t)e * N + n0 + (m % FR) * kRows + row) * K + kq * 4;
    auto run = [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        const float* x[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int slot = slot0 + min(c * kRows + row, rows - 1);
            if constexpr (NM == 2) {
                const int assignment = row_of_slot[slot];
                x[c] = ((stale != nullptr && stale[assignment] != 0) ? x_stale : src) + (size_t)(assignment / k) * K + kq * 4;
            } else {
                x[c] = src + (size_t)slot * K + kq * 4;
            }
        }
        f32x4 acc[NM * FR][NC], sum[NM * FR][NC];
        auto each = [&](auto f) {
#pragma unroll
            for (int m = 0; m < NM * FR; ++m)
#pragma unroll
                for (int c = 0; c < NC; ++c) f(acc[m][c], sum[m][c]);
        };
        each([](f32x4& a, f32x4& s) { a = s = f32x4{0.f, 0.f, 0.f, 0.f}; });
        const int quarter = K / kStepK / kWaves;
        int next = quarter - 1;  // last step of the quarter that is being added up
        dot_rows<NM * FR, NC>(w, x, quarter * kWaves, acc, [&](int s) {
            if (s != next) return;
            if (s < quarter) {
                each([](f32x4& a, f32x4& t) { t = a; a = f32x4{0.f, 0.f, 0.f, 0.f}; });
            } else {
                each([](f32x4& a, f32x4& t) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] += a[i];
                    a = f32x4{0.f, 0.f, 0.f, 0.f};
                });
            }
            next += quarter;
        });
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int slot = c * kRows + row;
            if (slot >= rows) continue;
#pragma unroll
            for (int f = 0; f < FR; ++f) {
                f32x4 o = sum[f][c];
                if constexpr (NM == 2) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[i] = sum[f][c][i] / (1.f + expf(-sum[f][c][i])) * sum[FR + f][c][i];
                }
                *reinterpret_cast<f32x4*>(dst + (size_t)(slot0 + slot) * N + n0 + f * kRows + kq * 4) = o;
            }
        }
    };
    const int groups = (rows + kRows - 1) / kRows;
    if constexpr (NC_MAX >= 4) {
        if (groups == 4) run(std::integral_constant<int, 4>{});
        if (groups == 3) run(std::integral_constant<int, 3>{});
    }
    if constexpr (NC_MAX >= 2) {
        if (groups == 2) run(std::integral_constant<int, 2>{});
    }
    if (groups == 1) run(std::integral_constant<int, 1>{});
}

// y[t, :] = sum_j w[t, j] * out[slot_of[t, j], :], j ascending, fp32.
__global__ __launch_bounds__(256) void combine_f32(const float* __restrict__ out, const float* __restrict__ w,
                                                   const int32_t* __restrict__ slot_of, int k, int H,
                                                   float* __restrict__ y) {
    const int t = blockIdx.x;
    for (int h = threadIdx.x * 4; h < H; h += 256 * 4) {
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int j = 0; j < k; ++j) {
            const float wj = w[(size_t)t * k + j];
            const float4 v = *reinterpret_cast<const float4*>(out + (size_t)slot_of[(size_t)t * k + j] * H + h);
            s.x = fmaf(wj, v.x, s.x);
            s.y = fmaf(wj, v.y, s.y);
            s.z = fmaf(wj, v.z, s.z);
            s.w = fmaf(wj, v.w, s.w);
        }
        *reinterpret_cast<float4*>(y + (size_t)t * H + h) = s;
    }
}

// Column groups of 16 slots a workgroup of gemm_f32 takes: the most that still leave kMinWorkgroups of them in tiles of 16 features,
// counting an expert's last unit as half full (with four groups the second GEMM takes two such tiles at once, so it may run half as
// many).  More groups re-read the weights less often; fewer keep more of the chip busy.
// (Measured at 256 and 4096 as well: 300 tokens, hidden 512, ffn 2048, 8 experts, second GEMM 57 / 47 / 47 us at 256 / 1024 /
// 4096, first GEMM 60 / 59 / 66.)
constexpr int kMinWorkgroups = 1024;
int pick_groups(int routed, int experts, int features) {
    for (int nc = 4; nc > 1; nc /= 2)
        if ((long)(routed / (nc * kRows) + (min(experts, routed) + 1) / 2) * (features / kRows) >= kMinWorkgroups) return nc;
    return 1;
}

struct F32Gemm {
    const float *src, *wa, *wb;
    const int32_t *offs, *row_of_slot;
    int E, k, N, K, routed;
    float* dst;
    StaleInput alt;
};

template <class Kernel>
void launch_units(Kernel kernel, const F32Gemm& g, int unit_rows, int tile_features, hipStream_t stream) {
    const int units = g.routed / unit_rows + min(g.E, g.routed);  // sum of the experts' ceil(rows / unit) at most
    const int tiles = (g.N + tile_features - 1) / tile_features, y = min(tiles, 1 << 15);  // (a grid's y ends at 65535)
    const dim3 grid((units + 7) / 8 * 8, y, (tiles + y - 1) / y);
    kernel<<<grid, kWaves * 64, 0, stream>>>(g.src, g.wa, g.wb, g.offs, g.row_of_slot, g.E, g.k, g.N, g.K, g.dst,
                                             static_cast<const float*>(g.alt.x_stale), g.alt.stale);
}

// gemm_f32_alone where there is work for every CU without cutting K over wavefronts, counted in 64 x 64 outputs with an
// expert's last 64 rows as half full.  Split / alone, us:
//   long K, 64 slots x 128 features, from 380 of them and 32 rows an expert on (and not for 64 features: half of every workgroup
//   would have none, K 4096 (407) 441 / 515).  First GEMM, K 4096: 2048 tokens 4119 / 2367, 256 tokens (768) 832 / 526; K 2048: 384 of them 212 / 147, 224 118 / 118; K 1024: 1088 231 / 154, 320 93 / 92 and
//   256 61 / 67; but K 4096 with 16 rows an expert 325 / 348, K 960 with 25 216 / 227, K 512 (528) 45 / 53, K 256 (1056) 72 / 82.
//   short K, 32 slots x 64 features (first) or x 128 (second), from as many of them as K has elements on: what the split
//   costs per output no longer hides behind the contraction.  K 64: 20000 tokens 39 / 20, second 22 / 14; hidden 4096 from ffn 64, 3000
//   tokens 570 / 233; 66 of them 12.8 / 8.5; K 128 (2112) 115 / 73; K 192 (1056) 66 / 59, but 65 11.6 / 12.2.
constexpr int kLongK = 576, kShortK = 192, kMinLongTiles = 380, kMinLongRows = 32;

template <int NM>
void launch_gemm_f32(const F32Gemm& g, hipStream_t stream) {
    const long tiles = (long)(g.routed / (4 * kRows) + (min(g.E, g.routed) + 1) / 2) * (g.N / (4 * kRows));
    if (g.K >= kLongK && tiles >= kMinLongTiles && g.routed >= kMinLongRows * g.E && g.N >= 2 * kWaves * kRows)
        return launch_units(gemm_f32_alone<NM, 2, 4, 1>, g, 4 * kRows, 2 * kWaves * kRows, stream);
    if (g.K <= kShortK && tiles >= g.K)
        return launch_units(gemm_f32_alone<NM, 3 - NM, 2, NM == 2 ? 4 : 3>, g, 2 * kRows, (3 - NM) * kWaves * kRows, stream);
    const int nc = pick_groups(g.routed, g.E, g.N);
    if (nc == 4) launch_units(gemm_f32<NM, NM == 1 ? 2 : 1, 4>, g, 4 * kRows, (NM == 1 ? 2 : 1) * kRows, stream);
    else if (nc == 2) launch_units(gemm_f32<NM, 1, 2>, g, 2 * kRows, kRows, stream);
    else launch_units(gemm_f32<NM, 1, 1>, g, kRows, kRows, stream);
}

}  // namespace

hipError_t launch_ffn_f32(const moe_shape_t& s, int tokens, const float* x, const float* topk_w, const float* w1,
                          const float* w3, const float* w2, float* y, const int32_t* offs,
                          const int32_t* row_of_slot, const int32_t* slot_of, float* act, float* out,
                          const StaleInput& alt, hipStream_t stream) {
    F32Gemm g{x, w1, w3, offs, row_of_slot, s.n_experts, s.top_k, s.ffn, s.hidden, tokens * s.top_k, act, alt};
    launch_gemm_f32<2>(g, stream);
    stage_mark(stream, kStageGemm1);
    g = {act, w2, nullptr, offs, row_of_slot, s.n_experts, s.top_k, s.hidden, s.ffn, tokens * s.top_k, out, {nullptr, nullptr}};
    launch_gemm_f32<1>(g, stream);
    stage_mark(stream, kStageGemm2);
    combine_f32<<<tokens, 256, 0, stream>>>(out, topk_w, slot_of, s.top_k, s.hidden, y);
    stage_mark(stream, kStageCombine);
    return hipGetLastError();
}

}  // namespace moe
