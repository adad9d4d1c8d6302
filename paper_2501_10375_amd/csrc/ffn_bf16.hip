// Grouped SwiGLU expert FFN for bf16 storage on the CDNA4 matrix cores
// (expert execution of DAOP Sec. II-A / Algorithm 1's parallel local expert
// execution; expert = W2 ( silu(W1 x) * (W3 x) ), shapes of Table III).
//
// Two grouped GEMMs, both "row . row" contractions with K contiguous in each
// operand, so operands go from HBM to LDS to MFMA registers without transposes:
//   gemm1: act[slot, f] = silu(x[tok(slot)] . w1[e, f]) * (x[tok(slot)] . w3[e, f])   K = H
//   gemm2: out[slot, h] = act[slot] . w2[e, h]                                        K = F
// followed by the gate-weighted combine over a token's k slots.
//
// The GEMM kernel itself (tiling, LDS pipeline, MFMA layout) is in grouped_gemm_bf16.h.
#include "grouped_gemm_bf16.h"
#include "moe_internal.h"

namespace moe {
namespace {

// Where a selection's row is, and where its pieces are if its tile was split (in every feature tile ft: tile number relative to the
// first split tile tile + ft * tile_step, and likewise units of the scratch memory).
struct CombineRow {
    float w;
    int slot, tile, tile_step, unit, unit_step, row;
};

__device__ inline float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

__device__ inline void accumulate(float (&s)[8], float w, float4 a, float4 b) {
    s[0] = fmaf(w, a.x, s[0]); s[1] = fmaf(w, a.y, s[1]);
    s[2] = fmaf(w, a.z, s[2]); s[3] = fmaf(w, a.w, s[3]);
    s[4] = fmaf(w, b.x, s[4]); s[5] = fmaf(w, b.y, s[5]);
    s[6] = fmaf(w, b.z, s[6]); s[7] = fmaf(w, b.w, s[7]);
}

__device__ inline void store_row(uint16_t* p, const float (&s)[8]) {
    uint4 pk;
    pk.x = pack_bf16x2(s[0], s[1]);
    pk.y = pack_bf16x2(s[2], s[3]);
    pk.z = pack_bf16x2(s[4], s[5]);
    pk.w = pack_bf16x2(s[6], s[7]);
    *reinterpret_cast<uint4*>(p) = pk;
}

// A selection's 8 values at column h, P parts added in their order.  The loads of all parts are requested together.
template <int P>
struct PartRows {
    float4 a[P], b[P];
    bool split;
    __device__ inline void load(const float* out, const float* pieces, const CombineRow& r, int n_split, size_t stride, int H, int h) {
        const int ft = h >> 8;
        split = (unsigned)(r.tile + ft * r.tile_step) < (unsigned)n_split;
        const float* src = out + (size_t)r.slot * H + h;
        a[0] = *reinterpret_cast<const float4*>(src);
        b[0] = *reinterpret_cast<const float4*>(src + 4);
        if (__ballot(split) == 0) return;
        const float* p = split ? pieces + (size_t)(r.unit + ft * r.unit_step) * gg::kUnitFloats + (size_t)r.row * 256 + (h & 255) : src;
#pragma unroll
        for (int i = 1; i < P; ++i) {
            a[i] = *reinterpret_cast<const float4*>(p);
            b[i] = *reinterpret_cast<const float4*>(p + 4);
            p += split ? stride : 0;
        }
    }
    __device__ inline void sum(float4& x, float4& y) const {
        x = a[0];
        y = b[0];
        if (split) {
#pragma unroll
            for (int i = 1; i < P; ++i) {
                x = add4(x, a[i]);
                y = add4(y, b[i]);
            }
        }
    }
};

// Tile and unit of a row of expert e at feature tile 0, relative to the first split tile, and what a feature tile adds.
__device__ inline CombineRow combine_row(const gg::SplitTable* __restrict__ split, const int32_t* __restrict__ offs, int e, int slot,
                                         int H) {
    const int first = offs[e], count = offs[e + 1] - first, slots = split->slots;
    const int m = (slot - first) / slots;
    const gg::TileList::Place at = gg::TileList::place(count, slots, (H + 255) / 256, m);
    CombineRow r;
    r.slot = slot;
    r.tile = split->first_tile[e] + at.tile - split->first_split;
    r.tile_step = at.tile_step;
    r.unit = split->units_before[e] + at.unit - split->first_unit;
    r.unit_step = at.unit_step;
    r.row = slot - first - m * slots;
    return r;
}

// y[t, :] = bf16( sum_j w[t, j] * out[slot_of[t, j], :] ), j ascending, fp32 sum, one rounding.  Where the second GEMM
// split a tile along K, `out` holds its first piece; the others are added from the scratch memory in piece order first.
//
// Long calls are bound by memory and want many wavefronts; short ones by the chain of loads, which with split tiles is one
// memory round trip per piece.  AHEAD (short calls) looks the rows up once per token, through LDS, and requests the rows and all
// pieces of two selections before it uses the first, at 118 registers instead of 34: 66 tokens, hidden 3008, 3 selections of 6
// parts 16.2 -> 9.9 us; 195 tokens, hidden 2944, 4 selections of 5 parts 19.8 -> 12.6; but 1500 tokens, hidden 2048, 12.5 -> 14.8.
template <bool AHEAD>
__global__ __launch_bounds__(256) void combine_bf16(const float* __restrict__ out, const float* __restrict__ w,
                                                    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ idx,
                                                    const int32_t* __restrict__ offs, const gg::SplitTable* __restrict__ split,
                                                    const float* __restrict__ pieces, int E, int k, int H,
                                                    uint16_t* __restrict__ y) {
    const int t = blockIdx.x;
    const int parts = split->parts, n_split = split->n_split;
    const size_t stride = (size_t)split->n_units * gg::kUnitFloats;
    const int h_first = (blockIdx.y * 256 + threadIdx.x) * 8, h_step = gridDim.y * 256 * 8;
    if (!AHEAD || parts <= 1) {
        for (int h = h_first; h < H; h += h_step) {
            float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int j = 0; j < k; ++j) {
                const int slot = slot_of[(size_t)t * k + j];
                const float* src = out + (size_t)slot * H + h;
                float4 a = *reinterpret_cast<const float4*>(src);
                float4 b = *reinterpret_cast<const float4*>(src + 4);
                if (!AHEAD && parts > 1) {
                    const int ft = h >> 8;
                    const CombineRow r = combine_row(split, offs, min(max(idx[(size_t)t * k + j], 0), E - 1), slot, H);
                    if ((unsigned)(r.tile + ft * r.tile_step) < (unsigned)n_split) {
                        const float* p = pieces + (size_t)(r.unit + ft * r.unit_step) * gg::kUnitFloats + (size_t)r.row * 256 + (h & 255);
                        for (int i = 1; i < parts; ++i, p += stride) {
                            a = add4(a, *reinterpret_cast<const float4*>(p));
                            b = add4(b, *reinterpret_cast<const float4*>(p + 4));
                        }
                    }
                }
                accumulate(s, w[(size_t)t * k + j], a, b);
            }
            store_row(y + (size_t)t * H + h, s);
        }
        return;
    }
    __shared__ CombineRow rows[8];
    if ((int)threadIdx.x < k) {
        const size_t a = (size_t)t * k + threadIdx.x;
        rows[threadIdx.x] = combine_row(split, offs, min(max(idx[a], 0), E - 1), slot_of[a], H);
        rows[threadIdx.x].w = w[a];
    }
    __syncthreads();
    auto run = [&](auto parts_c) {
        constexpr int P = decltype(parts_c)::value;
        for (int h = h_first; h < H; h += h_step) {
            float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            for (int j = 0; j < k; j += 2) {
                const bool two = j + 1 < k;
                PartRows<P> r0, r1;
                r0.load(out, pieces, rows[j], n_split, stride, H, h);
                if (two) r1.load(out, pieces, rows[j + 1], n_split, stride, H, h);
                float4 a, b;
                r0.sum(a, b);
                accumulate(s, rows[j].w, a, b);
                if (two) {
                    r1.sum(a, b);
                    accumulate(s, rows[j + 1].w, a, b);
                }
            }
            store_row(y + (size_t)t * H + h, s);
        }
    };
    if constexpr (AHEAD) {
        static_assert(gg::kMaxParts == 6, "one version per number of parts");
        switch (parts) {
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 5: run(std::integral_constant<int, 5>{}); break;
            default: run(std::integral_constant<int, 6>{}); break;
        }
    }
}

// Second half of a first GEMM whose tiles were all cut (CUT): act[slot, f] = silu(g) * u, g and u the sums over the tile's pieces
// in their order.  Four features a thread, all of their pieces requested together.  Bound by the latency of its two round
// trips (tables, pieces).
__global__ __launch_bounds__(256) void sum_swiglu_bf16(const float* __restrict__ pieces, const gg::SplitTable* __restrict__ split,
                                                       const int32_t* __restrict__ offs, int E, int F, int routed,
                                                       uint16_t* __restrict__ act) {
    __shared__ int first[65], tile_units[64];
    const int tid = threadIdx.x;
    if (tid <= E) first[tid] = offs[tid];
    if (tid < E) tile_units[tid] = split->units_before[tid];
    const int parts = split->parts, slots = split->slots;
    const size_t stride = (size_t)split->n_units * gg::kUnitFloats;
    __syncthreads();
    const int64_t item = (int64_t)blockIdx.x * 256 + tid;
    const int slot = (int)(item / (F / 4)), f = (int)(item - (int64_t)slot * (F / 4)) * 4;
    if (slot >= routed) return;
    int e = 0;  // the last expert whose first slot is not behind this one
#pragma unroll
    for (int d = 32; d > 0; d /= 2)
        if (e + d < E && first[e + d] <= slot) e += d;
    const int count = first[e + 1] - first[e], m = (slot - first[e]) / slots, ft = f >> 7;
    const gg::TileList::Place at = gg::TileList::place(count, slots, (F + 127) / 128, m);
    const float* src = pieces + (size_t)(tile_units[e] + at.unit + ft * at.unit_step) * gg::kUnitFloats +
                       (size_t)(slot - first[e] - m * slots) * 256 + (f & 127);
    auto run = [&](auto parts_c) {
        constexpr int P = decltype(parts_c)::value;
        float4 g[P], u[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            g[i] = *reinterpret_cast<const float4*>(src + i * stride);
            u[i] = *reinterpret_cast<const float4*>(src + i * stride + 128);
        }
#pragma unroll
        for (int i = 1; i < P; ++i) {
            g[0] = add4(g[0], g[i]);
            u[0] = add4(u[0], u[i]);
        }
        uint2 pk;
        pk.x = pack_bf16x2(swiglu(g[0].x, u[0].x), swiglu(g[0].y, u[0].y));
        pk.y = pack_bf16x2(swiglu(g[0].z, u[0].z), swiglu(g[0].w, u[0].w));
        *reinterpret_cast<uint2*>(act + (size_t)slot * F + f) = pk;
    };
    static_assert(gg::kMaxCutParts == 8, "one version per number of parts");
    switch (parts) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        default: run(std::integral_constant<int, 8>{}); break;
    }
}

// Raises a kernel's dynamic LDS limit once (idempotent; a race only repeats it).
template <typename Kernel>
hipError_t allow_lds(Kernel k, int bytes, bool& configured) {
    if (configured) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    configured = e == hipSuccess;
    return e;
}

// One persistent workgroup per CU (a multiple of the 8 XCDs); the kernels size their own work from `offs`.
int persistent_grid() { return max(gg::kXcds, compute_units() / gg::kXcds * gg::kXcds); }

// One of the two GEMMs in a launch of its own.
template <class G>
hipError_t launch_gemm(const gg::GemmArgs& a, hipStream_t stream) {
    auto kernel = gg::grouped_gemm_kernel<G>;
    static bool configured = false;
    const hipError_t e = allow_lds(kernel, G::kLdsBytes, configured);
    if (e != hipSuccess) return e;
    kernel<<<persistent_grid(), G::kThreads, G::kLdsBytes, stream>>>(a);
    return hipGetLastError();
}

// Both in one.
template <bool ALT>
hipError_t launch_linked(const gg::GemmArgs& a, const gg::GemmArgs& b, int32_t* done, uint32_t* status, hipStream_t stream) {
    using First = gg::Gemm<2, ALT, false, false, true>;
    auto kernel = gg::linked_grouped_gemm_kernel<First>;
    static bool configured = false;
    const hipError_t e = allow_lds(kernel, First::kLdsBytes, configured);
    if (e != hipSuccess) return e;
    kernel<<<persistent_grid(), First::kThreads, First::kLdsBytes, stream>>>(a, b, done, status, decode_spin_limit());
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_bf16(const moe_shape_t& s, int tokens, const void* x, const int32_t* topk_idx, const float* topk_w,
                           const void* w1, const void* w3, const void* w2, void* y, const int32_t* offs,
                           const int32_t* row_of_slot, const int32_t* slot_of, void* act, float* out,
                           int32_t* sync, uint32_t* status, float* partial, const StaleInput& alt, hipStream_t stream) {
    static_assert(gg::kXcds + 64 <= kGemmSyncInts && gg::kScratchFloats * sizeof(float) + 2 * sizeof(gg::SplitTable) <= kGemmScratchBytes,
                  "workspace layout");
    gg::GemmArgs g1{}, g2{};
    g1.tok = static_cast<const uint16_t*>(x);
    g1.wa = static_cast<const uint16_t*>(w1);
    g1.wb = static_cast<const uint16_t*>(w3);
    g1.offs = offs;
    g1.row_of_slot = row_of_slot;
    g1.E = s.n_experts;
    g1.topk = s.top_k;
    g1.N = s.ffn;
    g1.K = s.hidden;
    g1.dst = act;
    g1.sync = sync;
    g1.scratch = partial;
    g1.table = reinterpret_cast<gg::SplitTable*>(partial + gg::kScratchFloats);
    g1.tok_alt = static_cast<const uint16_t*>(alt.x_stale);
    g1.alt_mask = alt.stale;
    g2 = g1;
    g2.tok = static_cast<const uint16_t*>(act);
    g2.wa = static_cast<const uint16_t*>(w2);
    g2.wb = nullptr;
    g2.N = s.hidden;
    g2.K = s.ffn;
    g2.dst = out;
    g2.sync = sync + kGemmSyncInts;
    g2.table = g1.table + 1;
    const bool alternate = alt.stale != nullptr;
    const int routed = tokens * s.top_k;
    const long slot_tiles = routed / 256 + min(s.n_experts, routed);  // at most
    const long most_tiles = (s.ffn + 127) / 128 * slot_tiles;
    hipError_t e;
    const bool wide2 = gg::needs_wide(0, 256, s.ffn), wide1 = wide2 || gg::needs_wide((size_t)tokens * s.hidden * 2, gg::Gemm<2>::kBF, s.hidden);
    const bool cut = !wide1 && most_tiles <= gg::kMaxCutTiles && s.hidden / 64 >= gg::kMinCutKSteps;
    if (!wide1 && gg::links(most_tiles, (s.hidden + 255) / 256 * slot_tiles, persistent_grid(), routed, s.n_experts, s.hidden, s.ffn)) {
        int32_t* done = sync + gg::kXcds;
        e = alternate ? launch_linked<true>(g1, g2, done, status, stream) : launch_linked<false>(g1, g2, done, status, stream);
        stage_mark(stream, kStageFused);
    } else {
        if (wide1) {  // (with and without tok_alt alike: with nothing taken from it the results have the same bits)
            e = launch_gemm<gg::Gemm<2, false, true>>(g1, stream);
        } else if (cut) {
            e = alternate ? launch_gemm<gg::Gemm<2, true, false, true>>(g1, stream) : launch_gemm<gg::Gemm<2, false, false, true>>(g1, stream);
            const int64_t threads = (int64_t)routed * (s.ffn / 4);
            sum_swiglu_bf16<<<(unsigned)((threads + 255) / 256), 256, 0, stream>>>(partial, g1.table, offs, s.n_experts, s.ffn, routed,
                                                                                  static_cast<uint16_t*>(act));
        } else {
            e = alternate ? launch_gemm<gg::Gemm<2, true>>(g1, stream) : launch_gemm<gg::Gemm<2>>(g1, stream);
        }
        stage_mark(stream, kStageGemm1);
        if (e != hipSuccess) return e;
        e = wide2 ? launch_gemm<gg::Gemm<1, false, true>>(g2, stream) : launch_gemm<gg::Gemm<1>>(g2, stream);
        stage_mark(stream, kStageGemm2);
    }
    if (e != hipSuccess) return e;
    const int column_blocks = (s.hidden + 2047) / 2048;
    // AHEAD up to three workgroups a CU: 720 of them (360 tokens, hidden 4096) 17.0 -> 15.1 us, 1000 to 1050 are equal (14.1; 10.5 and
    // 10.4), 1200 take 11.8 without and 13.3 with it.
    // A workgroup for every 2048 columns up to six a CU: 512 tokens, hidden 4096 14.6 -> 13.6, 700 tokens 12.4 -> 10.4; 900 9.9 -> 10.1.
    const long blocks = (long)tokens * column_blocks;
    const bool ahead = blocks <= 3 * compute_units();
    (ahead ? combine_bf16<true> : combine_bf16<false>)<<<dim3(tokens, blocks <= 6 * compute_units() ? column_blocks : 1), 256, 0, stream>>>(
        out, topk_w, slot_of, topk_idx, offs, g2.table, partial, s.n_experts, s.top_k, s.hidden, static_cast<uint16_t*>(y));
    stage_mark(stream, kStageCombine);
    return hipGetLastError();
}

}  // namespace moe

