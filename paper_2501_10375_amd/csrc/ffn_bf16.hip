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

// y[t, :] = bf16( sum_j w[t, j] * out[slot_of[t, j], :] ), j ascending, fp32 sum, one rounding.  Where the second GEMM
// split a tile along K, `out` holds its first piece; the others are added from the scratch memory in piece order first.
__global__ __launch_bounds__(256) void combine_bf16(const float* __restrict__ out, const float* __restrict__ w,
                                                    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ idx,
                                                    const int32_t* __restrict__ offs, const gg::SplitTable* __restrict__ split,
                                                    const float* __restrict__ pieces, int E, int k, int H,
                                                    uint16_t* __restrict__ y) {
    const int t = blockIdx.x;
    const int parts = split->parts, slots = split->slots, n_split = split->n_split;
    const int n_ft = (H + 255) / 256;
    for (int h = threadIdx.x * 8; h < H; h += 256 * 8) {
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int j = 0; j < k; ++j) {
            const float wj = w[(size_t)t * k + j];
            const int slot = slot_of[(size_t)t * k + j];
            const float* src = out + (size_t)slot * H + h;
            float4 a = *reinterpret_cast<const float4*>(src);
            float4 b = *reinterpret_cast<const float4*>(src + 4);
            if (parts > 1) {
                const int e = min(max(idx[(size_t)t * k + j], 0), E - 1);
                const int first = offs[e], count = offs[e + 1] - first;
                const int m = (slot - first) / slots;
                const gg::TileList::Place at = gg::TileList::place(count, slots, n_ft, m, h >> 8);
                const int tile = split->first_tile[e] + at.tile - split->first_split;
                if (tile >= 0 && tile < n_split) {
                    const size_t stride = (size_t)split->n_units * gg::kUnitFloats;
                    const float* p = pieces + (size_t)(split->units_before[e] + at.unit - split->first_unit) * gg::kUnitFloats +
                                     (size_t)(slot - first - m * slots) * 256 + (h & 255);
                    for (int i = 1; i < parts; ++i, p += stride) {
                        const float4 c = *reinterpret_cast<const float4*>(p);
                        const float4 d = *reinterpret_cast<const float4*>(p + 4);
                        a.x += c.x; a.y += c.y; a.z += c.z; a.w += c.w;
                        b.x += d.x; b.y += d.y; b.z += d.z; b.w += d.w;
                    }
                }
            }
            s[0] = fmaf(wj, a.x, s[0]); s[1] = fmaf(wj, a.y, s[1]);
            s[2] = fmaf(wj, a.z, s[2]); s[3] = fmaf(wj, a.w, s[3]);
            s[4] = fmaf(wj, b.x, s[4]); s[5] = fmaf(wj, b.y, s[5]);
            s[6] = fmaf(wj, b.z, s[6]); s[7] = fmaf(wj, b.w, s[7]);
        }
        uint4 pk;
        pk.x = pack_bf16x2(s[0], s[1]);
        pk.y = pack_bf16x2(s[2], s[3]);
        pk.z = pack_bf16x2(s[4], s[5]);
        pk.w = pack_bf16x2(s[6], s[7]);
        *reinterpret_cast<uint4*>(y + (size_t)t * H + h) = pk;
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

// One of the two GEMMs.
template <class G>
hipError_t launch_gemm(const gg::GemmArgs& a, int stage, hipStream_t stream) {
    auto kernel = gg::grouped_gemm_kernel<G>;
    static bool configured = false;
    const hipError_t e = allow_lds(kernel, G::kLdsBytes, configured);
    if (e != hipSuccess) return e;
    kernel<<<persistent_grid(), G::kThreads, G::kLdsBytes, stream>>>(a);
    stage_mark(stream, stage);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_bf16(const moe_shape_t& s, int tokens, const void* x, const int32_t* topk_idx, const float* topk_w,
                           const void* w1, const void* w3, const void* w2, void* y, const int32_t* offs,
                           const int32_t* row_of_slot, const int32_t* slot_of, void* act, float* out,
                           int32_t* sync, float* partial, const StaleInput& alt, hipStream_t stream) {
    static_assert(gg::kXcds <= kGemmSyncInts && gg::kScratchFloats * sizeof(float) + sizeof(gg::SplitTable) <= kGemmScratchBytes,
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
    g2.scratch = partial;
    g2.table = reinterpret_cast<gg::SplitTable*>(partial + gg::kScratchFloats);
    hipError_t e;
    // (with tok_alt slot rows are addressed with pointers anyway: only the weight rows decide)
    if (gg::needs_wide(alt.stale != nullptr ? 0 : (size_t)tokens * s.hidden * 2, gg::Gemm<2>::kBF, s.hidden))
        e = launch_gemm<gg::Gemm<2, false, true>>(g1, kStageGemm1, stream);
    else if (alt.stale != nullptr) e = launch_gemm<gg::Gemm<2, true>>(g1, kStageGemm1, stream);
    else e = launch_gemm<gg::Gemm<2>>(g1, kStageGemm1, stream);
    if (e != hipSuccess) return e;
    e = gg::needs_wide(0, 256, s.ffn) ? launch_gemm<gg::Gemm<1, false, true>>(g2, kStageGemm2, stream)
                                      : launch_gemm<gg::Gemm<1>>(g2, kStageGemm2, stream);
    if (e != hipSuccess) return e;
    combine_bf16<<<tokens, 256, 0, stream>>>(out, topk_w, slot_of, topk_idx, offs,
                                             g2.table, partial, s.n_experts, s.top_k, s.hidden, static_cast<uint16_t*>(y));
    stage_mark(stream, kStageCombine);
    return hipGetLastError();
}

}  // namespace moe

