// Grouped bf16 GEMM for the expert FFN on the CDNA4 matrix cores (device code).
//
// Computes, per (expert, slot tile of at most 256 slots, feature tile),
//   NMAT = 2 (gemm1): act[slot, f] = silu(tok[slot] . wa[e, f]) * (tok[slot] . wb[e, f])   (bf16 out)
//   NMAT = 1 (gemm2): out[slot, n] = tok[slot] . wa[e, n]                                  (fp32 out)
// where tok rows are gathered rows of x (gemm1) or rows of act (gemm2), and every
// operand is K-contiguous ("row . row" contraction, no transposes anywhere).
//
// Organisation (gfx950):
//   * Tile 256 slots x 256 weight rows (NMAT = 2: 128 features of each matrix), K in steps of 64; four
//     wavefronts.  Weights are the MFMA "A" operand, slot rows the "B" operand, so a lane ends up holding 4
//     consecutive output features of one slot.
//   * Operand tiles go HBM/L2 -> LDS directly (16 bytes per lane, no register staging).  Each lane supplies
//     its own global address, which is how gathered rows and the XOR swizzle are expressed: the 16-byte piece
//     that must land at LDS position p is fetched by the lane whose data lands at p.  The swizzle makes the
//     ds_read_b128 operand reads bank-conflict free on the 64-bank LDS.  A load instruction moves whole
//     128-byte lines.
//   * The loads are issued from inline asm so the compiler does not serialise them against the
//     LDS reads of other stages; completion is enforced by hand: s_waitcnt vmcnt(n) on the issuing
//     wavefront, then a workgroup barrier, before any wavefront reads the stage.  One barrier per K step.
//   * Persistent schedule, one workgroup per CU, tiles handed out in rounds per XCD so the
//     workgroups of an XCD share operand tiles through its L2 (see persistent()).  A workgroup requests the first operands of its
//     next tile before it stores the results of the last one (see Gemm::run()).
//   * Calls of middle size run both GEMMs in one launch (see Link).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bf16_utils.h"
#include "hand_out.h"
#include "moe_internal.h"

// Everything is compiled into its kernel: what a call would return counts as different from lane to lane.
#define GG_INLINE __attribute__((always_inline)) inline
#define GG_LAMBDA __attribute__((always_inline))

namespace moe {
namespace gg {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kMaxWgsPerXcd = 32;  // persistent grid: at most 8 x 32 workgroups

// A launch uses kXcds counters (`sync`): the tiles handed out so far in each XCD (see persistent()); all zero when it starts.

// A K-split tile of the second GEMM leaves its first piece in the output and the others in the scratch memory, in rows of
// 256 columns, a tile's rows rounded up to whole units of 32.  All first pieces there come first, then all second ones; within
// them the tiles follow each other in the order of the tile list without gaps.  The kernel that combines a token's
// selections adds them.  The table tells it where they are: slots per tile, parts per split tile, number of the first split
// tile, how many are split, the units before the first of them and in all of them, and per expert the number of its first tile
// and the units before it.
constexpr int kUnitRows = 32;
struct SplitTable {
    int slots, parts, first_split, n_split, first_unit, n_units;
    int pad[2];
    int first_tile[64], units_before[64];
};
// K parts a leftover tile can be cut into, and the fewest K steps of 64 that a part has.
constexpr int kMaxParts = 6, kMinPartKSteps = 3;
// Shortest K (steps of 64) at which a workgroup whose XCD has nothing left looks for work elsewhere, see persistent().
constexpr int kMinStealKSteps = 48;
// Scratch memory for those pieces: enough to cut any 255 tiles of 256 rows into two parts, and low tiles into more.  The parts
// are chosen to fit.  (Twice as much let 129 to 170 full tiles have three.)  The tables follow the pieces.
constexpr size_t kUnitFloats = kUnitRows * 256;
constexpr int kScratchUnits = 255 * 8;
constexpr size_t kScratchFloats = kScratchUnits * kUnitFloats;

// Tile list.  The number of tiles depends on the routing (sum over experts of ceil(count / 256) slot tiles, times the
// feature tiles) and is only known on the device: every wavefront derives the list from `offs` when the kernel starts
// and keeps it across its lanes (at most 64 experts), so that looking a tile up is a ballot and a few scalar
// operations.
//
// Order: experts by descending row count.  Within an expert its slot tiles in groups of at most kGroup
// of nearly equal size, within a group feature tile by feature tile and within a feature tile slot tile by slot tile.  32 consecutive
// tiles (what the 32 CUs of an XCD work on at one time) are then about 8 slot tiles x 4 feature tiles of one
// expert: 12 distinct operand tiles feed 32 workgroups through the XCD's L2, and the groups of an expert with more
// than 8 slot tiles meet the same weights at about the same time.
constexpr int kGroup = 8;

// Sums over the lanes of a wavefront, all of them at once (a sum by itself is six LDS round trips).
template <int N>
__device__ GG_INLINE void wave_totals(int (&v)[N]) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], d, 64);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_amdgcn_readfirstlane(v[i]);
}
// A value that is the same in all lanes, in a scalar register.
__device__ GG_INLINE int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ GG_INLINE int wave_inclusive_sum(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

struct TileList {
    int n_ft;                 // feature tiles
    int slots;                // slots per tile
    int total, heavy;         // tiles; tiles of experts with two slot tiles or more (they come first)
    // lane r: the expert of rank r
    int expert, count, first_slot, first_tile;
    int units, first_unit;    // units of 32 rows of all tiles, and before an expert's (count_units())

    __device__ GG_INLINE TileList(const int32_t* __restrict__ offs, int E) {
        const int lane = threadIdx.x & 63;
        const int o = lane < E ? offs[lane] : 0;
        const int c = lane < E ? offs[lane + 1] - o : -1;
        int rank = lane < E ? 0 : lane;
        for (int i = 0; i < E; ++i) {
            const int ci = __builtin_amdgcn_readlane(c, i);
            if (lane < E) rank += (ci > c || (ci == c && i < lane)) ? 1 : 0;
        }
        n_ft = slots = total = heavy = first_tile = units = first_unit = 0;
        expert = __builtin_amdgcn_ds_permute(rank * 4, lane);
        count = __builtin_amdgcn_ds_permute(rank * 4, c);
        first_slot = __builtin_amdgcn_ds_permute(rank * 4, o);
    }

    static __device__ GG_INLINE int units_of(int rows) { return rows > 0 ? (rows + kUnitRows - 1) / kUnitRows : 0; }

    // Slot tiles of `s` rows of this lane's expert.
    __device__ GG_INLINE int slot_tiles(int s) const { return count > 0 ? (count + s - 1) / s : 0; }

    __device__ GG_INLINE void build(int slots_per_tile) {
        slots = slots_per_tile;
        const int tiles = slot_tiles(slots) * n_ft;
        const int tile_sum = wave_inclusive_sum(tiles);
        first_tile = tile_sum - tiles;
        total = __builtin_amdgcn_readlane(tile_sum, 63);
        const int n_heavy = __popcll(__ballot(count > slots));
        heavy = n_heavy > 0 ? __builtin_amdgcn_readlane(tile_sum, n_heavy - 1) : 0;
    }

    __device__ GG_INLINE void count_units() {
        const int own = units_of(count) * n_ft;
        const int sum = wave_inclusive_sum(own);
        first_unit = sum - own;
        units = __builtin_amdgcn_readlane(sum, 63);
    }

    // Tile `id` (r: its expert's rank), and the units of the tiles before it (valid after count_units()).
    __device__ GG_INLINE void find(int id, int& r, int& e, int& slot0, int& rows, int& ft, int& unit) const {
        r = __popcll(__ballot(first_tile <= id && count > 0)) - 1;
        const int c = __builtin_amdgcn_readlane(count, r);
        e = __builtin_amdgcn_readlane(expert, r);
        const int local = id - __builtin_amdgcn_readlane(first_tile, r);
        const int mt = (c + slots - 1) / slots;
        // `big` groups of `size` + 1 slot tiles, then groups of `size`
        const int groups = (mt + kGroup - 1) / kGroup;
        const int size = mt / groups, big = mt - size * groups;
        const int in_big = big * (size + 1) * n_ft;
        const bool b = local < in_big;
        const int gs = b ? size + 1 : size;
        const int in = b ? local : local - in_big;
        const int g = in / (gs * n_ft);
        const int in_grp = in - g * (gs * n_ft);
        ft = in_grp / gs;
        const int from = (b ? 0 : big * (size + 1)) + g * gs;  // the group's first slot tile
        const int m = from + (in_grp - ft * gs);
        slot0 = __builtin_amdgcn_readlane(first_slot, r) + m * slots;
        rows = min(slots, c - m * slots);
        unit = __builtin_amdgcn_readlane(first_unit, r) + local * (slots / kUnitRows) - (from + gs == mt ? ft * units_missing(c, mt, slots) : 0);
    }
    // What the last slot tile of an expert of c rows lacks of slots / 32 units.
    static __device__ GG_INLINE int units_missing(int c, int mt, int slots) { return slots / kUnitRows - units_of(c - (mt - 1) * slots); }

    // Inverse of find() within an expert of c rows: where slot tile m stands, number and units before it at feature tile 0, and
    // what each further feature tile adds.
    struct Place {
        int tile, tile_step, unit, unit_step;
    };
    static __device__ GG_INLINE Place place(int c, int slots, int n_ft, int m) {
        const int mt = (c + slots - 1) / slots;
        const int groups = (mt + kGroup - 1) / kGroup;
        const int size = mt / groups, big = mt - size * groups;
        const bool b = m < big * (size + 1);
        const int gs = b ? size + 1 : size;
        const int from = b ? m / gs * gs : big * (size + 1) + (m - big * (size + 1)) / gs * gs;  // the group's first slot tile
        const int tile = from * n_ft + m - from, full = slots / kUnitRows;
        return {tile, gs, tile * full, gs * full - (from + gs == mt ? units_missing(c, mt, slots) : 0)};
    }
};

// tok: gemm1 -> x [T, K] rows gathered via row_of_slot / topk; gemm2 -> act [A, K], rows = slots.
// wa, wb: [E, N, K]; dst: gemm1 -> bf16 [A, N]; gemm2 -> fp32 [A, N].
struct GemmArgs {
    const uint16_t *tok, *wa, *wb;
    const int32_t *offs, *row_of_slot;
    int E, topk, N, K;
    void* dst;
    int32_t* sync;
    float* scratch;              // second GEMM, CUT: pieces of split tiles, kScratchUnits units ...
    SplitTable* table;           // ... and where they are
    const uint16_t* tok_alt;     // gemm1 with per-selection input rows (ALT), else null
    const uint8_t* alt_mask;
};

template <int N>
__device__ GG_INLINE void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// Waits for all but the `stores` (2, 4, ..., 16) and eight loads that were issued last.
__device__ GG_INLINE void wait_stores(int stores) {
    switch (stores) {
        case 2: wait_vmcnt<10>(); break;
        case 4: wait_vmcnt<12>(); break;
        case 6: wait_vmcnt<14>(); break;
        case 8: wait_vmcnt<16>(); break;
        case 10: wait_vmcnt<18>(); break;
        case 12: wait_vmcnt<20>(); break;
        case 14: wait_vmcnt<22>(); break;
        case 16: wait_vmcnt<24>(); break;
        default: wait_vmcnt<8>(); break;
    }
}

// Workgroup barrier that orders LDS traffic only (no wait on outstanding global loads).
__device__ GG_INLINE void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders a wavefront's own LDS traffic (which the hardware does by itself; this is for the compiler).
__device__ GG_INLINE void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// LDS swizzle: the 16-byte piece `chunk` (of 8) of tile row `row` is stored at piece position
// swizzled(row, chunk) of that row.  The LDS has 64 four-byte banks (256 bytes per cycle), so a
// ds_read_b128 serves 16 lanes per cycle; the lanes of one MFMA operand read sit on 16
// consecutive rows at the same chunk, and the XOR below spreads them over all 64 banks.
__device__ GG_INLINE int swizzled(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// Both GEMMs in one launch (LINKED): a workgroup that finds no more tiles of the first GEMM goes on with the second one's, so neither
// the workgroups that end the first early nor the next kernel's start cost anything.  A tile of the second GEMM needs all of its
// expert's tiles of the first: `done` counts those per expert, and a workgroup looks at it before it requests the tile's first
// slot rows (its weights are on their way by then).  act is stored through to memory, a tile is counted when all of its stores
// have been acknowledged, and act is not read by anybody in this launch before that, so that no cache can hold an older copy.
//
// A workgroup only waits for tiles that others have already taken, and they wait for nobody in the first GEMM: every one of its tiles, a
// workgroup's first included, is claimed from a counter (see owns_first()), and when a workgroup goes on, nothing is left to claim in any
// XCD's list.  So the wait ends whatever part of the grid is resident.  It is bounded all the same (memory that an overlapping call
// clears must not hang the GPU): when it runs out the status word is raised and the tile's results are NaN.
//
// Which calls: see links().
struct Link {
    int32_t* done;       // tiles of the first GEMM that are stored, per expert (null: not linked)
    uint32_t* status;
    int spin_limit;
    int need, expert;    // lane r: of the expert of rank r
    uint64_t ready;      // ranks whose act is complete (the same in all wavefronts)
    unsigned char* told; // 8 bytes of LDS for share()

    __device__ GG_INLINE void finish(int e) { __hip_atomic_fetch_add(&done[e], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ GG_INLINE bool is_first() const { return threadIdx.x < 64; }
    __device__ GG_INLINE void pause() const { __builtin_amdgcn_s_sleep(8); }
    __device__ GG_INLINE uint64_t look() const {
        return __ballot(need == 0 || __hip_atomic_load(&done[expert], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= need);
    }
    __device__ GG_INLINE void report() const {
        if (threadIdx.x == 0) __hip_atomic_store(status, kDecodeGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ GG_INLINE uint64_t share(uint64_t r) const {
        if (threadIdx.x == 0) *reinterpret_cast<uint64_t*>(told) = r;
        lds_barrier();
        r = *reinterpret_cast<const uint64_t*>(told);
        return (uint64_t)(uint32_t)uniform((int)(r >> 32)) << 32 | (uint32_t)uniform((int)(uint32_t)r);
    }
    __device__ GG_INLINE bool await(int rank, unsigned char* lds_words) {
        told = lds_words;
        const bool complete = await_rank(rank, ready, spin_limit, *this);
        asm volatile("" ::: "memory");
        return complete;
    }
};

// Whether a call runs both GEMMs in one launch.  first, second: tiles of 256 slots that the two can have at most, grid: workgroups.  Handing act
// over costs 5 to 15 us; what it gives is the end of the first GEMM, filled with tiles of the second whose experts are complete.  So:
//   * more than two and a half rounds of the first GEMM (else little else is running while an expert completes), three quarters of a round of the
//     second, and 4e5 routed elements of the hidden dimension (with fewer the second GEMM is over as soon as it begins).  With 2e10 products of a
//     routed row and a weight, which take half a millisecond, nine sixteenths of a round of the second will do;
//   * or more than five quarters of a round of the first with 48 rows an expert, if the second has more than a round;
//   * in both cases at most 300 rows an expert, beyond which the second GEMM waits for too many tiles at a time, and 1.6e11 products, beyond
//     which the chip is at its power limit: time that is saved comes back as clock that is lost.
// Whole layer in us, apart / linked (hidden, ffn, experts, top-k, tokens; 184 sizes were timed).  Linked: 2048, 1408, 64, 6, 40 207 / 199, 400 248 / 236,
// 1003 284 / 277, 2500 375 / 363; 4096, 14336, 8, 2, 200 505 / 483, 512 617 / 594, 1024 783 / 768; 4096, 6400, 16, 2, 200 380 / 378, 2048 763 / 752; 2112, 5888, 16, 4,
// 349 +3.4 %; 4096, 2048, 16, 2, 700 238 / 223; 3456, 2624, 16, 1, 1616 +3.8 %.  On 90 sizes drawn after the rule was made, 25 of them linked, those are
// 2.6 % faster so on average, the worst is 1024, 1472, 64, 3, 1187 with 146 / 150.  Apart, few rounds or rows:
// 2432, 2624, 16, 2, 108 142 / 154, 300 150 / 158, 800 173 / 178; 1024, 4096, 12, 2, 100 78 / 86; 1536, 1984, 32, 3, 100 124 / 130; 3008, 5632, 16, 1, 100
// 292 / 305; 64, 1024, 64, 8, 40 43 / 47; little of the second: 640, 5824, 16, 3, 46 84 / 92; 1600, 4544, 16, 1, 47 75 / 88; 1024, 4032, 12, 2, 1052 113 / 120;
// 4096, 14336, 8, 2, 50 497 / 501, 77 512 / 514; many rows: 1664, 5888, 4, 4, 885 206 / 216; 3328, 7744, 4, 2, 1865 477 / 485; 896, 1792, 16, 4, 1554 106 / 121;
// long: 4096, 14336, 8, 2, 1400 932 / 945, 2048 1214 / 1235.  What this gives away: 3008, 5632, 12, 1, 66 259 / 242; 3648, 1664, 32, 1, 290 218 / 203.
constexpr bool links(long first, long second, int grid, long routed, int experts, long hidden, long ffn) {
    const long active = routed < experts ? routed : experts;
    const double macs = (double)routed * hidden * ffn;
    if (routed > 300 * active || macs > 1.6e11) return false;
    const bool long_first = first * 2 > grid * 5L && routed * hidden >= 400000 &&
                            (second * 4 >= grid * 3L || (second * 16 >= grid * 9L && macs >= 2e10));
    return long_first || (first * 4 > grid * 5L && second * 6 >= grid * 7L && routed >= 48 * active);
}

// ---- one tile: up to 256 slots x 256 weight rows, one wavefront per SIMD.
//
// What a tile of this size costs is set by two things: how many cycles of a K step are not MFMA cycles, and
// how fast the chip may clock while it runs them (the board is at its power limit throughout).  Measured on
// a dense 4096 x 4096 x 14336 problem, which the loop that this one replaced (8 wavefronts, 32x32x16 MFMAs,
// every load slot under a branch on "is there a later K step") ran at 1280 TFLOP/s:
//   * 16x16x32 MFMAs.  A loop of nothing but MFMAs on operands with random mantissas runs at 2.07 PFLOP/s
//     with them and at 1.80 with 32x32x16: per flop they move half the accumulator data through the register
//     file, and at the power limit that is clock (2.05 against 1.80 GHz).
//   * 2 x 2 wavefronts of 128 x 128 outputs each, accumulators in the AGPRs: a K step reads 128 KB of operand
//     fragments from LDS instead of 192 KB with 2 x 4 wavefronts, which again is power (8 wavefronts, otherwise
//     the same: 1351 against 1565 TFLOP/s).
//   * No branches between the MFMAs.  With a single wavefront on a SIMD nothing hides a branch; the load slots
//     of a K step cost 37 cycles each as `if (more) load`.  The last K steps, which load nothing, are separate
//     code: 2342 instead of 2886 cycles per K step, 2048 of which are the MFMAs.
//   * Between two MFMAs (16 cycles) go at most two other instructions: an LDS read (one address register per
//     operand and half K step, fragments at constant offsets), or half of a load (M0 in one slot, the load in
//     the next).  Loads take their row from a 32-bit lane offset and the K step from a scalar offset.
// The 160 KB of LDS hold five 32 KB operand tiles: three stages of weights, whose lines are the ones that come from
// memory and are requested two K steps ahead, and two of slots, whose lines mostly come from the L2 or the memory-side
// cache.  (Wavefronts of the first GEMM then wait for 9 % of their cycles, 35 % before.)
// In the layer, 4096 tokens of the Mixtral shape: first GEMM 1747 -> 1463 us, second 908 -> 761 us (1315 and 1264
// TFLOP/s of routed rows, 9 % padding not counted).  Calls with few rows per expert, which stream weights, run at 6.0 TB/s
// (77 tokens, first GEMM: 328 -> 313 us against 128-slot tiles on eight wavefronts).
//
// A tile of TFE * 32 slots or fewer runs a main loop that computes and stages only TFE (1 to 8) of the eight
// 32-slot groups: slots are dealt to the two slot groups of wavefronts in fragments of 16, and every wavefront
// stages 8 rows of each 32-slot group, so all four wavefronts get shorter by the same amount.
//
// ALT (first GEMM): a slot's row comes from tok_alt where alt_mask says so; slot rows are addressed with 64-bit pointers.
// WIDE: every operand is addressed with 64-bit pointers, and tok_alt is used if there is one.  For operands that a 32-bit
// lane offset does not reach: x of kWideBytes or more, or a tile of weight or slot rows of that size (see needs_wide()).
// CUT (first GEMM): every tile is cut along K, see choose_cut(); the sums of both matrices go to the scratch memory in fp32, 128
// columns of each side by side, and another kernel adds the pieces and applies SwiGLU.
// LINKED: both GEMMs run in one kernel, see Link.
template <int NMAT, bool ALT = false, bool WIDE = false, bool CUT = false, bool LINKED = false>
struct Gemm {
    static_assert(!(ALT && WIDE) && (!ALT || NMAT == 2), "only the first GEMM gathers rows of x");
    static_assert(!CUT || (NMAT == 2 && !WIDE), "the second GEMM cuts by itself");
    static_assert(!LINKED || (!WIDE && !CUT), "the other versions run in kernels of their own");
    static constexpr bool kLinked = LINKED, kCut = CUT, kFp32 = NMAT == 1 || CUT;
    static constexpr int kThreads = 256, kMats = NMAT;
    static constexpr int kBF = 256 / NMAT;            // features per tile (per matrix)
    static constexpr int kF = 8;                      // 16-row fragments of each operand per wavefront
    static constexpr int kStage = 32768;              // one operand tile: 256 rows of 128 bytes
    static constexpr uint32_t kSlotBase = 3 * kStage; // weights: three stages from 0, slots: two stages from here
    static constexpr int kLdsBytes = 5 * kStage;
    static constexpr int kRowsOffset = 1024;          // row numbers of the next item's slots, 256 bytes a wavefront, behind the item's number
    static constexpr int kToldOffset = 16;            // see Link::await()

    typedef __attribute__((address_space(3))) const unsigned char* lds_ptr;
    using Yes = std::true_type;
    using No = std::false_type;

    // M0 (the LDS address of the load that follows in a later slot; nothing in the loop writes it in between) ...
    static __device__ GG_INLINE void set_lds_target(uint32_t lds_base) { asm volatile("s_mov_b32 m0, %0" ::"s"(lds_base) : "memory"); }
    // ... and the load itself: 16 bytes per lane from base + lane offset + scalar offset to M0 + lane * 16.
    static __device__ GG_INLINE void load_lane(u32x4 base, uint32_t lane_off, uint32_t off) {
        asm volatile("buffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(lane_off), "s"(base), "s"(off) : "memory");
    }
    static __device__ GG_INLINE void load_word(const char* p) { asm volatile("global_load_lds_dword %0, off" ::"v"(p) : "memory"); }
    static __device__ GG_INLINE void load_ptr(const char* p) { asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(p) : "memory"); }
    // acc += a . b with the accumulator in AGPRs, in place.  (From the builtin, in a kernel with as many loops as this
    // one, the compiler gives the result another register than the operand and then spends the loop moving accumulators
    // between the two halves of the register file: 340 moves per 128 MFMAs.)  The compiler waits for the LDS reads of a
    // and b, as it does for any use; what it does not know is that the instruction is an MFMA, so between setting an
    // accumulator and the first one, and between the last one and any other use, there has to be settle(), held in its
    // place by pin(): asm statements keep their order among each other, but an access to a register that they don't name may
    // cross them.  What C++ cannot forbid is that the compiler moves a register between two MFMAs;
    // tests/test_isa_hazards.py reads the built kernels for that.
    static __device__ GG_INLINE void mfma_acc(f32x4& acc, bf16x8 a, bf16x8 b) {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    }
    static __device__ GG_INLINE void settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }  // 19 wait states at most
    // Every write of the accumulators above this comes before it, every use below it after.
    template <int TFE>
    static __device__ GG_INLINE void pin(f32x4 (&acc)[kF][TFE]) {
#pragma unroll
        for (int j = 0; j < kF; ++j)
#pragma unroll
            for (int i = 0; i < TFE; ++i) asm volatile("" : "+a"(acc[j][i]));
    }
    // An accumulator element.  (Read where it is used: left to the compiler, all 256 are copied to VGPRs at once.)
    static __device__ GG_INLINE float from_acc(float a) {
        float v;
        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
        return v;
    }
    static constexpr int kWriteThrough = 16;  // cache policy bit sc1
    static __device__ GG_INLINE void wait_state() { asm volatile("s_nop 0" ::: "memory"); }

    // Buffer descriptor of the memory from `p` on (wave-uniform), without a bound of its own.
    static __device__ GG_INLINE u32x4 descriptor(const void* p) {
        const uint64_t a = reinterpret_cast<uint64_t>(p);
        u32x4 d;
        d[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
        d[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
        d[2] = 0xffffffffu;
        d[3] = 0x00020000u;
        return d;
    }

    // One work item: a tile, or a piece of one.
    struct Item {
        int rank, e, slot0, rows, ft, kt_begin, k_steps;
        float* out;          // where fp32 rows go
        uint32_t out_stride;
        int from;            // XCD whose list it is from
        bool incomplete;     // second GEMM, LINKED: the wait for its slot rows ran out
    };

    // Works through items, beginning with `cur`.  claim(from) takes the number of the next one off a list (one lane), settle_claim(n, item,
    // from) turns it into an item's number and its list (wavefront 0; -1: none left), and decode(item, from, Item&) says what that is.
    // claims: whether the lists have anything to claim.  In a GEMM of one round they have not, and the claim and the look at the other
    // lists would stand between a tile's last MFMA and its stores (hidden 4096, ffn 3584, 8 experts, 64 tokens, first GEMM 88.8 -> 83.0 us, second
    // 54.5 -> 48.1; hidden 4096, ffn 512, 16 experts, 200 tokens, first 51.2 -> 44.2).
    //
    // The wavefronts go from tile to tile without emptying the memory pipe: the next item is claimed two K steps before the end of a
    // tile; when the last operands have been read, its first weights, the row numbers of its slots and then its first slot rows are
    // requested, and the results of the finished tile are stored while they arrive.  The results go through LDS in an 8 KB
    // region per wavefront inside slot stage 1, so that the only barriers between two tiles are the one after the last operand reads
    // (which also publishes the next item) and the one before the first.  (With the claim, the look-up and all requests after the stores a
    // tile cost 6 us more than its K steps, 3 now.  While all CUs stream, others use the bandwidth meanwhile: whole layer, Phi shape, 200
    // tokens 381 -> 368 us, 64 experts of hidden 2048 and ffn 1408, 3000 tokens 437 -> 429, Mixtral shape 512 to 4096 tokens 0.3 to 0.7 %.)
    template <class Claim, class SettleClaim, class Decode>
    static __device__ GG_INLINE void run(const GemmArgs& a, unsigned char* lds, Item cur, const Claim& claim, const SettleClaim& settle_claim,
                                      const Decode& decode, bool claims, Link& link) {
        const int N = a.N, K = a.K;
        const lds_ptr lds3 = (lds_ptr)lds;
        const uint32_t lds0 = (uint32_t)(uintptr_t)lds3;
        const uint32_t row_bytes = (uint32_t)K * 2u;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int wt = wave & 1, wq = wave >> 1;      // slot group, weight-row group
        const uint32_t wave_lds = lds0 + (uint32_t)wave * 1024;
        auto next_w = [](uint32_t s) GG_LAMBDA { return s == 2 * kStage ? 0u : s + kStage; };

        // ---- staging: load q of wavefront w covers rows q * 32 + w * 8 .. + 7 of an operand tile, lane l the 16-byte
        // piece that belongs at position l % 8 of row l / 8 (see swizzled(); the same for every q).
        constexpr int kWOffs = 8 / NMAT;              // both matrices use the same lane offsets
        u32x4 base_a, base_b, base_s;
        uint32_t w_off[WIDE ? 1 : kWOffs];
        const char* w_ptr[WIDE ? 8 : 1];
        uint32_t s_off[WIDE || ALT ? 1 : 8];
        const char* s_ptr[WIDE || ALT ? 8 : 1];
        auto weight_load = [&](int q, uint32_t k_off) GG_LAMBDA {
            if constexpr (WIDE) load_ptr(w_ptr[q] + k_off);
            else load_lane(NMAT == 2 && q >= 4 ? base_b : base_a, w_off[q % kWOffs], k_off);
        };
        auto slot_load = [&](int q, uint32_t k_off) GG_LAMBDA {
            if constexpr (WIDE || ALT) load_ptr(s_ptr[q] + k_off);
            else load_lane(base_s, s_off[q], k_off);
        };
        auto weight_stage = [&](uint32_t stage, uint32_t k_off) GG_LAMBDA {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                set_lds_target(wave_lds + stage + q * 4096);
                wait_state();
                weight_load(q, k_off);
            }
        };
        auto slot_stage0 = [&](const Item& t) GG_LAMBDA {
            const int groups = (t.rows + 31) / 32;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q >= groups) break;
                set_lds_target(wave_lds + kSlotBase + q * 4096);
                wait_state();
                slot_load(q, (uint32_t)t.kt_begin * 128);
            }
        };
        // First requests of an item: the row numbers of its slots (first GEMM), which go to the weight stage `w0` + 2 (not used
        // before its third K step), and its first weights, into stage w0.  The second GEMM's slot rows are consecutive rows: the first ones go out as well.
        auto request_first = [&](Item& t, uint32_t w0) GG_LAMBDA {
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63;
            const int lrow = wave * 8 + (lane >> 3);
            const int chunk = swizzled(lrow, lane & 7);
            if constexpr (NMAT == 2) {  // lane l: the row that lanes 8 * (l % 8) ... of load l / 8 fetch
                const int r = min((lane >> 3) * 32 + wave * 8 + (lane & 7), t.rows - 1);  // rows past the end re-read the last valid row
                set_lds_target(lds0 + next_w(next_w(w0)) + kRowsOffset + (uint32_t)wave * 256);
                wait_state();
                load_word(reinterpret_cast<const char*>(a.row_of_slot + t.slot0 + r));
            }
            const int n0 = t.ft * kBF;
            const size_t w_first = ((size_t)t.e * N + n0) * K;
            base_a = descriptor(a.wa + w_first);
            base_b = descriptor(NMAT == 2 ? a.wb + w_first : a.wa + w_first);
#pragma unroll
            for (int q = 0; q < (WIDE ? 8 : kWOffs); ++q) {
                const int f = min((q % kWOffs) * 32 + lrow, N - 1 - n0);  // features past the end re-read the last one
                if constexpr (WIDE)
                    w_ptr[q] = reinterpret_cast<const char*>((NMAT == 2 && q >= 4 ? a.wb : a.wa) + w_first) + (size_t)f * row_bytes + (size_t)chunk * 16;
                else
                    w_off[q] = (uint32_t)f * row_bytes + (uint32_t)chunk * 16;
            }
            weight_stage(w0, (uint32_t)t.kt_begin * 128);
            if constexpr (NMAT == 1) {
                base_s = descriptor(a.tok + (size_t)t.slot0 * K);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = min(q * 32 + lrow, t.rows - 1);
                    if constexpr (WIDE)
                        s_ptr[q] = reinterpret_cast<const char*>(a.tok + (size_t)t.slot0 * K) + (size_t)r * row_bytes + (size_t)chunk * 16;
                    else
                        s_off[q] = (uint32_t)r * row_bytes + (uint32_t)chunk * 16;
                }
                if constexpr (LINKED) t.incomplete = !link.await(t.rank, lds + next_w(next_w(w0)) + kToldOffset);
                slot_stage0(t);
            }
        };
        // First GEMM: looks the slot rows up and requests those of the first K step.  At most eight loads (the weights) are younger than the row numbers.
        auto request_slots = [&](const Item& t, uint32_t w0) GG_LAMBDA {
            if constexpr (NMAT == 2) {
                int tid = threadIdx.x;
                asm volatile("" : "+v"(tid));
                const int lane = tid & 63;
                const int chunk = swizzled(wave * 8 + (lane >> 3), lane & 7);
                wait_vmcnt<8>();
                const int assignment = *reinterpret_cast<__attribute__((address_space(3))) const int*>(
                    lds3 + next_w(next_w(w0)) + kRowsOffset + wave * 256 + lane * 4);   // t * topk + j
                const int token = assignment / a.topk;
                if constexpr (WIDE || ALT) {
                    const bool from_alt = (ALT || a.alt_mask != nullptr) && a.alt_mask[assignment] != 0;
                    uint64_t tok = reinterpret_cast<uint64_t>(a.tok), alt = reinterpret_cast<uint64_t>(a.tok_alt);
                    asm volatile("" : "+s"(tok), "+s"(alt));  // (else the two are picked from an array in scratch memory)
                    const uint64_t at = (from_alt ? alt : tok) + (uint64_t)token * row_bytes;
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const int src = (q * 8 + (lane >> 3)) * 4;
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)at);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)(at >> 32));
                        s_ptr[q] = reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo) + chunk * 16;
                    }
                } else {
                    base_s = descriptor(a.tok);
                    const uint32_t at = (uint32_t)token * row_bytes;
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        s_off[q] = (uint32_t)__builtin_amdgcn_ds_bpermute((q * 8 + (lane >> 3)) * 4, (int)at) + (uint32_t)chunk * 16;
                }
                slot_stage0(t);
            }
        };

        uint32_t w0 = 0;  // weight stage of an item's first K step
        int finished = -1, stores = 0;  // first GEMM, LINKED: expert of the item before this one, and its stores
        request_first(cur, w0);
        request_slots(cur, w0);
        for (;;) {
        // (opaque, so that the compiler computes lane addresses where they are used instead of keeping those of every
        // version of the epilogue in registers across the whole kernel)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const int KT = cur.k_steps;
        const uint32_t k_first = (uint32_t)cur.kt_begin * 128;
        bool counted = !(LINKED && NMAT == 2) || KT <= 2;
        if (KT > 1) {
            weight_stage(next_w(w0), k_first + 128);
            if (counted) wait_vmcnt<8>();
            else wait_stores(stores);  // the first item's stores go through to memory: not waited for before the first K step
        } else {
            wait_vmcnt<0>();
        }
        lds_barrier();
        if constexpr (LINKED && NMAT == 2)
            if (counted && tid == 0 && finished >= 0) link.finish(finished);

        // ---- operand fragments: 16 rows x 32 K elements, lane l holds row l % 16, piece l / 16 of the half K step.
        // Row r, piece p sits at r * 128 + ((p ^ ((r >> 1) & 7)) << 4): fragments are 2048 bytes apart (the swizzle
        // repeats every 16 rows), the two halves of a K step differ in bit 6.
        // Weight fragment j: NMAT == 2 -> matrix j / 4, features wq * 64 + (j % 4) * 16; NMAT == 1 -> features
        // wq * 128 + j * 16.  Slot fragment i: slots (2 i + wt) * 16.
        const int frow = lane & 15, fpiece = lane >> 4;
        const uint32_t in_row = (uint32_t)(frow * 128 + ((((frow >> 1) & 7) ^ fpiece) << 4));
        const uint32_t w_read = (uint32_t)(wq * (NMAT == 2 ? 64 : 128)) * 128 + in_row;
        const uint32_t s_read = kSlotBase + (uint32_t)wt * 2048 + in_row;
        constexpr auto w_frag = [](int j) constexpr { return (uint32_t)(NMAT == 2 ? (j / 4) * 16384 + (j % 4) * 2048 : j * 2048); };

        Item next;
        bool more_items = false;
        // The whole tile for TFE valid 32-slot groups.  Everything from the accumulators to the stores is inside, so
        // that the eight versions have no code in common behind their loops (where they join, the compiler would have
        // to agree on registers for 256 accumulators and spills instead).
        auto tile = [&](auto tfe_c) GG_LAMBDA {
            constexpr int TFE = decltype(tfe_c)::value;
            f32x4 acc[kF][TFE];  // [weight fragment][slot fragment]
#pragma unroll
            for (int j = 0; j < kF; ++j)
#pragma unroll
                for (int i = 0; i < TFE; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
            pin(acc);
            settle();

            constexpr int kM = kF * TFE, kR = kF + TFE;
            bf16x8 wf[2][kF], tf[2][TFE];
            // Half a K step: the MFMAs of fragment buffer mbuf, between them the LDS reads of half `half` of the stages
            // at w_stage / s_stage into buffer 1 - mbuf, and the loads of one operand (LOADS 1: TFE slot loads, 2: 8
            // weight loads) for a later K step.
            auto half_step = [&](auto mfma, auto mbuf_c, auto read, int half, uint32_t w_stage, uint32_t s_stage, auto loads,
                                 uint32_t target, uint32_t k_off) GG_LAMBDA {
                constexpr int mbuf = decltype(mbuf_c)::value, rbuf = 1 - mbuf;
                constexpr int LOADS = decltype(loads)::value;
                constexpr int n_loads = LOADS == 1 ? TFE : LOADS == 2 ? 8 : 1;
                constexpr int gap = kM / n_loads;
                constexpr int read_slots = kM - kM / 8;   // the last reads get some MFMAs' time before they are used
                const lds_ptr wp = lds3 + ((w_read ^ (uint32_t)(half << 6)) + w_stage);
                const lds_ptr sp = lds3 + ((s_read ^ (uint32_t)(half << 6)) + s_stage);
#pragma unroll
                for (int m = 0; m < kM; ++m) {
                    if constexpr (decltype(mfma)::value) {
                        const int i = m / kF, j = m % kF;
                        mfma_acc(acc[j][i], wf[mbuf][j], tf[mbuf][i]);
                    }
                    if constexpr (decltype(read)::value) {
#pragma unroll
                        for (int x = 0; x < kR; ++x) {
                            if (x * read_slots / kR != m) continue;
                            if (x < kF)
                                wf[rbuf][x] = *reinterpret_cast<__attribute__((address_space(3))) const bf16x8*>(wp + w_frag(x));
                            else
                                tf[rbuf][x - kF] = *reinterpret_cast<__attribute__((address_space(3))) const bf16x8*>(sp + (x - kF) * 4096);
                        }
                    }
                    if constexpr (LOADS != 0) {
                        const int q = m / gap;
                        if (m % gap == 0) {
                            set_lds_target(target + q * 4096);
                            if (gap == 1) wait_state();
                        }
                        if (m % gap == gap / 2) {
                            if constexpr (LOADS == 1) slot_load(q, k_off);
                            else weight_load(q, k_off);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            using Buf0 = std::integral_constant<int, 0>;
            using Buf1 = std::integral_constant<int, 1>;
            using None = std::integral_constant<int, 0>;
            using Slots = std::integral_constant<int, 1>;
            using Weights = std::integral_constant<int, 2>;

            // first half of K step 0 into buffer 0; slots of K step 1 requested
            uint32_t w_stage = w0, s_stage = 0;                // of K step kt
            half_step(No{}, Buf1{}, Yes{}, 0, w_stage, s_stage, None{}, 0u, 0u);
            if (KT > 1) {
#pragma unroll
                for (int q = 0; q < TFE; ++q) {
                    set_lds_target(wave_lds + kSlotBase + kStage + q * 4096);
                    wait_state();
                    slot_load(q, k_first + 128);
                }
            }
            uint32_t k_off = k_first + 256;                    // of K step kt + 2
            auto k_step = [&](auto more) GG_LAMBDA {  // second half of K step kt, first half of K step kt + 1
                const uint32_t w1 = next_w(w_stage), w2 = next_w(w1), s1 = s_stage ^ kStage;
                // Stage w2 held K step kt - 1, which every wavefront had read before the last barrier.
                half_step(Yes{}, Buf0{}, Yes{}, 1, w_stage, s_stage, std::conditional_t<decltype(more)::value, Weights, None>{},
                          wave_lds + w2, k_off);
                // Outstanding, oldest first: weights of K step kt + 1, its slots, weights of K step kt + 2, or the first wavefront's claim.
                if constexpr (decltype(more)::value) wait_vmcnt<8>();
                else if (wave == 0 && claims) wait_vmcnt<1>();
                else wait_vmcnt<0>();
                lds_barrier();
                half_step(Yes{}, Buf1{}, Yes{}, 0, w1, s1, std::conditional_t<decltype(more)::value, Slots, None>{},
                          wave_lds + kSlotBase + s_stage, k_off);
                w_stage = w1;
                s_stage = s1;
                k_off += 128;
            };
            int kt = 0;
            for (int until = counted ? KT - 2 : 1;;) {
                for (; kt < until; ++kt) k_step(Yes{});
                if (counted) break;
                // The stores of the item before were older than what the first K step has waited for, in every wavefront.
                if constexpr (LINKED && NMAT == 2)
                    if (tid == 0 && finished >= 0) link.finish(finished);
                counted = true;
                until = KT - 2;
            }
            // The next item is claimed now; the answer is needed after the last K step.
            int claimed = 0;
            if (claims && tid == 0) claimed = claim(cur.from);
            if (KT > 1) k_step(No{});
            half_step(Yes{}, Buf0{}, Yes{}, 1, w_stage, s_stage, None{}, 0u, 0u);
            half_step(Yes{}, Buf1{}, No{}, 0, 0u, 0u, None{}, 0u, 0u);
            settle();
            pin(acc);

            if constexpr (LINKED && NMAT == 2) {
                finished = cur.e;
                stores = 2 * TFE;
            }
            // ---- the next item: its number and list in the weight stage that the last two K steps did not use
            const uint32_t handoff = next_w(w_stage);
            asm volatile("" ::"v"(claimed));  // (every wavefront waits here: where the answer may be outstanding, the main loop gets waits for it)
            if (wave == 0) {
                int item = -1, from = cur.from;
                if (claims) settle_claim(claimed, item, from);
                if (tid == 0) *reinterpret_cast<int2*>(lds + handoff) = make_int2(item, from);
            }
            lds_barrier();  // every wavefront is done reading operand tiles; no load is outstanding
            const int2 got = *reinterpret_cast<const int2*>(lds + handoff);
            const int item = __builtin_amdgcn_readfirstlane(got.x);
            w0 = next_w(handoff);  // (so that the stage with the number is the last to be written again)
            more_items = item >= 0;
            if (more_items) {
                decode(item, __builtin_amdgcn_readfirstlane(got.y), next);
                request_first(next, w0);
            }

            // ---- epilogue: transpose through LDS so that global stores are whole 128-byte lines, each wavefront by itself.
            // MFMA 16x16 result: lane holds column (slot) lane % 16 and rows (features) 4 * (lane / 16) + c.
            // LDS rows are XOR-swizzled in 16-byte units so that both ways are conflict free.
            unsigned char* own = lds + kSlotBase + kStage + wave * 8192;
            const int n0 = cur.ft * kBF;
            if constexpr (NMAT == 2 && !CUT) {
                // [up to 64 slots][64 features] bf16, 128-byte rows, unit v of row r at position v ^ ((r >> 1) & 7)
                const int n = n0 + wq * 64 + (lane & 7) * 8;
                const __amdgpu_buffer_rsrc_t act_rows = __builtin_amdgcn_make_buffer_rsrc(
                    static_cast<uint16_t*>(a.dst) + (size_t)cur.slot0 * N, 0, (int)((uint32_t)cur.rows * N * 2u), 0x00020000);
#pragma unroll
                for (int i4 = 0; i4 < TFE; i4 += 4) {
#pragma unroll
                    for (int i = i4; i < i4 + 4 && i < TFE; ++i) {
                        __builtin_amdgcn_sched_barrier(0);  // one fragment's values in registers at a time
                        const int lr = (i - i4) * 16 + frow;
#pragma unroll
                        for (int j = 0; j < kF / 2; ++j) {
                            float o[4];
#pragma unroll
                            for (int c = 0; c < 4; ++c) o[c] = swiglu(from_acc(acc[j][i][c]), from_acc(acc[kF / 2 + j][i][c]));
                            uint2 pk;
                            pk.x = pack_bf16x2(o[0], o[1]);
                            pk.y = pack_bf16x2(o[2], o[3]);
                            *reinterpret_cast<uint2*>(own + lr * 128 + (((j * 2 + (fpiece >> 1)) ^ ((lr >> 1) & 7)) << 4) + (fpiece & 1) * 8) = pk;
                        }
                    }
                    wave_order();
                    if (i4 == 0 && more_items) request_slots(next, w0);
#pragma unroll
                    for (int i = i4; i < i4 + 4 && i < TFE; ++i)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int lr = (i - i4) * 16 + h * 8 + (lane >> 3);
                            const int row = (2 * i + wt) * 16 + h * 8 + (lane >> 3);
                            const u32x4 v = *reinterpret_cast<const u32x4*>(own + lr * 128 + (((lane & 7) ^ ((lr >> 1) & 7)) << 4));
                            if constexpr (LINKED)  // (always issued, see wait_stores(): what does not exist lies past the end of the buffer)
                                __builtin_amdgcn_raw_buffer_store_b128(v, act_rows, n < N ? ((uint32_t)row * N + n) * 2u : ~15u, 0, kWriteThrough);
                            else if (row < cur.rows && n < N)
                                *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(a.dst) + (size_t)(cur.slot0 + row) * N + n) = v;
                        }
                    wave_order();
                }
            } else {
                // [16 slots][128 columns] fp32, 512-byte rows, unit v of row r at v ^ r.  Columns: NMAT == 1 wq * 128 + 0 .. 127;
                // NMAT == 2 64 of each matrix, wq * 64 + 0 .. 63 and 128 + wq * 64 + 0 .. 63.
                const int unit = lane & 31;
                const int col = NMAT == 1 ? wq * 128 + unit * 4 : (unit >> 4) * 128 + wq * 64 + (unit & 15) * 4;
                const bool stores = n0 + (col & (kBF - 1)) < N;
                if (more_items) request_slots(next, w0);
#pragma unroll
                for (int i = 0; i < TFE; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < kF; ++j) {
                        f32x4 v;
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = from_acc(acc[j][i][c]);
                        *reinterpret_cast<f32x4*>(own + frow * 512 + (((j * 4 + fpiece) ^ frow) << 4)) = v;
                    }
                    wave_order();
#pragma unroll
                    for (int h = 0; h < 8; ++h) {
                        const int lr = h * 2 + (lane >> 5);
                        const int row = (2 * i + wt) * 16 + lr;
                        f32x4 v = *reinterpret_cast<const f32x4*>(own + lr * 512 + ((unit ^ lr) << 4));
                        if constexpr (LINKED)
                            if (cur.incomplete) v = f32x4{NAN, NAN, NAN, NAN};
                        if (row < cur.rows && stores) *reinterpret_cast<f32x4*>(cur.out + (size_t)row * cur.out_stride + col) = v;
                    }
                    wave_order();
                }
            }
        };
        switch (__builtin_amdgcn_readfirstlane((cur.rows + 31) / 32)) {
            case 1: tile(std::integral_constant<int, 1>{}); break;
            case 2: tile(std::integral_constant<int, 2>{}); break;
            case 3: tile(std::integral_constant<int, 3>{}); break;
            case 4: tile(std::integral_constant<int, 4>{}); break;
            case 5: tile(std::integral_constant<int, 5>{}); break;
            case 6: tile(std::integral_constant<int, 6>{}); break;
            case 7: tile(std::integral_constant<int, 7>{}); break;
            default: tile(std::integral_constant<int, 8>{}); break;
        }
        if (!more_items) break;
        cur = next;
        }
        if constexpr (LINKED && NMAT == 2) {
            wait_vmcnt<0>();
            lds_barrier();  // (and nobody reads the last item's number any more)
            if (threadIdx.x == 0) link.finish(finished);
        }
    }
};

// Operands of this many bytes and more are addressed with 64-bit pointers: a lane offset plus the K offset must fit 32 bits and
// stay below the bound of the buffer descriptor.
constexpr size_t kWideBytes = (size_t)15 << 28;
// Whether a GEMM needs the WIDE kernel: `gathered` is the size of the tensor that slot rows are gathered from (0 where they
// are a tile's consecutive rows), `tile_rows` the weight or slot rows that are addressed from one base.
constexpr bool needs_wide(size_t gathered, size_t tile_rows, size_t k_elements) {
    return gathered >= kWideBytes || tile_rows * k_elements * 2 >= kWideBytes;
}

// Slots per tile and parts of a leftover tile for the second GEMM.  A smaller tile costs less per round, but there are more of
// them; more parts make a shorter last round, but each is a prologue and an epilogue, and rows that are written and read again.
// Lane l prices one of the 30 plans (slots 256 - 32 * (l / 6), l % 6 + 1 parts); the first of the cheapest is taken.  In 10 ns:
//   the larger of   full rounds x (K steps x (90 + 6 x slots / 32) + 400) and the same for the rounds of pieces  (MFMAs)
//            and    the active experts' weights at 6.6 TB/s + 600 a round                                       (memory)
//   + 300 + 2 a unit of 32 rows of pieces, if there are any.
// Fitted to all plans of 72 shapes, 33 to 3400 tokens, 4 to 64 experts, 8 to 224 K steps, the combination's time included, and
// with 36 others: chosen plans are 1.3 % above the best on average and 8.6 % at most.  (The MFMA term alone, with 14 K
// steps or more a part, as it was: 4.4 % and 46 %; Phi shape, 200 tokens, 152 + 12 us in four parts where 131 + 6 is had in one;
// 16 experts, hidden 640, ffn 1728, 627 tokens: 34 -> 23 us.)  The lanes do it side by side because 30 prices one after the
// other take 2 us.
__device__ GG_INLINE void choose_plan(const TileList& list, int N, int KT, int members, int& slots, int& parts) {
    static_assert(kMaxParts == 6, "30 plans");
    const int lane = threadIdx.x & 63;
    const int i = min(lane / 6, 4), p = lane - lane / 6 * 6 + 1, s = 256 - 32 * i;
    int sums[6] = {TileList::units_of(list.count)};
#pragma unroll
    for (int n = 0; n < 5; ++n) sums[n + 1] = list.slot_tiles(256 - 32 * n);
    const int most_rows = __builtin_amdgcn_readlane(list.count, 0);
    const int active = __popcll(__ballot(list.count > 0));
    wave_totals(sums);
    int tiles = sums[1];
#pragma unroll
    for (int n = 1; n < 5; ++n) tiles = i == n ? sums[n + 1] : tiles;
    tiles *= list.n_ft;
    const int full = tiles / (kXcds * members), left = tiles - full * (kXcds * members);
    const int chunk = (left + kXcds - 1) / kXcds;
    const int units = min(left * TileList::units_of(min(s, most_rows)), sums[0] * list.n_ft);  // of the leftover tiles, at most
    const int rounds = (chunk * p + members - 1) / members;
    const bool allowed = p == 1 || (chunk > 0 && units * (p - 1) <= kScratchUnits && KT >= p * kMinPartKSteps);
    const float step = 90 + 6 * s / 32;
    const float work = full * (KT * step + 400.f) + rounds * ((KT + p - 1) / p * step + 400.f);
    const float stream = active * (float)N * KT * (1.f / 516.f) + (full + rounds) * 600.f;
    float cost = fmaxf(work, stream) + (p > 1 ? 300.f + 2.f * units * (p - 1) : 0.f);
    if (lane >= 30 || !allowed) cost = INFINITY;
    float best = cost;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) best = fminf(best, __shfl_xor(best, d, 64));
    const int winner = __ffsll((long long)__ballot(cost == best)) - 1;
    slots = __builtin_amdgcn_readlane(s, winner);
    parts = __builtin_amdgcn_readlane(p, winner);
}

// Parts of the first GEMM's tiles in calls of few tiles (CUT): priced as in choose_plan(), for one height of tiles and with all
// parts in the scratch memory.  Lane l prices l + 1 parts.
constexpr int kMaxCutParts = 8;
// Most tiles that such a call can have, which the launcher knows from the token count, and the fewest K steps.  Few tiles leave most CUs
// idle for a whole K loop; cut, they keep them busy for part of one, but the other kernel takes 6 us.  First GEMM, whole / cut:
// 16 tiles of 64 K steps 51 / 23 us, 32 52 / 31, 84 56 / 47, 96 of 48 56 / 51, 48 of 24 27 / 22, 88 of 25 29 / 27; but 128 of 64 with few
// rows, which as they are stream at 4 TB/s, 70 / 79, 128 of 32 36 / 38, 64 of 16 20 / 21, 32 of 16 15 / 17.
constexpr int kMaxCutTiles = 96, kMinCutKSteps = 24;

__device__ GG_INLINE void choose_cut(const TileList& list, int N, int KT, int members, int& parts) {
    const int p = (threadIdx.x & 63) + 1;
    const int most_rows = __builtin_amdgcn_readlane(list.count, 0);
    const int active = __popcll(__ballot(list.count > 0));
    int sums[2] = {TileList::units_of(list.count), list.slot_tiles(256)};
    wave_totals(sums);
    const int units = sums[0] * list.n_ft, chunk = (sums[1] * list.n_ft + kXcds - 1) / kXcds;
    const int rounds = (chunk * p + members - 1) / members;
    const float step = 90 + 6 * TileList::units_of(min(256, most_rows));
    const float work = rounds * ((KT + p - 1) / p * step + 400.f);
    const float stream = active * 2.f * N * KT * (1.f / 516.f) + rounds * 600.f;
    float cost = fmaxf(work, stream) + 2.f * units * p;
    if (p > 1 && (p > kMaxCutParts || units * p > kScratchUnits || KT < p * kMinPartKSteps)) cost = INFINITY;
    float best = cost;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) best = fminf(best, __shfl_xor(best, d, 64));
    parts = __ffsll((long long)__ballot(cost == best));
}

// Persistent schedule: the grid is one workgroup per CU.  Workgroup b belongs to XCD b % 8 (the
// hardware deals workgroups round-robin to the XCDs) and is its member b / 8.  An XCD works
// through the tile list in rounds of `members` consecutive tiles, so that its workgroups work on
// tiles that share operand lines at about the same time and most lines are pulled into the
// XCD's L2 once per round instead of once per workgroup.  A workgroup starts with the tile of
// its member number (or, see owns_first(), with one that it claims) and then takes the XCD's next tile from a counter whenever it has finished
// one: tiles differ in cost (ragged slot tiles skip the MFMAs of their empty fragments, tiles
// of cold experts wait for memory), and the members of a round don't wait for each other.  Letting the members drift
// apart by a fraction of a K step is also faster than holding them in step, because fewer of
// them then ask for the same line at the same moment.
//
// Hot experts' tiles are bound by the MFMAs, those of an expert with a single slot tile by streaming its weights from
// memory, and a CU alone can pull 40 GB/s from memory where 256 at once get 23 each.  So rounds of the two kinds are
// interleaved in proportion, and among the light ones the ones with more rows and with fewer rows in turn (first GEMM
// at 2048 tokens of the Phi shape: 507 -> 460 us; with all experts' tiles in descending order the light rounds take as
// long as their bytes at the full chip's rate).
//
// Second GEMM: it has few tiles with many K steps (2048 tokens of the Mixtral shape: 320 tiles of 224 K steps for 256
// CUs), so what the last round costs matters.  The tiles left over after the last full round are cut along K into
// `parts` pieces, handed out like tiles; see SplitTable for their sums, choose_plan() for their number.
// The first GEMM has many short tiles (4096 tokens: 15 rounds); cutting its leftover tiles gained nothing.  For calls in which it
// has few, see choose_cut().
//
// Which tiles are left over: the last ones, those of the coldest experts, except in a second GEMM of one full round of which
// hot tiles alone would fill 7 tenths or more.  Such a round is bound by the MFMAs and the leftovers by memory, with little to
// interleave; so the leftovers are taken from around the border of the two kinds in their proportion.  Phi shape, second GEMM,
// leftovers at the end / amid: 900, 1300 and 1500 tokens (160 of 256 hot tiles) 193 / 202, 211 / 222, 221 / 232 us; 1700, 2048 and
// 2300 tokens (192 and more) 270 / 253, 298 / 276, 322 / 292; Mixtral shape, 2600 tokens 511 / 493.  (With more full rounds it
// only moves hot tiles to the end, 3500 tokens: 372 -> 387 us, first GEMM at 600 tokens: 326 -> 335 us).
//
// A workgroup whose XCD has handed out all its items takes one from the XCD with most left, in calls with at least 48 K steps.
// The look at the counters costs each GEMM about 1.5 us at its end and tiles taken over share fewer lines: 22 K steps, the
// 64-expert shape at 1003 tokens, first GEMM 100.5 -> 103 us with it.  Between 32 and 64 K steps it does not matter (eight
// shapes, hidden and ffn 2048 to 3584: within 2 % either way).  With 64 and 100 of the Phi shape, 700 tokens, 523 -> 509 us; 64 and
// 224 of the Mixtral shape, 512 tokens, 630 -> 625, 4096 tokens, both GEMMs, 2168 -> 2164.
// claimed: thread 0's first claim of its XCD's counter, where workgroups don't own their first item (see owns_first()).  Returns the
// slots per tile.
template <class G>
__device__ GG_INLINE int persistent(const GemmArgs& a, unsigned char* lds, TileList list, Link& link, int claimed = 0) {
    list.n_ft = (a.N + G::kBF - 1) / G::kBF;
    const int KT = a.K / 64;
    const int xcd = blockIdx.x % kXcds, member = blockIdx.x / kXcds;
    const int members = min((int)gridDim.x / kXcds, kMaxWgsPerXcd);
    const int per_super_round = kXcds * members;
    int slots = 256, parts = 1;
    if constexpr (G::kMats == 1) choose_plan(list, a.N, KT, members, slots, parts);
    if constexpr (G::kCut) choose_cut(list, a.N, KT, members, parts);
    list.build(slots);
    if constexpr (G::kMats == 2 && !G::kCut) {
        // A call whose tiles are one round takes the lowest ones with which it still is: a K step takes less time (hidden 4096,
        // ffn 2048, 8 experts, 256 tokens 77 -> 67 us; hidden 3584, ffn 1088, 8 experts, 509 tokens 72 -> 63; no shape is slower).
        if (list.total <= per_super_round && __builtin_amdgcn_readlane(list.count, 0) > 128) {
            int tiles[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) tiles[n] = list.slot_tiles(128 + 32 * n);
            wave_totals(tiles);
#pragma unroll
            for (int n = 3; n >= 0; --n)
                if (tiles[n] * list.n_ft <= per_super_round) slots = 128 + 32 * n;
            list.build(slots);
        }
    }
    const int total = list.total;
    const int full_rounds = G::kCut ? 0 : total / per_super_round;  // (CUT: every tile counts as left over)
    const int left = total - full_rounds * per_super_round;
    const int chunk = (left + kXcds - 1) / kXcds;
    const bool amid = G::kMats == 1 && full_rounds == 1 && list.heavy * 10 >= 7 * per_super_round;  // (see above)
    const int first_left = amid ? list.heavy - (int)((long)left * list.heavy / total) : total - left;
    int first_unit = 0, n_units = 0;  // of the leftover tiles
    if (parts > 1 || G::kCut) {
        int r, e, slot0, rows, ft;
        list.count_units();
        list.find(first_left, r, e, slot0, rows, ft, first_unit);
        n_units = list.units;
        if (first_left + left < total) list.find(first_left + left, r, e, slot0, rows, ft, n_units);
        n_units -= first_unit;
    }
    if ((G::kMats == 1 || G::kCut) && blockIdx.x == 0 && threadIdx.x < 64) {
        SplitTable* table = a.table;
        if (threadIdx.x == 0) {
            table->slots = slots;
            table->parts = parts;
            table->first_split = first_left;
            table->n_split = left;
            table->first_unit = first_unit;
            table->n_units = n_units;
        }
        if (threadIdx.x < a.E) {
            table->first_tile[list.expert] = list.first_tile;
            table->units_before[list.expert] = list.first_unit;
        }
    }
    // Work items of an XCD in hand-out order: its whole tiles, then the pieces of its leftover tiles.
    const int n_whole = full_rounds * members;
    constexpr bool kOwnsFirst = owns_first(G::kLinked, G::kMats);
    const HandOut<kOwnsFirst> hand{members, n_whole, left, chunk, parts};
    // rounds of `members` whole tiles that lie in the heavy part of the list / in the rest
    const int n_rounds = full_rounds * kXcds;
    const int heavy_rounds = min(n_rounds, min(list.heavy, first_left) / members);
    const int light_rounds = n_rounds - heavy_rounds;
    // round * light_rounds / n_rounds by multiplication (any spacing does that takes every light round once, in order)
    const uint32_t light_step = n_rounds > 0 ? (uint32_t)(((uint64_t)(uint32_t)light_rounds << 32) / (uint32_t)n_rounds) + 1u : 0u;
    auto light_before = [&](int round) GG_LAMBDA { return light_rounds == n_rounds ? round : (int)__umulhi((uint32_t)round, light_step); };
    // Item `item` of XCD `from`, see above.
    auto decode = [&](int item, int from, typename G::Item& t) GG_LAMBDA {
        int tile_index, part = 0;
        if (item >= n_whole) {
            const int rem = hand.left_of(from), q = item - n_whole;  // piece number
            part = q / rem;
            tile_index = first_left + from * chunk + q - part * rem;
            t.kt_begin = uniform(KT * part / parts);
            t.k_steps = uniform(KT * (part + 1) / parts) - t.kt_begin;
        } else {
            int round = item / members;
            const int at = item - round * members;
            round = round * kXcds + from;
            const int l0 = light_before(round), l1 = light_before(round + 1);
            round = l1 > l0 ? heavy_rounds + ((l0 & 1) != 0 ? light_rounds - 1 - l0 / 2 : l0 / 2) : round - l0;
            tile_index = round * members + at;
            if (tile_index >= first_left) tile_index += left;
            t.kt_begin = 0;
            t.k_steps = KT;
        }
        int unit;
        list.find(tile_index, t.rank, t.e, t.slot0, t.rows, t.ft, unit);
        t.slot0 = uniform(t.slot0);
        t.rows = uniform(t.rows);
        t.ft = uniform(t.ft);
        t.from = from;
        if constexpr (G::kFp32) {
            t.out = static_cast<float*>(a.dst) + (size_t)t.slot0 * a.N + t.ft * G::kBF;
            t.out_stride = (uint32_t)a.N;
            if (part > 0 || G::kCut) {
                t.out = a.scratch + (size_t)uniform((G::kCut ? part : part - 1) * n_units + unit - first_unit) * kUnitFloats;
                t.out_stride = 256;
            }
        }
    };
    auto claim = [&](int from) GG_LAMBDA {
        int counter = from;
        asm volatile("" : "+v"(counter));  // (at an address that the compiler knows to be uniform it reads the result at once, and waits)
        return __hip_atomic_fetch_add(&a.sync[counter], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto settle_claim = [&](int n, int& item, int& from) GG_LAMBDA {
        item = hand.claimed(__builtin_amdgcn_readfirstlane(n), from);
        if (item >= 0) return;
        // That XCD's items are all handed out: go on with one of the XCD that has most left.
        if (KT < kMinStealKSteps && !(G::kLinked && G::kMats == 2)) return;
        const int lane = threadIdx.x & 63;
        for (;;) {  // a try that loses the race has seen the victim's last item go: the sum of `open` falls every time
            int open = lane < kXcds ? hand.open(lane, __hip_atomic_load(&a.sync[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0;
            int most = 0;
            for (int x = 0; x < kXcds; ++x) {
                const int o = __builtin_amdgcn_readlane(open, x);
                if (o > most) { most = o; from = x; }
            }
            if (most == 0) return;
            int got = 0;
            if (lane == 0) got = __hip_atomic_fetch_add(&a.sync[from], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            item = hand.claimed(__builtin_amdgcn_readfirstlane(got), from);
            if (item >= 0) return;
        }
    };
    int item = hand.first(member, xcd), from = xcd;
    if (item < 0) {
        // (no item of its own: it takes one like everybody's second, or, where the XCD has fewer items than workgroups, looks elsewhere at once)
        int* handoff = reinterpret_cast<int*>(lds);
        if (!hand.any()) return slots;
        if (threadIdx.x < 64) {
            settle_claim(kOwnsFirst ? hand.items(xcd) : claimed, item, from);
            if (threadIdx.x == 0) {
                handoff[0] = item;
                handoff[1] = from;
            }
        }
        lds_barrier();
        item = __builtin_amdgcn_readfirstlane(handoff[0]);
        from = __builtin_amdgcn_readfirstlane(handoff[1]);
        lds_barrier();  // (loads into this memory follow)
        if (item < 0) return slots;
    }
    typename G::Item first;
    decode(item, from, first);
    G::run(a, lds, first, claim, settle_claim, decode, hand.any(), link);
    return slots;
}

template <class G>
__global__ __launch_bounds__(G::kThreads, 1) void grouped_gemm_kernel(GemmArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_dyn[];
    if ((int)blockIdx.x / kXcds >= min((int)gridDim.x / kXcds, kMaxWgsPerXcd)) return;
    Link link{};
    persistent<G>(a, lds_dyn, TileList(a.offs, a.E), link);
}

// Both GEMMs, see Link.  First: Gemm<2, ALT, false, false, true>.
template <class First>
__global__ __launch_bounds__(First::kThreads, 1) void linked_grouped_gemm_kernel(GemmArgs a, GemmArgs b, int32_t* done, uint32_t* status, int spin_limit) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds_dyn[];
    if ((int)blockIdx.x / kXcds >= min((int)gridDim.x / kXcds, kMaxWgsPerXcd)) return;
    int claimed = 0;  // (requested before the list is built)
    if (threadIdx.x == 0) claimed = __hip_atomic_fetch_add(&a.sync[blockIdx.x % kXcds], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const TileList list(a.offs, a.E);
    Link link{done, status, spin_limit, 0, 0, 0, nullptr};
    const int slots = persistent<First>(a, lds_dyn, list, link, claimed);
    link.need = list.slot_tiles(slots) * ((a.N + First::kBF - 1) / First::kBF);
    link.expert = list.count > 0 ? list.expert : 0;
    persistent<Gemm<1, false, false, false, true>>(b, lds_dyn, list, link);
}

}  // namespace gg
}  // namespace moe
