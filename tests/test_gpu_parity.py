"""Parity of the HIP library (through its C ABI) with the CPU oracle, element by element,
at sizes the oracle finishes in seconds: several tiles, ragged tails, degenerate cases."""
import numpy as np
import pytest
import torch

from paper_2501_10375_amd import moe, synth
from parity_util import (check_layer, check_routing, host, output_error, second_gemm_plan, second_gemm_tiles, tile_aware_sample,
                         to_f64)

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _run(T, H, F, E, k, dtype, seed=0, zipf=1.2, predict=True):
    d = synth.moe_layer_inputs(T, H, F, E, dtype, DEV, seed=seed, zipf_s=zipf, with_next=predict)
    shape = moe.make_shape(H, F, E, k, dtype)
    out = moe.LayerOutputs(shape, max(T, 1), dtype, DEV, predict=predict)
    res = moe.run_layer(shape, d, out, predict=predict)
    return d, shape, out, res


def test_config0_tiny_fp32_layer(oracle):
    d, shape, out, res = _run(64, 256, 512, 8, 2, torch.float32)
    r = check_layer(oracle, d, shape, res, torch.float32, label="config0")
    print("config0", r)
    assert r["compared_tokens"] >= 60


@pytest.mark.parametrize("T,H,F,E,k", [
    (300, 256, 512, 8, 2),     # about 75 rows an expert: ragged slot tiles of one to several 32-slot groups
    (129, 128, 192, 4, 2),     # F not a multiple of the 128 feature tile
    (77, 64, 64, 16, 2),       # smallest legal widths, many cold experts
    (200, 256, 256, 8, 1),     # top-1
    (50, 128, 256, 8, 4),      # top-4
    (40, 128, 128, 64, 8),     # widest router, top-8
    (17, 256, 512, 8, 2),      # just above the decode threshold
    (90, 192, 128, 32, 3),     # two 16-expert blocks in the router
    (40, 8192, 128, 8, 2),     # hidden dimension longer than one register chunk of the router
    (60, 128, 128, 12, 3),     # expert count that is not a power of two
    (32, 256, 512, 8, 2), (33, 256, 320, 16, 2), (64, 256, 512, 8, 2), (65, 256, 512, 8, 2),   # weight-streaming sizes and the first size past them
])
def test_bf16_prefill_path(oracle, T, H, F, E, k):
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 T={T}")
    print(r)


@pytest.mark.parametrize("T,H,F,E,k", [
    (1100, 256, 512, 2, 2),    # ~9 slot tiles of 256, everything in one round whose tiles are split along K
    (700, 512, 384, 1, 1),     # one expert, top-1: a dense SwiGLU MLP; F = 3 feature tiles of gemm1
    (1300, 320, 448, 2, 2),    # F ends in a half feature tile, K = 5 steps of 64 (odd number of ring turns)
    (2100, 1024, 320, 4, 2),   # 16 K steps: the weight ring wraps 5 times; ragged last slot tiles
    (3000, 256, 2048, 2, 2),   # more tiles than compute units: one full round, then a split round
])
def test_bf16_full_tile_flavour_every_token(oracle, T, H, F, E, k):
    """Calls with at least 512 routed rows per expert, as long prefill calls have them: full slot tiles of up to 256 slots.
    Narrow layers let the oracle check every token, so every wavefront's fragment rows and every epilogue position of
    the 256 x 256 tile is compared, including tiles whose K range is split between workgroups."""
    assert T * k >= E * 512
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 full tiles T={T}")
    print(r)
    assert r["compared_tokens"] >= T - r["excluded"] - 2


@pytest.mark.parametrize("T,H,F,E,k,seed", [
    (200, 256, 256, 2, 2, 0),    # 200 rows per expert: one ragged tile of seven 32-slot groups each
    (150, 256, 384, 4, 4, 1),    # hot expert: a full slot tile and a short one; cold experts: one or two fragments
    (330, 320, 448, 2, 2, 2),    # second slot tile of every expert ragged
    (140, 128, 640, 1, 1, 3),    # one expert with 140 rows: five 32-slot groups, the last of 12 rows
    (520, 192, 256, 8, 2, 4),    # 130 rows per expert on average: cold experts below one group
    (300, 256, 512, 2, 1, 5),    # top-1, about 150 rows per expert
])
def test_bf16_ragged_fragments_of_full_tiles_every_token(oracle, T, H, F, E, k, seed):
    """A ragged slot tile computes and stages only the 32-slot groups that have slots (a main loop per number of
    groups, 1 to 8).  Every token is compared; the numbers of groups that these shapes leave out are in
    test_bf16_slot_groups_and_short_k_loops."""
    assert E * 128 <= T * k
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16, seed=seed)
    counts = res["counts"].cpu().tolist()
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 T={T} ragged fragments")
    print(r, "rows per expert:", counts)
    assert r["compared_tokens"] >= T - r["excluded"] - 2


@pytest.mark.parametrize("T,H,F", [
    (320, 64, 64), (352, 128, 192), (384, 192, 128), (401, 64, 320), (440, 320, 64), (470, 256, 128), (512, 128, 64),
    (513, 192, 192), (545, 64, 128),
])
def test_bf16_slot_groups_and_short_k_loops(oracle, T, H, F):
    """One expert, so the last slot tile of the call has T - 256 (or T - 512) rows: 1 to 8 groups of 32 slots,
    among them single rows of a group; 1 to 5 K steps of 64 in each GEMM (the loop's first and last K steps are
    separate code).  Every token is compared; the tolerance is the layer's (two roundings to bf16)."""
    d, shape, out, res = _run(T, H, F, 1, 1, torch.bfloat16, seed=T)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 T={T} one expert")
    print(r)
    assert r["compared_tokens"] == T


@pytest.mark.parametrize("T,H,F,E,k", [
    (70, 320, 1856, 5, 3),      # 29 K steps in the second GEMM: two parts at most; the last feature tile is a quarter one
    (257, 64, 3584, 1, 1),      # one expert: a full slot tile and one with a single row, cut into up to 4 parts
    (900, 512, 5504, 4, 2),     # 86 K steps that the parts do not divide; slot tiles of unequal height
    (34, 4096, 896, 64, 8),     # more tiles than compute units: whole tiles first, then 14-step pieces of the coldest experts
    (1200, 2048, 1792, 6, 2),   # hot experts whose slot tiles are shared, leftover tiles among them
    (2700, 320, 1792, 2, 1),    # more slot tiles an expert than a group holds, the last ones ragged, all cut
    (2300, 256, 2048, 3, 2),    # the same with a single feature tile and two groups of different size
    (333, 576, 5376, 7, 3),     # ragged single slot tiles of every expert, pieces without gaps between them
    (64, 512, 1152, 2, 2),      # 18 K steps, 6 parts of 3
    (50, 2112, 1216, 3, 1),     # 19 K steps: parts of unequal length
    (290, 640, 320, 4, 2),      # 5 K steps: whole tiles only
])
def test_bf16_second_gemm_pieces_every_token(oracle, T, H, F, E, k):
    """The second GEMM cuts the tiles left over after its last full round along K; their pieces are added by the kernel
    that combines a token's selections.  Every token is compared."""
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16, seed=T + E)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 T={T} pieces")
    print(r)
    assert r["compared_tokens"] >= T - r["excluded"] - 2


@pytest.mark.parametrize("gib,precalc", [(3, False), (4, False), (4, True)])
def test_bf16_hidden_states_of_many_gib(oracle, gib, precalc):
    """Row offsets of x around 32 bits: at 3 GiB lane offsets have their top bit set; past 3.75 GiB the first GEMM
    addresses slot rows with 64-bit pointers, of two tensors with selections pre-calculated on another input.  Compared on
    tokens from both ends of x (tokens are independent, so the oracle gets those rows alone)."""
    H, F, E, k, dtype = 4096, 64, 2, 1, torch.bfloat16
    T = (gib << 30) // (2 * H) + 300
    d = synth.moe_layer_inputs(1, H, F, E, dtype, DEV, seed=5, with_next=False)
    g = torch.Generator(device=DEV).manual_seed(9)
    x = torch.randn((T, H), generator=g, dtype=dtype, device=DEV)
    idx = (torch.arange(T, device=DEV, dtype=torch.int32) % 3 == 0).int().reshape(T, 1)
    w = torch.ones((T, 1), dtype=torch.float32, device=DEV)
    y = torch.empty((T, H), dtype=dtype, device=DEV)
    shape = moe.make_shape(H, F, E, k, dtype)
    ws = moe.alloc_workspace(shape, T)
    if precalc:
        x_stale = torch.randn((T, H), generator=g, dtype=dtype, device=DEV)
        stale = (torch.arange(T, device=DEV) % 2).to(torch.uint8).reshape(T, 1)
        moe.moe_expert_ffn_precalc(shape, x, x_stale, stale, idx, w, d["w1"], d["w3"], d["w2"], y, ws)
        x = torch.where(stale != 0, x_stale, x)  # what each selection was evaluated on
    else:
        moe.moe_expert_ffn(shape, x, idx, w, d["w1"], d["w3"], d["w2"], y, ws)
    torch.cuda.synchronize()
    tok = torch.cat([torch.arange(0, 40), torch.arange(T // 2, T // 2 + 40), torch.arange(T - 350, T)])
    h = host(d)
    ref = oracle.expert_ffn(synth.to_numpy(x[tok.to(DEV)]), idx[tok.to(DEV)].cpu().numpy(),
                            w[tok.to(DEV)].cpu().numpy().astype(np.float64), h["w1"], h["w3"], h["w2"])
    assert output_error(to_f64(y[tok.to(DEV)]), ref) <= 2e-2


@pytest.mark.parametrize("T,H,F,E,k", [
    (33, 1536, 64, 1, 1),        # one tile, half a feature tile; 24 K steps: the shortest rows that are cut, 8 parts
    (100, 4096, 512, 8, 2),      # 32 tiles, 8 parts of 8 K steps
    (70, 1664, 320, 5, 3),       # 26 K steps: parts of unequal length; the last feature tile is half
    (64, 2048, 2048, 8, 2),      # 128 tiles: the most that are cut
    (64, 2048, 2112, 8, 2),      # one more feature tile: not cut
    (2500, 1536, 192, 4, 3),     # several slot tiles an expert, the last ones ragged
    (4000, 1536, 128, 1, 1),     # more slot tiles than a group of the tile list holds
    (40, 1536, 128, 64, 1),      # experts without rows
])
def test_bf16_first_gemm_pieces_every_token(oracle, T, H, F, E, k):
    """In calls of few tiles the first GEMM cuts all of them along K and another kernel adds the pieces and applies SwiGLU.
    Every token is compared, and every selection of moe_expert_ffn_precalc once with mixed inputs."""
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16, seed=T + E)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 T={T} first GEMM cut")
    print(r)
    assert r["compared_tokens"] >= T - r["excluded"] - 2
    x_stale = synth.normal((T, H), 99, 3, 1.0, torch.bfloat16, DEV)
    g = torch.Generator().manual_seed(T)
    stale = (torch.rand((T, k), generator=g) < 0.4).to(torch.uint8).to(DEV)
    y = torch.empty_like(d["x"])
    for mask, want in ((torch.zeros_like(stale), None), (stale, "mixed")):
        moe.moe_expert_ffn_precalc(shape, d["x"], x_stale, mask, res["idx"], res["w"], d["w1"], d["w3"], d["w2"], y, out.workspace)
        torch.cuda.synchronize()
        if want is None:
            assert torch.equal(y, res["y"])
        else:
            h = host(d)
            ref = oracle.expert_ffn_precalc(h["x"], synth.to_numpy(x_stale), mask.cpu().numpy(), res["idx"].cpu().numpy(),
                                            res["w"].cpu().numpy().astype(np.float64), h["w1"], h["w3"], h["w2"])
            assert output_error(to_f64(y), ref) <= 2e-2


def _swiglu_expert_rows(x, w1, w3, w2, chunk=1 << 20):
    """One expert on a few rows as plain torch: fp32 products, fp64 sums, the intermediate rounded to bf16."""
    H, F = w1.shape[1], w1.shape[0]
    g = torch.zeros((x.shape[0], F), dtype=torch.float64, device=x.device)
    u = torch.zeros_like(g)
    for h in range(0, H, chunk):
        for f in range(0, F, chunk):
            xs = x[:, h:h + chunk].float()
            g[:, f:f + chunk] += (xs @ w1[f:f + chunk, h:h + chunk].float().T).double()
            u[:, f:f + chunk] += (xs @ w3[f:f + chunk, h:h + chunk].float().T).double()
    act = (torch.nn.functional.silu(g) * u).to(torch.bfloat16)
    y = torch.zeros((x.shape[0], H), dtype=torch.float32, device=x.device)
    for h in range(0, H, chunk):
        s = torch.zeros((x.shape[0], min(chunk, H - h)), dtype=torch.float64, device=x.device)
        for f in range(0, F, chunk):
            s += (act[:, f:f + chunk].float() @ w2[h:h + chunk, f:f + chunk].float().T).double()
        y[:, h:h + chunk] = s.float()
    return y


@pytest.mark.parametrize("T,H,F", [
    (257, 256, (1 << 23) + (1 << 20)),   # second GEMM: 256 rows of act or of w2 span more than 4 GiB
    (34, (1 << 24) + (1 << 20), 128),    # first GEMM: 128 rows of w1 or w3 do
])
def test_bf16_rows_of_a_tile_span_more_than_4_gib(T, H, F):
    """Very long rows are accepted and computed like any other: offsets within a tile then exceed 32 bits.  The second
    call takes every other selection from another tensor (moe_expert_ffn_precalc).  Rows of the tile's end are compared."""
    g = torch.Generator(device=DEV).manual_seed(F)

    def normal(shape, std):
        return torch.randn(shape, generator=g, dtype=torch.bfloat16, device=DEV).mul_(std)

    x, x_stale = normal((T, H), 1.0), normal((T, H), 1.0)
    w1, w3, w2 = normal((1, F, H), H ** -0.5), normal((1, F, H), H ** -0.5), normal((1, H, F), F ** -0.5)
    idx = torch.zeros((T, 1), dtype=torch.int32, device=DEV)
    w = torch.ones((T, 1), dtype=torch.float32, device=DEV)
    shape = moe.make_shape(H, F, 1, 1, torch.bfloat16)
    ws = moe.alloc_workspace(shape, T)
    y = torch.empty_like(x)
    stale = (torch.arange(T, device=DEV) % 2).to(torch.uint8).reshape(T, 1)
    tok = torch.tensor([0, 1, T - 3, T - 2, T - 1], device=DEV)
    mixed = torch.where(stale[tok] != 0, x_stale[tok], x[tok])
    for precalc, rows in ((False, x[tok]), (True, mixed)):
        y.fill_(float("nan"))
        if precalc:
            moe.moe_expert_ffn_precalc(shape, x, x_stale, stale, idx, w, w1, w3, w2, y, ws)
        else:
            moe.moe_expert_ffn(shape, x, idx, w, w1, w3, w2, y, ws)
        ref = _swiglu_expert_rows(rows, w1[0], w3[0], w2[0])
        torch.cuda.synchronize()
        got = y[tok].float()
        err = ((got - ref).abs() / ref.abs().clamp_min(ref.square().mean().sqrt())).max().item()
        assert err <= 2e-2, (precalc, err)
        assert torch.isfinite(y[:, ::1 << 12]).all()


@pytest.mark.parametrize("T,H,F,E,k", [
    (1, 256, 512, 8, 2), (5, 256, 512, 8, 2), (16, 256, 512, 8, 2), (8, 512, 1600, 16, 2), (3, 64, 64, 4, 1),
    (16, 128, 320, 8, 8), (7, 2048, 1024, 8, 2), (4, 128, 128, 64, 8), (9, 192, 256, 32, 2), (6, 8192, 128, 8, 2),
    (5, 128, 128, 6, 2),
])
def test_bf16_decode_path(oracle, T, H, F, E, k):
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"decode T={T}")
    print(r)


def _random_shapes(n, seed):
    """Seeded sweep over legal shapes: token counts on both sides of every path boundary (16, 32,
    256), widths that do not divide the tile sizes, few and many experts, every top_k."""
    rng = np.random.default_rng(seed)
    shapes = []
    for i in range(n):
        T = int(rng.choice([1, 2, 3, 7, 15, 16, 17, 24, 31, 32, 33, 48, 63, 64, 80, 127, 200, 255, 256, 257, 300]))
        H = 64 * int(rng.integers(1, 9))
        F = 64 * int(rng.integers(1, 25))
        E = int(rng.choice([1, 2, 3, 4, 5, 8, 11, 16, 24, 32, 64]))
        k = int(rng.integers(1, min(E, 8) + 1))
        shapes.append((T, H, F, E, k, i))
    return shapes


@pytest.mark.parametrize("T,H,F,E,k,seed", _random_shapes(36, 20250110))
def test_bf16_random_shapes(oracle, T, H, F, E, k, seed):
    d, shape, out, res = _run(T, H, F, E, k, torch.bfloat16, seed=seed, zipf=1.2 if seed % 3 else None)
    r = check_layer(oracle, d, shape, res, torch.bfloat16, label=f"bf16 random T={T} H={H} F={F} E={E} k={k}")
    print(r)


@pytest.mark.parametrize("T,H,F,E,k", [(100, 128, 192, 8, 2), (5, 64, 128, 4, 2), (130, 256, 64, 16, 3)])
def test_fp32_path(oracle, T, H, F, E, k):
    d, shape, out, res = _run(T, H, F, E, k, torch.float32)
    r = check_layer(oracle, d, shape, res, torch.float32, label=f"fp32 T={T}")
    print(r)


@pytest.mark.parametrize("T,H,F,E,k,zipf", [
    (1, 64, 64, 4, 1, None),         # one slot, one K step a wavefront in both GEMMs
    (17, 128, 320, 1, 1, None),      # 17 slots of one expert: a full 16-slot group and a single row; 2 and 5 K steps
    (16, 192, 64, 8, 8, None),       # every expert has all 16 tokens
    (95, 64, 2048, 2, 2, None),      # 95 slots an expert in units of 64 or 32: ragged last units; 32 K steps
    (260, 320, 1024, 3, 2, 1.2),     # units of 64 slots in the first GEMM, of 16 in the second
    (700, 512, 2048, 4, 3, 1.2),     # units of 64 slots in both, one to four groups in the last ones
    (33, 64, 64, 64, 8, 0.5),        # 64 experts; 128 selections to rank in a block
    (40, 4096, 64, 33, 5, 1.2),      # four blocks of experts in the router, more than one chunk of its K steps
    (37, 1088, 128, 17, 2, 1.2),     # router: 68 K steps over 16 wavefronts, two blocks of experts, the second with one
])
def test_fp32_units_groups_and_router_blocks(oracle, T, H, F, E, k, zipf):
    d, shape, out, res = _run(T, H, F, E, k, torch.float32, zipf=zipf)
    r = check_layer(oracle, d, shape, res, torch.float32, label=f"fp32 units T={T}")
    # fp32 sums of n terms are off by less than n * 2^-24 of their terms' size; a tenth of the general tolerance covers H + F
    assert r["err"] <= 1e-5, r


@pytest.mark.parametrize("T,H,F,E,zipf", [
    (600, 3072, 3072, 8, 1.2),   # 48 K steps: the fewest with which work is taken over
    (150, 4096, 6400, 16, 1.5),  # 64 and 100 K steps, single slot tiles
    (1500, 4096, 3584, 6, 0.5),  # several rounds in both GEMMs
])
def test_bf16_work_taken_over_between_xcds_repeats_bit_for_bit(T, H, F, E, zipf):
    """Which workgroup makes a tile depends on timing there; the plan, and with it every sum, depends on the counts alone."""
    d, shape, out, res = _run(T, H, F, E, 2, torch.bfloat16, zipf=zipf, predict=False)
    torch.cuda.synchronize()
    first = res["y"].clone()
    for i in range(8):
        out.workspace.fill_(255 if i % 2 else 0)
        out.y.fill_(0)
        res = moe.run_layer(shape, d, out, predict=False)
        torch.cuda.synchronize()
        assert torch.equal(res["y"], first), i


@pytest.mark.parametrize("T,H,F,E,k", [
    (800, 1024, 1024, 4, 2),    # both GEMMs: one wavefront sums K alone, 64 slots x 128 features
    (700, 576, 1600, 3, 3),     # the shortest long K; features that are no multiple of 128
    (900, 640, 512, 2, 1),      # only the first GEMM has a long K
    (2000, 64, 192, 8, 2),      # K 64 and 192: short K, 32 slots
    (3000, 128, 64, 5, 4),      # features of the second GEMM that are no multiple of 128; K 128 and 64
    (300, 192, 2112, 1, 1),     # short and long K, one expert, ragged last units
])
def test_fp32_kernels_for_long_calls_give_the_same_bits(oracle, T, H, F, E, k):
    """A slot's sums have one order in all fp32 GEMM kernels: a long call equals the calls on its slices bit for bit, with
    selections evaluated on another input among them.  A few tokens are compared with the oracle as well."""
    d = synth.moe_layer_inputs(T, H, F, E, torch.float32, DEV, seed=T, with_next=False)
    shape = moe.make_shape(H, F, E, k, torch.float32)
    g = torch.Generator().manual_seed(T)
    idx = torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).int().to(DEV)
    w = torch.softmax(torch.rand((T, k), generator=g), 1).to(DEV)
    x_stale = synth.normal((T, H), 5, 3, 1.0, torch.float32, DEV)
    stale = (torch.rand((T, k), generator=g) < 0.4).to(torch.uint8).to(DEV)
    ws = moe.alloc_workspace(shape, T)

    def run(lo, hi):
        y = torch.empty((2, hi - lo, H), device=DEV)
        part = [t[lo:hi].clone() for t in (d["x"], x_stale, stale, idx, w)]
        moe.moe_expert_ffn(shape, part[0], part[3], part[4], d["w1"], d["w3"], d["w2"], y[0], ws)
        moe.moe_expert_ffn_precalc(shape, *part, d["w1"], d["w3"], d["w2"], y[1], ws)
        return y

    whole = run(0, T)
    assert torch.equal(whole, torch.cat([run(lo, min(T, lo + 37)) for lo in range(0, T, 37)], 1))
    tok = np.unique(np.linspace(0, T - 1, 12).astype(int))
    h = host(d)
    ref = oracle.expert_ffn(h["x"], idx.cpu().numpy(), w.cpu().numpy().astype(np.float64), h["w1"], h["w3"], h["w2"], tokens=tok)
    # fp32 sums of n terms are off by less than n * 2^-24 of their terms' size
    assert output_error(to_f64(whole[0])[tok], ref) <= 1e-5


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("E", [7, 21, 61])
@pytest.mark.parametrize("H", [64, 448, 1024, 1536, 2304, 2624, 3008, 3584, 4160])
def test_router_steps_per_wavefront(oracle, H, E, dtype):
    """Sixteen wavefronts share the K steps: 0 to 10 (bf16) or 17 (fp32) steps each, in chunks of 1, 4 or 8 with every remainder."""
    T, k = 35, 3
    d = synth.moe_layer_inputs(T, H, 64, E, dtype, DEV, seed=H + E)
    shape = moe.make_shape(H, 64, E, k, dtype)
    idx = torch.empty((T, k), dtype=torch.int32, device=DEV)
    w = torch.empty((T, k), dtype=torch.float32, device=DEV)
    counts = torch.empty(E, dtype=torch.int32, device=DEV)
    moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, moe.alloc_workspace(shape, T, route_only=True))
    torch.cuda.synchronize()
    h = host(d)
    check_routing(idx, w, counts, oracle.route(h["x"], h["wg"], h["bias"], k), E, f"H={H} E={E}")


@pytest.mark.parametrize("T,F,E,zipf", [
    (1100, 1024, 12, 1.5),     # second GEMM: one full round and whole leftover tiles from the middle of the list; no work taken over
    (1100, 3072, 12, 1.5),     # one full round with few hot tiles: the coldest are left over and cut; 48 K steps: work is taken over
    (2600, 3072, 4, 1.2),      # one full round of hot tiles alone, leftover tiles cut
    (5000, 3072, 3, 0.5),      # two full rounds: the leftover tiles are the last ones
])
def test_bf16_leftover_tiles_of_the_second_gemm(oracle, T, F, E, zipf):
    H, k, dtype = 4096, 2, torch.bfloat16
    d, shape, out, res = _run(T, H, F, E, k, dtype, zipf=zipf, predict=False)
    torch.cuda.synchronize()
    plan = second_gemm_plan(out.workspace, shape, T)
    counts = res["counts"].cpu().numpy()
    tiles = second_gemm_tiles(counts, H, plan["slots"])
    print(plan, "tiles", len(tiles), "hot", sum(counts[e] > plan["slots"] for e, _ in tiles), counts)
    assert plan["count"] == len(tiles) % 256 and 0 <= plan["first"] <= len(tiles) - plan["count"]
    sample = tile_aware_sample(res["idx"].cpu().numpy(), E, 16, plan, H, n_cold=0)
    # every token against a second call with its rows in another order: other tiles, other pieces, sums equal to the
    # last bits of fp32, so a bf16 result may round to its neighbour
    check_layer(oracle, d, shape, res, dtype, tokens=sample, label=f"leftover T={T} F={F} E={E}", predict=False)
    perm = torch.randperm(T, generator=torch.Generator().manual_seed(1)).to(DEV)
    d2 = dict(d, x=d["x"][perm].contiguous())
    out2 = moe.LayerOutputs(shape, T, dtype, DEV, predict=False)
    res2 = moe.run_layer(shape, d2, out2, predict=False)
    torch.cuda.synchronize()
    assert torch.equal(res2["idx"], res["idx"][perm])
    a, b = res["y"][perm].float(), res2["y"].float()
    assert torch.all((a - b).abs() <= 2.0 ** -7 * a.abs().clamp_min(a.square().mean().sqrt()))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T", [9, 30, 64, 150])
def test_layer_equals_route_predict_ffn_bitwise(dtype, T):
    H, F, E, k = 256, 512, 8, 2
    d, shape, out, res = _run(T, H, F, E, k, dtype)
    idx = torch.empty((T, k), dtype=torch.int32, device=DEV)
    w = torch.empty((T, k), dtype=torch.float32, device=DEV)
    counts = torch.full((E,), -7, dtype=torch.int32, device=DEV)
    pidx = torch.empty((T, k), dtype=torch.int32, device=DEV)
    pw = torch.empty((T, k), dtype=torch.float32, device=DEV)
    pcounts = torch.full((E,), -7, dtype=torch.int32, device=DEV)
    y = torch.empty((T, H), dtype=dtype, device=DEV)
    ws = moe.alloc_workspace(shape, T)
    moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, ws)
    moe.moe_predict_next(shape, d["x"], d["wg_next"], d["bias_next"], pidx, pw, pcounts, ws)
    moe.moe_expert_ffn(shape, d["x"], idx, w, d["w1"], d["w3"], d["w2"], y, ws)
    torch.cuda.synchronize()
    assert torch.equal(idx, res["idx"]) and torch.equal(w, res["w"]) and torch.equal(counts, res["counts"])
    assert torch.equal(pidx, res["pred_idx"])
    assert torch.equal(y.view(torch.uint8), res["y"].view(torch.uint8))
    assert pcounts.sum().item() == T * k
    assert torch.equal(pcounts, torch.bincount(pidx.flatten().long(), minlength=E).int())
    assert torch.all((pw.sum(1) - 1).abs() < 1e-5)


@pytest.mark.parametrize("T", [8, 48, 260])
def test_repeatable_and_independent_of_workspace_contents(T):
    H, F, E, k, dtype = 256, 512, 8, 2, torch.bfloat16
    d, shape, out, res = _run(T, H, F, E, k, dtype)
    y0, i0, c0 = res["y"].clone(), res["idx"].clone(), res["counts"].clone()
    for fill in (0xFF, 0x7F, 0x00):
        out.workspace.fill_(fill)   # 0xFF.. is NaN in bf16 and fp32 and -1 as an index
        out.y.fill_(0)
        res = moe.run_layer(shape, d, out)
        torch.cuda.synchronize()
        assert torch.equal(res["y"].view(torch.int16), y0.view(torch.int16))
        assert torch.equal(res["idx"], i0) and torch.equal(res["counts"], c0)


@pytest.mark.parametrize("T,H,F,E,k", [(1, 256, 512, 8, 2), (6, 256, 512, 8, 2), (16, 128, 320, 8, 8), (3, 64, 64, 4, 1),
                                       (24, 256, 512, 8, 2), (300, 256, 512, 8, 2), (600, 1024, 2048, 8, 2)])
def test_sequence_of_calls_on_one_workspace_small_shapes(T, H, F, E, k):
    """Calls with changing inputs share one workspace at sizes where everything stays in the caches
    between launches: what an earlier call left there (intermediate values, K-split pieces,
    rendezvous flags and counters) must never be what a later call reads.  Every call is compared
    bit for bit with the same call on a fresh workspace filled with a byte pattern."""
    dtype = torch.bfloat16
    d = synth.moe_layer_inputs(T, H, F, E, dtype, DEV, seed=3, zipf_s=1.2, with_next=True)
    shape = moe.make_shape(H, F, E, k, dtype)
    shared = moe.LayerOutputs(shape, T, dtype, DEV, predict=True)
    for step in range(8):
        call = dict(d, x=synth.normal((T, H), 3000 + step, synth.TID_X, 1.0, dtype, DEV))
        got = moe.run_layer(shape, call, shared, predict=True)
        y, idx, pred = got["y"].clone(), got["idx"].clone(), got["pred_idx"].clone()
        fresh = moe.LayerOutputs(shape, T, dtype, DEV, predict=True)
        fresh.workspace.fill_(0x5A)
        ref = moe.run_layer(shape, call, fresh, predict=True)
        torch.cuda.synchronize()
        assert torch.equal(idx, ref["idx"]) and torch.equal(pred, ref["pred_idx"]), f"step {step}"
        assert torch.equal(y.view(torch.int16), ref["y"].view(torch.int16)), f"step {step}"


def test_alternating_long_and_decode_calls_on_one_workspace():
    """A serving loop alternates prefill-size and single-token calls on one workspace.  The decode
    kernel derives its rendezvous epoch from a launch count it keeps in the workspace, and flags left
    by its previous launch carry the previous epoch; a long call in between must leave both alone
    (they sit at fixed offsets ahead of everything whose size depends on the call).  Every call is
    compared bit for bit with the same call on a fresh workspace filled with a byte pattern."""
    H, F, E, k, dtype = 256, 512, 8, 2, torch.bfloat16
    d = synth.moe_layer_inputs(1024, H, F, E, dtype, DEV, seed=11, zipf_s=1.2, with_next=True)
    shape = moe.make_shape(H, F, E, k, dtype)
    shared = moe.LayerOutputs(shape, 1024, dtype, DEV, predict=True)
    shared.workspace.zero_()
    for step, T in enumerate([1, 1024, 1, 1, 1024, 300, 1, 24, 1, 1024, 1]):
        call = dict(d, x=synth.normal((T, H), 4000 + step, synth.TID_X, 1.0, dtype, DEV))
        got = moe.run_layer(shape, call, shared, predict=True)
        y, idx = got["y"].clone(), got["idx"].clone()
        fresh = moe.LayerOutputs(shape, T, dtype, DEV, predict=True)
        fresh.workspace.fill_(0x5A)
        ref = moe.run_layer(shape, call, fresh, predict=True)
        torch.cuda.synchronize()
        assert torch.equal(idx, ref["idx"]), f"step {step} T={T}"
        assert torch.equal(y.view(torch.int16), ref["y"].view(torch.int16)), f"step {step} T={T}"
    assert not moe.moe_decode_status(shared.workspace)


def test_decode_rendezvous_reports_when_it_gives_up(oracle):
    """The decode-size kernel's workgroups wait for one another with a bounded spin.  Normally nobody
    gives up and the status word stays clear.  With the spin bound lowered to zero from the host every
    rendezvous gives up at once (all kernels still run to their end): the call then reports it through
    moe_decode_status and marks its output with NaN instead of returning numbers computed from an
    intermediate that may not have been written yet."""
    T, H, F, E, k, dtype = 4, 256, 512, 8, 2, torch.bfloat16
    d, shape, out, res = _run(T, H, F, E, k, dtype)
    torch.cuda.synchronize()
    good = res["y"].clone()
    assert not moe.moe_decode_status(out.workspace, reset=True)
    try:
        moe.moe_measure_set_decode_spin_limit(0)
        res = moe.run_layer(shape, d, out)
        torch.cuda.synchronize()
        assert torch.isnan(res["y"].float()).all()
        assert moe.moe_decode_status(out.workspace)            # reported ...
        assert moe.moe_decode_status(out.workspace, reset=True)  # ... and sticky until reset
        assert not moe.moe_decode_status(out.workspace)
    finally:
        moe.moe_measure_set_decode_spin_limit(1 << 22)
    res = moe.run_layer(shape, d, out)
    torch.cuda.synchronize()
    assert torch.equal(res["y"].view(torch.int16), good.view(torch.int16))
    assert not moe.moe_decode_status(out.workspace)
    r = check_layer(oracle, d, shape, res, dtype, label="after a reported give-up")
    print(r)


@pytest.mark.parametrize("T,H,F,E,k,dtype", [
    (1, 256, 512, 8, 2, torch.bfloat16), (8, 512, 1024, 8, 2, torch.bfloat16), (16, 128, 320, 8, 8, torch.bfloat16),
    (24, 256, 512, 8, 2, torch.bfloat16),      # two column groups of the streaming kernel
    (6, 8192, 128, 8, 2, torch.bfloat16),      # hidden size past the register-resident token operand
    (300, 256, 512, 8, 2, torch.bfloat16),     # ragged slot tiles
    (1100, 256, 512, 2, 2, torch.bfloat16),    # full 256-slot tiles, split-K round
    (64, 256, 512, 8, 2, torch.float32), (5, 64, 128, 4, 2, torch.float32),
])
def test_expert_ffn_with_precalculated_selections(oracle, T, H, F, E, k, dtype):
    """Sec. IV-C pre-calculation as one library call: selections flagged stale are evaluated on an
    earlier hidden state, the rest on the true input, in one pass over the weights.  Compared with the
    oracle's definition at the layer's own tolerance; an all-zero mask must equal moe_expert_ffn."""
    d = synth.moe_layer_inputs(T, H, F, E, dtype, DEV, seed=31, zipf_s=1.2, with_next=False)
    x_stale = synth.normal((T, H), 4242, synth.TID_X, 1.0, dtype, DEV)
    shape = moe.make_shape(H, F, E, k, dtype)
    ws = moe.alloc_workspace(shape, T)
    idx = torch.empty((T, k), dtype=torch.int32, device=DEV)
    w = torch.empty((T, k), dtype=torch.float32, device=DEV)
    counts = torch.zeros((E,), dtype=torch.int32, device=DEV)
    moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, ws)
    g = torch.Generator(device="cpu").manual_seed(T * 7 + H)
    stale = (torch.rand((T, k), generator=g) < 0.4).to(torch.uint8)
    stale[0, 0] = 1
    if k > 1:
        stale[0, 1] = 0
    stale = stale.to(DEV)
    y = torch.empty((T, H), dtype=dtype, device=DEV)
    moe.moe_expert_ffn_precalc(shape, d["x"], x_stale, stale, idx, w, d["w1"], d["w3"], d["w2"], y, ws)
    torch.cuda.synchronize()
    h = host(dict(d, x_stale=x_stale))
    ref = oracle.expert_ffn_precalc(h["x"], h["x_stale"], stale.cpu().numpy(), idx.cpu().numpy(),
                                    w.cpu().numpy().astype(np.float64), h["w1"], h["w3"], h["w2"])
    err = output_error(to_f64(y), ref)
    print("precalc", T, H, F, E, k, dtype, "err", err)
    assert err <= {torch.bfloat16: 2e-2, torch.float32: 1e-4}[dtype]
    # the mask matters: the plain call differs where a selection is stale
    y_plain = torch.empty_like(y)
    moe.moe_expert_ffn(shape, d["x"], idx, w, d["w1"], d["w3"], d["w2"], y_plain, ws)
    y_zero = torch.empty_like(y)
    moe.moe_expert_ffn_precalc(shape, d["x"], x_stale, torch.zeros_like(stale), idx, w, d["w1"], d["w3"], d["w2"], y_zero, ws)
    torch.cuda.synchronize()
    assert torch.equal(y_zero.view(torch.uint8), y_plain.view(torch.uint8))
    assert not torch.equal(y[0], y_plain[0])


def test_prepared_call_equals_run_layer():
    """The binding's pre-marshalled call object enqueues the same call as run_layer."""
    T, H, F, E, k, dtype = 6, 256, 512, 8, 2, torch.bfloat16
    d, shape, out, res = _run(T, H, F, E, k, dtype)
    y, idx, pred, counts = res["y"].clone(), res["idx"].clone(), res["pred_idx"].clone(), res["counts"].clone()
    out2 = moe.LayerOutputs(shape, T, dtype, DEV, predict=True)
    call = moe.PreparedLayerCall(shape, d, out2, predict=True)
    for _ in range(3):
        got = call()
    torch.cuda.synchronize()
    assert torch.equal(got["idx"], idx) and torch.equal(got["pred_idx"], pred) and torch.equal(got["counts"], counts)
    assert torch.equal(got["y"].view(torch.int16), y.view(torch.int16))


def test_counts_accumulate_over_calls_and_zero_tokens(oracle):
    H, F, E, k, dtype = 256, 512, 8, 2, torch.bfloat16
    d, shape, out, res = _run(40, H, F, E, k, dtype)
    c1 = res["counts"].clone()
    moe.run_layer(shape, d, out, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(out.counts, 2 * c1)
    # decode-size call adds its own tokens
    d1 = dict(d)
    d1["x"] = d["x"][:3].contiguous()
    moe.run_layer(shape, d1, out, accumulate=True)
    torch.cuda.synchronize()
    assert out.counts.sum().item() == (40 * 2 + 3) * k
    # 17 to 32 tokens: the weight-streaming kernel counts the selections of the routing kernel before it
    d2 = dict(d)
    d2["x"] = d["x"][:20].contiguous()
    before = out.counts.clone()
    r2 = moe.run_layer(shape, d2, out, accumulate=True)
    torch.cuda.synchronize()
    hist = torch.bincount(r2["idx"].flatten().long(), minlength=E).to(torch.int32)
    assert torch.equal(out.counts, before + hist)
    moe.run_layer(shape, d2, out, accumulate=False)
    torch.cuda.synchronize()
    assert torch.equal(out.counts, hist)
    moe.run_layer(shape, d, out, accumulate=False)
    moe.run_layer(shape, d, out, accumulate=True)
    moe.run_layer(shape, d1, out, accumulate=True)
    torch.cuda.synchronize()
    # zero tokens: counts untouched with accumulate, cleared without
    d0 = dict(d)
    d0["x"] = d["x"][:0]
    before = out.counts.clone()
    moe.run_layer(shape, d0, out, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(out.counts, before)
    moe.run_layer(shape, d0, out, accumulate=False)
    torch.cuda.synchronize()
    assert out.counts.sum().item() == 0
    ws = moe.alloc_workspace(shape, 1, route_only=True)
    cnt = torch.full((E,), 5, dtype=torch.int32, device=DEV)
    moe.moe_route(shape, d0["x"], d["wg"], None, out.topk_idx[:0], out.topk_w[:0], cnt, False, ws)
    torch.cuda.synchronize()
    assert cnt.sum().item() == 0


def test_all_tokens_to_one_expert_equals_its_dense_ffn(oracle):
    # the degenerate grouping: one expert owns every slot (k = 1, +50 bias), both paths
    H, F, E, dtype = 256, 512, 8, torch.bfloat16
    for T in (12, 16, 17, 32, 33, 64, 65, 300):
        d = synth.moe_layer_inputs(T, H, F, E, dtype, DEV, zipf_s=None, with_next=False)
        d["bias"] = torch.zeros(E, dtype=torch.float32, device=DEV)
        d["bias"][5] = 50.0
        shape = moe.make_shape(H, F, E, 1, dtype)
        out = moe.LayerOutputs(shape, T, dtype, DEV, predict=False)
        res = moe.run_layer(shape, d, out, predict=False)
        torch.cuda.synchronize()
        assert torch.all(res["idx"] == 5) and res["counts"][5].item() == T
        assert torch.all(res["w"] == 1.0)
        x64 = to_f64(d["x"])
        w1, w3, w2 = to_f64(d["w1"][5]), to_f64(d["w3"][5]), to_f64(d["w2"][5])
        g = x64 @ w1.T
        dense = ((g / (1 + np.exp(-g))) * (x64 @ w3.T)) @ w2.T
        assert output_error(to_f64(res["y"]), dense) <= 2e-2


def test_routing_entry_points_alone(oracle):
    T, H, E, k = 1000, 512, 16, 2
    for dtype in (torch.float32, torch.bfloat16):
        d = synth.moe_layer_inputs(T, H, 64, E, dtype, DEV, zipf_s=1.5)
        shape = moe.make_shape(H, 64, E, k, dtype)
        ws = moe.alloc_workspace(shape, T, route_only=True)
        idx = torch.empty((T, k), dtype=torch.int32, device=DEV)
        w = torch.empty((T, k), dtype=torch.float32, device=DEV)
        counts = torch.zeros((E,), dtype=torch.int32, device=DEV)
        moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, ws)
        torch.cuda.synchronize()
        h = host(d)
        ref = oracle.route(h["x"], h["wg"], h["bias"], k)
        n_excl, _ = check_routing(idx, w, counts, ref, E, "moe_route")
        assert n_excl < 0.02 * T
        # same gate as "next" gate: the prediction equals the routing
        pidx = torch.empty((T, k), dtype=torch.int32, device=DEV)
        moe.moe_predict_next(shape, d["x"], d["wg"], d["bias"], pidx, None, None, ws)
        torch.cuda.synchronize()
        assert torch.equal(pidx, idx)


def test_mfma_calibration_probe_is_sane():
    """The register-only MFMA loop: plausible rates, and constant operands never slower than random ones."""
    const = moe.moe_calibrate_mfma(False, 4096)
    rnd = moe.moe_calibrate_mfma(True, 4096)
    assert const["flop"] == rnd["flop"] > 0
    assert 500 < rnd["tflops"] <= const["tflops"] * 1.05 and const["tflops"] < 2600
    assert 0.5 < rnd["ghz"] <= const["ghz"] * 1.05 and const["ghz"] < 2.6


def test_read_stream_probe_is_sane():
    """The plain read stream: a plausible rate, and the bytes it reports are what it was given (rounded down)."""
    buf = torch.empty(1 << 29, dtype=torch.uint8, device=DEV).fill_(1)     # 512 MB
    r = moe.moe_calibrate_read_stream(buf)
    assert 0.9 * buf.numel() <= r["bytes"] <= buf.numel()
    assert 1000 < r["GBps"] < 8000
