"""Routing at the edges of its kernels: blocks of 16 tokens and 16 experts, units of 128 bytes dealt to the wavefronts, the decode-size
routine on the vector lanes (up to two tokens) and on the matrix cores, and predictions made in the same call."""
import pytest
import torch

from paper_2501_10375_amd import moe, synth
from parity_util import check_layer, check_routing, host

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _route(oracle, T, H, E, k, dtype):
    d = synth.moe_layer_inputs(T, H, 64, E, dtype, DEV, seed=T + H + E, zipf_s=0.7, with_next=True)
    shape = moe.make_shape(H, 64, E, k, dtype)
    idx = torch.full((T, k), -1, dtype=torch.int32, device=DEV)
    w = torch.full((T, k), -1.0, device=DEV)
    counts = torch.full((E,), 7, dtype=torch.int32, device=DEV)
    pidx, pw, pcounts = torch.full_like(idx, -1), torch.full_like(w, -1.0), torch.full_like(counts, 7)
    ws = moe.alloc_workspace(shape, T, route_only=True)
    h = host(d)
    for fill in (0, 0xFF):
        ws.fill_(fill)
        for _ in range(2):
            moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, ws)
            moe.moe_predict_next(shape, d["x"], d["wg_next"], d["bias_next"], pidx, pw, pcounts, ws)
        torch.cuda.synchronize()
        check_routing(idx, w, counts, oracle.route(h["x"], h["wg"], h["bias"], k), E, f"T={T} H={H} E={E}")
        check_routing(pidx, pw, pcounts, oracle.predict_next(h["x"], h["wg_next"], h["bias_next"], k), E, f"T={T} H={H} E={E} next")
    before = counts.clone()
    moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, True, ws)
    assert torch.equal(counts, 2 * before)
    # the whole layer makes the same choices, bit for bit
    out = moe.LayerOutputs(shape, T, dtype, DEV, predict=True)
    res = moe.run_layer(shape, d, out)
    torch.cuda.synchronize()
    assert torch.equal(res["idx"], idx) and torch.equal(res["w"], w) and torch.equal(res["counts"], before)
    assert torch.equal(res["pred_idx"], pidx)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,H,E,k", [
    (17, 64, 16, 2),       # one or two units for 16 wavefronts
    (33, 192, 17, 2),      # one expert in the second block
    (40, 1088, 33, 3),     # units that do not divide the wavefronts; one expert in the third block
    (50, 4096, 48, 8),     # three of four blocks
    (33, 64, 33, 2),       # one or two units, each shared by four wavefronts
    (50, 128, 64, 8),      # two (shared by four) or four (by two)
    (17, 192, 48, 3),      # three shared by two, or six
    (40, 256, 64, 6),      # four shared by two, or eight
    (24, 320, 40, 4),      # five and ten: not shared
    (31, 8256, 8, 1),      # several chunks a wavefront and a rest
    (70, 2112, 64, 8),
    (100, 4160, 32, 4),
    (530, 128, 5, 2),      # more than 512 selections
    (512, 64, 16, 2),      # 1024 selections: the last workgroup permutes them
    (513, 64, 16, 2),      # one more than it takes
    (1040, 64, 3, 2),      # 65 blocks
    (768, 64, 64, 1),      # 3072 counts: the most that the last workgroup adds
    (4096, 64, 6, 1),      # 256 blocks: the most whose counts it adds
    (2100, 64, 64, 1),     # more counts than one workgroup adds
])
def test_prefill_sizes(oracle, T, H, E, k, dtype):
    _route(oracle, T, H, E, k, dtype)


@pytest.mark.parametrize("T", [1, 2, 3, 9, 16])
@pytest.mark.parametrize("H,E,k", [
    (64, 16, 2),           # one piece for eight wavefronts
    (320, 17, 2),
    (2112, 33, 8),         # half a chunk and a rest
    (4096, 8, 2),
    (4160, 64, 6),         # a chunk and a rest
    (8192, 24, 1),
])
def test_decode_sizes(oracle, T, H, E, k):
    _route(oracle, T, H, E, k, torch.bfloat16)


def test_values_that_are_not_finite_stay_where_they_are():
    """An infinite gate weight, or a token with one, concerns that expert or token only, also where loads are padded."""
    T, H, E, k = 9, 320, 12, 2
    d = synth.moe_layer_inputs(T, H, 64, E, torch.bfloat16, DEV, seed=3, zipf_s=0.0, with_next=False)
    d["x"][4, 0] = float("inf")
    shape = moe.make_shape(H, 64, E, k, torch.bfloat16)
    idx, w = torch.empty((T, k), dtype=torch.int32, device=DEV), torch.empty((T, k), device=DEV)
    counts, ws = torch.empty(E, dtype=torch.int32, device=DEV), moe.alloc_workspace(shape, 40, route_only=True)
    moe.moe_route(shape, d["x"], d["wg"], None, idx, w, counts, False, ws)
    p = (d["x"].double() @ d["wg"].double().T).softmax(-1)
    torch.cuda.synchronize()
    for t in (0, 3, 5, 8):
        ref = p[t].gather(0, idx[t].long())
        assert torch.allclose(w[t].double(), ref / ref.sum(), atol=1e-5) and p[t].topk(k).indices.sort().values.tolist() == sorted(idx[t].tolist())
    d["x"][4, 0] = 1.0
    d["wg"][11, 0] = -float("inf")
    d["x"][:, 0] = d["x"][:, 0].abs() + 0.5          # that expert's logit is -inf, the others are what they are
    for n in (9, 1):
        moe.moe_route(shape, d["x"][:n].contiguous(), d["wg"], None, idx[:n], w[:n], counts, False, ws)
        p = (d["x"].double() @ d["wg"].double().T).softmax(-1)
        torch.cuda.synchronize()
        assert not (idx[:n] == 11).any() and torch.isfinite(w[:n]).all()
        ref = p[:n].gather(1, idx[:n].long())
        assert torch.allclose(w[:n].double(), ref / ref.sum(1, keepdim=True), atol=1e-5)


@pytest.mark.parametrize("T", [1, 2, 16, 24])
@pytest.mark.parametrize("H,F,E,k", [
    (2048, 320, 20, 3),    # phase 1 of a decode step with four K steps a wavefront; one token: tiles of 8 features, fewer than workgroups
    (2112, 192, 9, 2),     # eight K steps, one of them there
    (4096, 2752, 8, 2),    # one token: 8-feature tiles, more than two rounds
    (1984, 128, 8, 2),     # just below what takes 8-feature tiles
    (4160, 128, 12, 2),    # longer than the token operand that registers hold
])
def test_decode_step_tiles(oracle, T, H, F, E, k):
    d = synth.moe_layer_inputs(T, H, F, E, torch.bfloat16, DEV, seed=T + F, zipf_s=0.7, with_next=True)
    shape = moe.make_shape(H, F, E, k, torch.bfloat16)
    out = moe.LayerOutputs(shape, T, torch.bfloat16, DEV, predict=True)
    check_layer(oracle, d, shape, moe.run_layer(shape, d, out), torch.bfloat16, label=f"decode T={T} H={H} F={F}")


@pytest.mark.parametrize("T,E,launches", [(17, 8, 1), (4096, 8, 1), (4097, 8, 2), (768, 64, 1), (769, 64, 2), (16384, 8, 2)])
def test_counts_of_long_calls_are_another_kernels(T, E, launches):
    """Where every workgroup would read very many counts, that takes longer than a launch."""
    d = synth.moe_layer_inputs(T, 64, 64, E, torch.bfloat16, DEV, seed=T, zipf_s=0.7, with_next=False)
    shape = moe.make_shape(64, 64, E, 1, torch.bfloat16)
    idx, w = torch.empty((T, 1), dtype=torch.int32, device=DEV), torch.empty((T, 1), device=DEV)
    counts, ws = torch.empty(E, dtype=torch.int32, device=DEV), moe.alloc_workspace(shape, T, route_only=True)
    moe.moe_stage_timing_begin(1)
    moe.moe_route(shape, d["x"], d["wg"], d["bias"], idx, w, counts, False, ws)
    stages = moe.moe_stage_timing_end()
    assert stages["route"][1] + stages["permute"][1] == launches
    assert torch.equal(counts, torch.bincount(idx.flatten(), minlength=E).int())
