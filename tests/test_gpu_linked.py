"""bf16 calls of middle size run both grouped GEMMs in one launch, whose workgroups go on with the second one's tiles as soon as the
tiles of the first that these need are stored.  Every token of narrow layers that take this route is compared with the oracle."""
import numpy as np
import pytest
import torch

from paper_2501_10375_amd import moe, synth
from parity_util import check_layer, host, output_error, to_f64

pytestmark = pytest.mark.gpu
DEV, DTYPE = "cuda", torch.bfloat16


def _layer(T, H, F, E, k, zipf=1.2, linked=True):
    # the route (256 compute units), whatever the routing: two and a half rounds of the first GEMM's tiles and three quarters of the second's,
    # or five quarters of both with 48 rows an expert; 300 rows an expert at most
    slot_tiles = T * k // 256 + min(E, T * k)
    first, second = -(-F // 128) * slot_tiles, -(-H // 256) * slot_tiles
    route = (first > 640 and second >= 192 and T * k * H >= 4e5) or (first > 320 and second >= 300 and T * k >= 48 * E)
    assert linked == (route and T * k <= 300 * E and T * k * H * F <= 1.6e11 and T > 32), (first, second)
    d = synth.moe_layer_inputs(T, H, F, E, DTYPE, DEV, seed=T + H, zipf_s=zipf, with_next=True)
    shape = moe.make_shape(H, F, E, k, DTYPE)
    out = moe.LayerOutputs(shape, T, DTYPE, DEV, predict=True)
    return d, shape, out


def _stages(shape, d, out):
    moe.moe_stage_timing_begin(1)
    res = moe.run_layer(shape, d, out)
    stages = moe.moe_stage_timing_end()
    return res, stages


@pytest.mark.parametrize("T,H,F,E,k", [
    (1024, 320, 896, 64, 8),   # five K steps in the first GEMM: the fewest; a quarter of a feature tile at the end of the second
    (2400, 768, 320, 64, 8),   # five K steps in the second GEMM: the fewest; 300 rows an expert: the most
    (88, 576, 1344, 64, 8),    # nine K steps; half a feature tile at the end; experts with a handful of rows
    (100, 1088, 1728, 48, 4),
    (600, 2048, 1024, 32, 4),  # little more than a round of both
    (512, 2560, 4160, 16, 2),  # tall and low tiles, 65 K steps in the second GEMM; work is taken over between XCDs
    (1500, 1536, 2560, 16, 3), # full tiles of several slot groups
    (900, 576, 1600, 64, 1),   # skewed routing over many experts, some without rows
])
def test_every_token(oracle, T, H, F, E, k):
    _every_token(oracle, T, H, F, E, k, True)


@pytest.mark.parametrize("T,H,F,E,k", [
    (40, 64, 1024, 64, 8),     # first GEMM of one K step: nothing to overlap in a tile
    (40, 128, 1088, 64, 8),    # two K steps; half a feature tile at the end
    (40, 192, 1024, 64, 8),    # three
    (45, 256, 1024, 64, 8),    # four; experts with a handful of rows
    (300, 320, 4160, 8, 2),    # second GEMM: a quarter of a feature tile at the end, 65 K steps
    (600, 512, 8192, 4, 2),    # tall and low tiles; work is taken over between XCDs
    (1500, 256, 2944, 3, 2),   # full tiles of several slot groups
    (900, 192, 1600, 64, 1),   # skewed routing over many experts, some without rows
])
def test_every_token_of_two_launches(oracle, T, H, F, E, k):
    """Two rounds of the first GEMM with too little of the second for one launch."""
    _every_token(oracle, T, H, F, E, k, False)


def _every_token(oracle, T, H, F, E, k, linked):
    d, shape, out = _layer(T, H, F, E, k, zipf=3.0 if k == 1 else 1.2, linked=linked)
    res, stages = _stages(shape, d, out)
    assert stages["fused"][1] == linked and stages["gemm1"][1] == stages["gemm2"][1] == (not linked), stages
    r = check_layer(oracle, d, shape, res, DTYPE, label=f"linked T={T}")
    print(r)
    assert r["compared_tokens"] >= T - r["excluded"] - 2
    good = res["y"].clone()
    for fill in (0xFF, 0x00):   # leftovers in the workspace
        out.workspace.fill_(fill)
        res = moe.run_layer(shape, d, out)
        torch.cuda.synchronize()
        assert torch.equal(res["y"].view(torch.int16), good.view(torch.int16))
    # pre-calculated selections: none, and mixed
    x_stale = synth.normal((T, H), 99, 3, 1.0, DTYPE, DEV)
    stale = (torch.rand((T, k), generator=torch.Generator().manual_seed(T)) < 0.4).to(torch.uint8).to(DEV)
    y = torch.empty_like(d["x"])
    args = (res["idx"], res["w"], d["w1"], d["w3"], d["w2"], y, out.workspace)
    moe.moe_expert_ffn_precalc(shape, d["x"], x_stale, torch.zeros_like(stale), *args)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), good.view(torch.int16))
    moe.moe_expert_ffn_precalc(shape, d["x"], x_stale, stale, *args)
    torch.cuda.synchronize()
    h = host(d)
    ref = oracle.expert_ffn_precalc(h["x"], synth.to_numpy(x_stale), stale.cpu().numpy(), res["idx"].cpu().numpy(),
                                    res["w"].cpu().numpy().astype(np.float64), h["w1"], h["w3"], h["w2"])
    assert output_error(to_f64(y), ref) <= 2e-2


def test_reports_when_a_wait_runs_out():
    """With no polling round allowed (every kernel still runs to its end) the output is NaN and the status word is raised."""
    d, shape, out = _layer(88, 576, 1344, 64, 8)
    good = moe.run_layer(shape, d, out)["y"].clone()
    assert not moe.moe_decode_status(out.workspace, reset=True)
    try:
        moe.moe_measure_set_decode_spin_limit(0)
        res = moe.run_layer(shape, d, out)
        torch.cuda.synchronize()
        assert torch.isnan(res["y"].float()).all()
        assert moe.moe_decode_status(out.workspace, reset=True)
    finally:
        moe.moe_measure_set_decode_spin_limit(1 << 22)
    res = moe.run_layer(shape, d, out)
    torch.cuda.synchronize()
    assert torch.equal(res["y"].view(torch.int16), good.view(torch.int16))
    assert not moe.moe_decode_status(out.workspace)


@pytest.mark.parametrize("T,H,F,E,k", [(88, 576, 1344, 64, 8), (512, 2560, 4160, 16, 2)])
def test_what_is_not_right_is_nan_and_reported(T, H, F, E, k):
    """Waits that run out for some workgroups and not for others, and close to the moment when the rows are complete."""
    d, shape, out = _layer(T, H, F, E, k)
    good = moe.run_layer(shape, d, out)["y"].clone()
    assert not moe.moe_decode_status(out.workspace, reset=True)
    reported = 0
    try:
        for limit in [*range(1, 25)] * 6:
            moe.moe_measure_set_decode_spin_limit(limit)
            out.workspace.fill_(0x3F)   # rows that are read too early are finite and wrong
            y = moe.run_layer(shape, d, out)["y"]
            torch.cuda.synchronize()
            nan = torch.isnan(y.float())
            assert bool(((y.view(torch.int16) == good.view(torch.int16)) | nan).all()), limit
            raised = moe.moe_decode_status(out.workspace, reset=True)
            assert raised == bool(nan.any()), limit
            reported += raised
    finally:
        moe.moe_measure_set_decode_spin_limit(1 << 22)
    assert reported > 0


def test_replays_from_a_graph():
    d, shape, out = _layer(88, 576, 1344, 64, 8)
    x = d["x"].clone()
    call = moe.PreparedLayerCall(shape, dict(d, x=x), out)
    eager = moe.LayerOutputs(shape, 88, DTYPE, DEV, predict=True)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for step in range(4):
        xs = synth.normal((88, 576), 700 + step, synth.TID_X, 1.0, DTYPE, DEV)
        ref = moe.run_layer(shape, dict(d, x=xs), eager)["y"].clone()
        torch.cuda.synchronize()
        x.copy_(xs)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(call.result["y"].view(torch.int16), ref.view(torch.int16)), step


def test_two_streams_at_once():
    """Two calls that share the chip, each with a workspace of its own: whatever part of a grid is resident at a time, a call ends and is right."""
    d, shape, out = _layer(512, 2560, 4160, 16, 2)
    good = moe.run_layer(shape, d, out)["y"].clone()
    calls = [(torch.cuda.Stream(), moe.LayerOutputs(shape, 512, DTYPE, DEV, predict=True)) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(8):
        for stream, o in calls:
            with torch.cuda.stream(stream):
                moe.run_layer(shape, d, o)
        torch.cuda.synchronize()
        for _, o in calls:
            assert torch.equal(o.y.view(torch.int16), good.view(torch.int16))
            assert not moe.moe_decode_status(o.workspace)
