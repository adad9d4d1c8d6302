"""Where both grouped GEMMs run in one launch, workgroups of the second wait for tiles of the first.  That ends whatever part of the grid is
resident (another stream or a CU mask may hold the rest back) only if the resident workgroups alone can come to every tile of the
first GEMM.  A host model of the hand-out, on the arithmetic that the kernels use, looks at that.  Where a wait runs out all the same, the
wavefronts of a workgroup, which multiply each other's rows, have to agree about it."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2501_10375_amd", "csrc")
XCDS = 8


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("hand_out") / "model.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-pthread", "-I", CSRC, "-o", path, os.path.join(HERE, "hand_out_model.cpp")],
                   check=True)
    return ctypes.CDLL(path)


@pytest.fixture(scope="module")
def model(library):
    def run(linked, mats, members, tiles, parts, resident, seed, steal=True):
        """How often each item is computed by the resident workgroups, [XCD][item]; items that no list has are -1."""
        rounds = tiles // (XCDS * members)
        left = tiles - rounds * XCDS * members
        chunk = -(-left // XCDS)
        items = [rounds * members + max(0, min(left, (x + 1) * chunk) - x * chunk) * parts for x in range(XCDS)]
        stride = max(items) + 1
        done = np.zeros((XCDS, stride), dtype=np.int32)
        mask = (ctypes.c_ubyte * (XCDS * members))(*resident)
        run.accesses = library.hand_out_model(int(linked), mats, members, rounds * members, left, parts, mask, int(steal), ctypes.c_uint(seed),
                           done.ctypes.data_as(ctypes.c_void_p), stride)
        for x in range(XCDS):
            assert (done[x, items[x]:] == 0).all()
            done[x, items[x]:] = -1
        return done

    return run


def subsets(members, rng):
    n = XCDS * members
    yield [1] * n
    for b in (0, n - 1, rng.randrange(n)):
        yield [int(i == b) for i in range(n)]       # one workgroup
        yield [int(i != b) for i in range(n)]       # all but one
    yield [int(i < n // 2) for i in range(n)]       # the first half of the grid
    yield [int(i % XCDS == 3) for i in range(n)]    # one XCD
    yield [int(i % XCDS != 5) for i in range(n)]    # an XCD is missing
    for share in (0.25, 0.5, 0.9):
        m = [int(rng.random() < share) for _ in range(n)]
        m[rng.randrange(n)] = 1
        yield m


@pytest.mark.parametrize("members", [1, 3, 32])
@pytest.mark.parametrize("tiles", [1, 5, 8, 255, 256, 257, 321, 520, 1008, 1290])
def test_any_part_of_the_grid_computes_every_tile_that_others_wait_for(model, members, tiles):
    rng = random.Random(tiles * 100 + members)
    for mask in subsets(members, rng):
        done = model(True, 2, members, tiles, 1, mask, rng.randrange(1 << 31))
        assert ((done == 1) | (done == -1)).all()


@pytest.mark.parametrize("linked,mats", [(True, 1), (False, 1), (False, 2)])
@pytest.mark.parametrize("tiles,parts", [(5, 1), (160, 3), (256, 1), (300, 2), (1008, 1)])
@pytest.mark.parametrize("steal", [True, False])
def test_the_whole_grid_computes_every_item_once(model, linked, mats, tiles, parts, steal):
    done = model(linked, mats, 32, tiles, parts, [1] * 256, tiles, steal)
    assert ((done == 1) | (done == -1)).all()


def test_the_model_sees_items_that_nobody_holds(model):
    """Where a workgroup's first item is its own (launches in which nobody waits), half of the grid leaves the other half's."""
    done = model(False, 2, 32, 1008, 1, [int(i < 128) for i in range(256)], 1)
    assert (done == 0).sum() == 128 and (done <= 1).all()


@pytest.mark.parametrize("mats", [1, 2])
@pytest.mark.parametrize("tiles,parts,accesses", [(5, 1, 0), (128, 2, 0), (256, 1, 0), (129, 2, 1), (257, 1, 1), (512, 1, 1)])
def test_one_round_does_without_the_counters(model, mats, tiles, parts, accesses):
    model(False, mats, 32, tiles, parts, [1] * 256, 3)
    assert (model.accesses > 0) == accesses


@pytest.mark.parametrize("ready_at", [(1, 1, 1, 1), (1, 9, 1, 1), (9, 1, 1, 1), (1, 9, 9, 9), (4, 5, 4, 5), (5, 4, 5, 4), (99, 99, 99, 99)])
@pytest.mark.parametrize("limit", [0, 1, 4])
def test_the_wavefronts_of_a_workgroup_give_up_together(library, ready_at, limit):
    answers, after = (ctypes.c_int * 4)(), (ctypes.c_int * 4)()
    reports = library.await_model(63, limit, (ctypes.c_int * 4)(*ready_at), answers, after)
    assert len(set(answers)) == 1 and len(set(after)) == 1
    assert reports == (0 if answers[0] else 1)
    assert answers[0] == (ready_at[0] <= limit)
    assert after[0] == (limit if answers[0] else min(limit, 1))
