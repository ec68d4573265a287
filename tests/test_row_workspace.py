"""The batches that take the row-tile path, and its weight-gradient workspace, which holds every
launch a context can make: the critics', the actor's or both, at every batch up to the created
one. Host arithmetic of the library itself (no GPU)."""
import ctypes
import math
import os
import random

import pytest

HIDDEN = [(32, 32), (64, 64), (100, 50), (128, 128), (64,), (96, 96, 96), (256, 256), (200, 120), (256, 128),
          (400, 300), (192, 192, 192), (256, 256, 256), (320, 320), (512, 512), (512, 512, 512), (480,) * 6]


@pytest.fixture(scope="module")
def workspace():
    from paper_2312_06126_amd import spz
    if not os.path.exists(spz.LIB_PATH):
        pytest.fail("libspz.so is not built; run __graft_entry__.build()")
    f = spz.load().spzt_row_workspace
    i32, p64 = ctypes.c_int32, ctypes.POINTER(ctypes.c_int64)
    f.argtypes = [i32, i32, i32, i32, ctypes.POINTER(i32), i32, i32, i32, p64, p64]
    f.restype = ctypes.c_int

    def run(td3, bf16, obs, act, hidden, created, batch):
        cap, need = ctypes.c_int64(), ctypes.c_int64()
        h = (i32 * len(hidden))(*hidden)
        assert f(td3, bf16, obs, act, h, len(hidden), created, batch, ctypes.byref(cap), ctypes.byref(need)) == 0
        return cap.value, need.value
    return run


@pytest.mark.parametrize("td3,bf16,obs,act,hidden,batch,need", [
    (0, 0, 17, 6, (256, 256), 32768, 7864320), (0, 1, 17, 6, (256, 256), 65536, 7864320),
    (0, 1, 11, 3, (256, 256), 98304, 7864320), (1, 0, 111, 8, (400, 300), 16384, 7151616),
    (1, 1, 17, 6, (400, 300), 32768, 7142400), (0, 1, 67, 21, (256, 256, 256), 32768, 7995392),
    (0, 1, 17, 6, (512, 512), 20000, 7962624)])
def test_joint_launch_needs_the_most(workspace, td3, bf16, obs, act, hidden, batch, need):
    assert workspace(td3, bf16, obs, act, hidden, batch, batch) == (need, need)


def test_workspace_covers_every_launch_and_batch(workspace):
    rng = random.Random(7)
    fits = 0
    for _ in range(40000):
        obs, act = round(math.exp(rng.uniform(0, 6.3))), round(math.exp(rng.uniform(0, 3.4)))
        created = round(math.exp(rng.uniform(0, math.log(300000))))
        batch = created if rng.random() < 0.5 else rng.randint(1, created)
        case = (rng.randint(0, 1), rng.randint(0, 1), obs, act, rng.choice(HIDDEN), created, batch)
        cap, need = workspace(*case)
        fits += need > 0
        assert cap >= need, case
    assert fits > 20000


@pytest.mark.parametrize("td3,bf16,seq,streams,graphs,obs,hidden,expect", [
    # float32: everything, but for long weights with few tiles
    (0, 0, 0, 2, 0, 17, (256, 256), (1, 2**31 - 1)), (0, 0, 1, 2, 0, 376, (256, 256), (1, 2**31 - 1)),
    (0, 0, 1, 2, 0, 17, (400, 300), (1, 2**31 - 1)), (0, 0, 1, 2, 0, 376, (400, 300), (3072, 2**31 - 1)),
    (0, 0, 0, 2, 0, 376, (400, 300), (1, 2**31 - 1)), (0, 0, 0, 2, 1, 376, (400, 300), (2048, 2**31 - 1)),
    (0, 0, 0, 1, 1, 376, (512, 512, 512), (1, 2**31 - 1)), (0, 0, 0, 2, 0, 17, (512, 512, 512), (2048, 2**31 - 1)),
    (1, 0, 0, 1, 0, 376, (400, 300), (2048, 2**31 - 1)), (1, 0, 1, 1, 0, 17, (512, 512), (3072, 2**31 - 1)),
    # bfloat16: ragged layers everywhere; 128-multiple ones up to where a tile's weights cost most
    (0, 1, 0, 2, 0, 376, (400, 300), (1, 2**31 - 1)), (0, 1, 0, 2, 0, 17, (256, 256), (1024, 2**31 - 1)),
    (0, 1, 0, 2, 0, 376, (256, 256), (1024, 65536)), (1, 1, 0, 2, 0, 376, (256, 256), (1, 65536)),
    (0, 1, 0, 2, 0, 376, (128, 128), (1024, 2**31 - 1)), (0, 1, 0, 2, 0, 17, (512,) * 4, (1024, 32768)),
    (0, 1, 0, 2, 0, 17, (512, 512), (1024, 65536)), (0, 1, 0, 2, 0, 376, (512, 512), (1024, 16384)),
    (1, 1, 0, 2, 0, 376, (512, 512, 512), (1, 16384)), (0, 1, 0, 2, 0, 376, (512,) * 6, (1024, 8192)),
    (0, 1, 0, 2, 0, 376, (512, 480, 512), (1, 16384)), (0, 1, 0, 2, 0, 376, (384, 384, 384), (1024, 2**31 - 1)),
    # past the tiles
    (0, 1, 0, 2, 0, 17, (640,), (0, 0)), (0, 0, 0, 2, 0, 3000, (64, 64), (0, 0))])
def test_batches_of_the_row_tile_path(workspace, td3, bf16, seq, streams, graphs, obs, hidden, expect):
    from paper_2312_06126_amd import spz
    i32 = ctypes.c_int32
    lo, hi = i32(), i32()
    h = (i32 * len(hidden))(*hidden)
    assert spz.load().spzt_row_range(td3, bf16, seq, streams, graphs, obs, 6, h, len(hidden), ctypes.byref(lo),
                                     ctypes.byref(hi)) == 0
    assert (lo.value, hi.value) == expect
