"""Workspace sizes and kernels planned for the attention calls (host planner through the C ABI, no GPU)."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2605_26289_amd import binding as dk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _pool(n_slots, arena_cells, hq, hkv, d=128, dtype=dk.BF16, granule=0):
    return dk.pool_create(dk.PoolDesc(n_slots, 0, arena_cells, granule, hq, hkv, d, dtype, 256 * 10, 256 * 20, 256 * 30, 1 << 20))


def _fused_and_appended(hq, hkv, hist, delta, d=128, dtype=dk.BF16, granule=0):
    """(bytes the query for append_attend asks for, bytes the batch needs once its tokens have been appended)"""
    pool = _pool(len(hist), sum(hist) + sum(delta) + 1024 * (len(hist) + 1), hq, hkv, d, dtype, granule)
    slots = [dk.seq_acquire(pool) for _ in hist]
    dk.kv_reserve(pool, slots, np.concatenate([[0], np.cumsum(hist)]))
    cu = np.concatenate([[0], np.cumsum(delta)])
    asked = dk.attend_workspace_bytes(pool, slots, cu, 2)
    dk.kv_reserve(pool, slots, cu)
    needed = dk.attend_workspace_bytes(pool, slots, cu, 0)
    dk.pool_destroy(pool)
    return asked, needed


@pytest.mark.parametrize("hq,hkv,hist,delta", [
    (32, 8, [23, 50, 2030, 200], [68, 269, 1, 128]),
    (32, 4, [168, 1, 1103, 217], [143, 150, 52, 63]),
    (8, 2, [3000 + 7 * i for i in range(17)], [1] * 17),
    (8, 2, [1146], [388]),
])
def test_the_query_for_append_attend_covers_the_plan_made_after_the_append(hq, hkv, hist, delta):
    asked, needed = _fused_and_appended(hq, hkv, hist, delta)
    assert asked >= needed


@pytest.mark.parametrize("seed", range(8))
def test_the_query_for_append_attend_covers_random_batches(seed):
    """Batches on both sides of what can be folded into the attention kernel, in every route of the planner: whatever the
    plan of the appended batch turns out to be, the query made before the append has asked for enough."""
    rng = np.random.default_rng(500 + seed)
    shapes = [(32, 8, 128, dk.BF16), (32, 4, 128, dk.BF16), (8, 2, 128, dk.BF16), (16, 1, 128, dk.BF16), (8, 8, 128, dk.BF16),
              (32, 8, 64, dk.BF16), (24, 8, 128, dk.BF16), (14, 2, 64, dk.BF16), (8, 2, 128, dk.F32), (4, 1, 64, dk.F32)]
    for _ in range(400):
        hq, hkv, d, dtype = shapes[int(rng.integers(len(shapes)))]
        n_seqs = int(rng.integers(1, 25))
        top = int(rng.choice([300, 3000, 16000]))
        hist = rng.integers(1, top, size=n_seqs).tolist()
        most = int(rng.choice([1, 9, 40, 150, 400]))
        delta = rng.integers(1, most + 1, size=n_seqs).tolist()
        granule = int(rng.choice([16, 64, 256]))
        asked, needed = _fused_and_appended(hq, hkv, hist, delta, d, dtype, granule)
        assert asked >= needed, (hq, hkv, d, dtype, hist, delta, granule, asked, needed)


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 2, 128, dk.BF16), (8, 2, 64, dk.BF16), (6, 2, 128, dk.BF16), (8, 2, 128, dk.F32)])
def test_a_batch_longer_than_the_pool_is_refused_before_its_arrays_are_read(hq, hkv, d, dtype):
    """n_seqs is checked against the slots, entry by entry: the arrays of a wrong call need not reach as far as it says.
    (In a process of its own, which a read past their end would kill.)"""
    code = f"""
import ctypes as C, numpy as np
from paper_2605_26289_amd import binding as dk
pool = dk.pool_create(dk.PoolDesc(2, 0, 4096, 0, {hq}, {hkv}, {d}, {dtype}, 256 * 10, 256 * 20, 256 * 30, 1 << 20))
s = dk.seq_acquire(pool)
slots, cu = np.array([s, s], dtype=np.int32), np.array([0, 0, 0], dtype=np.int32)
out = C.c_int64()
print(dk.STATUS_NAMES[dk.lib().dk_attend_workspace_bytes(pool, 1 << 30, slots.ctypes.data, cu.ctypes.data, 1, C.byref(out))])
"""
    run = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "DUP_SLOT", (run.returncode, run.stdout, run.stderr[-500:])


def _planned(hq, hkv, d, hist, delta, **tuning):
    pool = _pool(len(hist), sum(hist) + 1024 * (len(hist) + 1), hq, hkv, d)
    for name, value in tuning.items():
        dk.set_tuning(pool, name, value)
    slots = [dk.seq_acquire(pool) for _ in hist]
    dk.kv_reserve(pool, slots, np.concatenate([[0], np.cumsum(hist)]))
    dk.attend_workspace_bytes(pool, slots, np.concatenate([[0], np.cumsum(delta)]), 1)
    plan = dk.last_plan(pool)
    dk.pool_destroy(pool)
    return plan


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (8, 2, 128), (24, 8, 128), (32, 8, 64)])
def test_the_rule_for_small_batches_can_be_switched_off(hq, hkv, d):
    rows = hq // hkv
    hist, delta = [800, 300], [300 // rows, 3]
    small = _planned(hq, hkv, d, hist, delta)
    assert small["row_items"] == 0 and small["stream_items"] > 0
    assert _planned(hq, hkv, d, hist, delta, small_units=0)["row_items"] > 0
    assert _planned(hq, hkv, d, hist, delta, small_units=1)["row_items"] > 0


@pytest.mark.parametrize("hq,hkv", [(32, 8), (8, 2)])
@pytest.mark.parametrize("sessions", [1, 6, 24])
def test_a_row_limit_that_is_set_holds_in_batches_of_any_size(hq, hkv, sessions):
    """65 to 96 packed rows: to the streaming kernel, or to the tile kernel once the limit is below them."""
    group = hq // hkv
    delta = [64 // group + 1 + i % (32 // group) for i in range(sessions)]
    hist = [100 + 37 * i for i in range(sessions)]
    assert _planned(hq, hkv, 128, hist, delta)["row_items"] == 0
    assert _planned(hq, hkv, 128, hist, delta, stream_rows=96)["row_items"] == 0
    limited = _planned(hq, hkv, 128, hist, delta, stream_rows=64)
    assert limited["row_items"] > 0 and limited["stream_items"] == 0


@pytest.mark.parametrize("hq,hkv,hist,delta,rows", [
    # measured, us a step, streaming kernel in short row tiles / tile kernel
    (16, 16, [1749, 1550, 2523], [252, 195, 172], False),                                    # 27.7 / 41.6 (one height for all entries: 50.5)
    (32, 4, [1812, 1505, 2058, 1221, 777, 929, 1995, 2318, 1783, 2337, 1508, 2451, 2777, 894, 1732, 1892],
     [15, 22, 13, 13, 16, 14, 23, 15, 18, 16, 22, 23, 13, 22, 22, 22], False),                # 31.1 / 45.3 (one height: 54.9)
    (32, 8, [12798], [146], True),                                                           # 65.8 / 59.7
    (32, 8, [800], [150], False),                                                            # 17.8 / 33.5
    (8, 2, [1856, 700], [60, 50], False),
])
def test_small_batches_go_to_the_kernel_that_was_measured_faster(hq, hkv, hist, delta, rows):
    plan = _planned(hq, hkv, 128, hist, delta)
    assert (plan["row_items"] > 0) == rows and (plan["stream_items"] > 0) != rows
