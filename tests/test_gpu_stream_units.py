"""Streaming units of one, two and three row blocks in one launch: each workgroup one unit, or chains of them (whose first unit
has the most row blocks), and entries that are cut into tiles and pieces of their own."""
import numpy as np
import pytest
import torch

from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk

pytestmark = pytest.mark.gpu

# rows per KV head on both sides of a block (31, 32, 33, 64, 65, 96), keys on both sides of a 32- or 64-key tile and of a piece
SHAPES = [(32, 8, 128), (31, 1, 128), (8, 8, 128), (32, 8, 64), (24, 8, 128)]


@pytest.mark.parametrize("small_units,repeat", [(256, 1), (0, 1), (0, 12)])
@pytest.mark.parametrize("hq,hkv,d", SHAPES)
def test_units_of_all_heights(hq, hkv, d, small_units, repeat):
    group = hq // hkv
    gen = torch.Generator(device="cuda")
    gen.manual_seed(group * d + repeat)
    rows = lambda n, h: torch.randn((n, h, d), generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    hist = [63, 511, 1, 1029, 130, 2048] * repeat
    delta = [max(1, r // group) for r in (31, 32, 33, 64, 65, 96)] * repeat
    pool = DevicePool(len(hist), sum(hist) + sum(delta) + 512 * (len(hist) + 2), hq, hkv, d, "bf16")
    dk.set_tuning(pool.handle, "small_units", small_units)
    slots = [pool.acquire() for _ in hist]
    pool.append(slots, np.concatenate([[0], np.cumsum(hist)]).astype(np.int32), rows(sum(hist), hkv), rows(sum(hist), hkv))
    cu = np.concatenate([[0], np.cumsum(delta)]).astype(np.int32)
    q, k, v = rows(sum(delta), hq), rows(sum(delta), hkv), rows(sum(delta), hkv)
    lse = torch.empty((sum(delta), hq), dtype=torch.float32, device="cuda")
    out = pool.attend(slots, cu, q, d ** -0.5, k, v, lse=lse).clone()
    plan, got = dk.last_plan(pool.handle), lse.clone()
    assert plan["stream_items"] > 0 or d == 64  # (64-wide heads: more than 64 rows may take the whole batch elsewhere)
    dk.set_attend_variant(pool.handle, 1)
    ref = pool.attend(slots, cu, q, d ** -0.5, k, v, lse=lse).float()
    # weights as bf16: 2^-9 of each term of a row's weighted sum, whose terms are at most the largest |v| of the row's keys
    # times weights that sum to one; both results stored as bf16: 2^-8 of the value each
    bound = 2.0 ** -7 * ref.abs() + 2.0 ** -8 * 6.0
    assert ((out.float() - ref).abs() <= bound).all()
    assert (got - lse).abs().max().item() < 1e-3
    pool.close()
