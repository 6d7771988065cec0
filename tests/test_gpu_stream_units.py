"""Streaming units of one, two and three row blocks in one launch: each workgroup one unit, or chains of them (whose first unit
has the most row blocks), and entries that are cut into tiles and pieces of their own."""
import numpy as np
import pytest
import torch

from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk

pytestmark = pytest.mark.gpu

# rows per KV head on both sides of a block (31, 32, 33, 64, 65, 96; with 64-wide heads the streaming kernel takes 64 beside
# longer ones), keys on both sides of a 32- or 64-key tile and of a piece, and enough of them for every stage to be used again
SHAPES = [(32, 8, 128), (31, 1, 128), (8, 8, 128), (32, 8, 64), (24, 8, 128)]


@pytest.mark.parametrize("small_units,repeat", [(256, 1), (0, 1), (0, 12)])
@pytest.mark.parametrize("hq,hkv,d", SHAPES)
def test_units_of_all_heights(hq, hkv, d, small_units, repeat):
    group = hq // hkv
    gen = torch.Generator(device="cuda")
    gen.manual_seed(group * d + repeat)
    rows = lambda n, h: torch.randn((n, h, d), generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    hist = [63, 511, 1, 1029, 130, 2048] * repeat + ([9001] if repeat == 1 else [])
    most = 64 if d == 64 else 96
    delta = [max(1, min(r, most) // group) for r in (31, 32, 33, 64, 65, 96)] * repeat + ([most // group] if repeat == 1 else [])
    cu_hist = np.concatenate([[0], np.cumsum(hist)]).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(delta)]).astype(np.int32)
    kh, vh = rows(sum(hist), hkv), rows(sum(hist), hkv)
    q, k, v = rows(sum(delta), hq), rows(sum(delta), hkv), rows(sum(delta), hkv)

    def attend(vh, v, scalar):
        pool = DevicePool(len(hist), sum(hist) + sum(delta) + 512 * (len(hist) + 2), hq, hkv, d, "bf16")
        dk.set_tuning(pool.handle, "small_units", small_units)
        dk.set_attend_variant(pool.handle, 1 if scalar else 0)
        slots = [pool.acquire() for _ in hist]
        pool.append(slots, cu_hist, kh, vh)
        lse = torch.empty((sum(delta), hq), dtype=torch.float32, device="cuda")
        out = pool.attend(slots, cu, q, d ** -0.5, k, v, lse=lse).float()
        plan = dk.last_plan(pool.handle)
        pool.close()
        return out, lse, plan

    out, lse, plan = attend(vh, v, False)
    assert plan["stream_items"] > 0 and plan["row_items"] == 0, plan
    ref, ref_lse, _ = attend(vh, v, True)
    absolute, _, _ = attend(vh.abs(), v.abs(), True)  # (each row's sum of p |v|)
    # Weights as bf16: at most 2^-8 of each term of a row's weighted sum (a tenth more for what the scores and exponentials of
    # both kernels differ in, 1e-4 by the check of the log-sum-exp); both results stored as bf16: 2^-8 of the value each.
    bound = 1.1 * 2.0 ** -8 * absolute + 2.0 ** -7 * ref.abs() + 1e-5
    diff = (out - ref).abs()
    assert (diff <= bound).all(), float((diff / bound).max())
    # Over a row's channels these are independent and uniform, 2^-8 / sqrt(3) each: of the row's norm that makes 2^-8 / sqrt(3)
    # for the weights (outputs are the norm of the weights in size, V being normal) and sqrt(2) times as much for the two stores,
    # 2^-8 together, allowed four times.  One 32-key tile of V taken for another is 8 % of a row over 9000 keys, 20 % over 1000.
    row = diff.norm(dim=-1) / ref.norm(dim=-1)
    print(f"worst element {float((diff / bound).max()):.2f} of its bound, worst row {float(row.max()):.2e}")
    assert row.max().item() <= 4 * 2.0 ** -8
    assert (lse - ref_lse).abs().max().item() < 1e-4
