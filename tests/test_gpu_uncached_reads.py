"""Batches whose K/V exceed the Infinity Cache are streamed with non-temporal loads, except where sessions share a prefix:
the results must be those of the reference kernel, whichever mixture of the two a session's segments take."""
import numpy as np
import pytest
import torch

from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,delta", [(32, 8, 128, 1), (32, 8, 128, 9), (32, 8, 128, 24), (32, 8, 64, 9), (24, 8, 128, 2)])
def test_large_batch_with_and_without_shared_prefixes(hq, hkv, d, delta):
    slots, per = 24, 3700 * 128 // d
    gen = torch.Generator(device="cuda")
    gen.manual_seed(delta)
    rows = lambda n, heads: torch.randn((n, heads, d), generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    pool = DevicePool(slots, slots * (per + 512) + 4096, hq, hkv, d, "bf16")
    assert slots * per * hkv * d * 4 > 256 << 20
    ids = [pool.acquire() for _ in range(slots)]
    pool.append(ids[:1], [0, 1500], rows(1500, hkv), rows(1500, hkv))
    for s in ids[1:6]:
        pool.alias(ids[0], s, 1333)  # five sessions share a prefix with the first, the others have their own
    hist = [per + 17 * i for i in range(slots)]
    cu = np.concatenate([[0], np.cumsum(hist)]).astype(np.int32)
    pool.append(ids, cu, rows(int(cu[-1]), hkv), rows(int(cu[-1]), hkv))
    total = slots * delta
    cu = np.arange(0, total + 1, delta, dtype=np.int32)
    q, kn, vn = rows(total, hq), rows(total, hkv), rows(total, hkv)
    out = pool.attend(ids, cu, q, d ** -0.5, kn, vn)
    dk.set_attend_variant(pool.handle, 1)
    ref = pool.attend(ids, cu, q, d ** -0.5, kn, vn)
    # the two differ by the rounding of the weights to bf16 (2^-9 each, averaged over thousands of keys) and by one bf16 step
    # of the stored results, at most 2^-7 of the value
    err = (out.float() - ref.float()).abs()
    bound = 2.0 ** -7 * ref.float().abs() + 2.0 ** -9 * ref.float().square().mean().sqrt() * 8
    assert torch.isfinite(out.float()).all() and (err <= bound).all(), float((err / bound).max())
    pool.close()
