"""The general MFMA kernels (64-wide heads, groups of query heads that are no power of two up to 16) and the fp32 kernel
against the oracle, at the edges of their row blocks, key tiles and key splits, and against the reference kernel where a
call falls back to it.

Bounds.  bf16: the probabilities enter the second product with 16 bits of mantissa and everything else is fp32, so a result is off
by the rounding of the bf16 store, at most 2^-8 |o|, plus about 2^-16 of the largest |v| (asserted: 2^-14).  fp32: a score
sums up to 128 products of order one, a result a few thousand weighted values: a few 2^-22 of the largest |v| (asserted:
2^-18)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import Mirror, to_dev
from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk
from paper_2605_26289_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(out, ref, vmax, what, dtype="bf16"):
    g = out.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all(), what
    diff = np.abs(g - ref)
    bound = 2.0 ** -8 * np.abs(ref) + 2.0 ** -14 * vmax if dtype == "bf16" else np.full_like(ref, 2.0 ** -18 * vmax)
    assert (diff <= bound).all(), (what, float((diff / bound).max()), float(diff.max()))


SHAPES = [(4, 4, 64, "bf16"), (8, 2, 64, "bf16"), (14, 2, 64, "bf16"), (6, 2, 128, "bf16"), (5, 1, 128, "bf16"),
          (32, 1, 128, "bf16"), (24, 8, 128, "bf16"), (4, 1, 64, "f32"), (4, 4, 64, "f32"), (6, 2, 64, "f32"),
          (8, 2, 128, "f32"), (5, 1, 128, "f32"), (32, 8, 128, "f32")]
# packed rows on both sides of the stream kernel's blocks (32, 64, 96) and of the block kernel's 128, keys on both sides of
# the tiles of 16, 32 and 64 keys (and, fp32, on both sides of what takes items of 16 or 32 rows), and ranges long enough to be cut
SIZES = [(0, 1), (1, 2), (63, 1), (64, 9), (200, 21), (31, 33), (700, 43), (3000, 2), (2500, 65), (129, 150)]


@pytest.mark.parametrize("hq,hkv,d,dtype", SHAPES)
def test_shapes_that_no_tile_kernel_serves(hq, hkv, d, dtype):
    sh = wl.Shape(hq, hkv, d, dtype)
    for n, delta in SIZES:
        m = Mirror(sh, 2, n + delta + 256, granule=32, seed=hq * 1000 + n + delta)
        m.pool.k_arena.fill_(float("nan"))  # cells outside the slots must never reach a result
        m.pool.v_arena.fill_(float("nan"))
        s, t = m.acquire(), m.acquire()
        if n:
            m.append([s], [n])
            m.alias(s, t, max(1, n - 5)) if n > 1 else None
        nt = m.pool.length(t)
        q = m.draw(2 * delta, hq)
        kn, vn = m.draw(2 * delta, hkv), m.draw(2 * delta, hkv)
        cu = [0, delta, 2 * delta]
        lse = torch.empty((2 * delta, hq), dtype=torch.float32, device="cuda")
        out = m.pool.attend([s, t], cu, to_dev(q, dtype), sh.scale, to_dev(kn, dtype), to_dev(vn, dtype), lse=lse)
        refs = [oracle.delta_attend(q[cu[b]:cu[b + 1]], *m.cache(x), kn[cu[b]:cu[b + 1]], vn[cu[b]:cu[b + 1]], sh.scale)
                for b, x in enumerate((s, t))]
        ref, ref_lse = np.concatenate([r[0] for r in refs]), np.concatenate([r[1] for r in refs])
        vmax = max(np.abs(vn).max(), np.abs(m.cache(s)[1]).max() if n else 0.0)
        _check(out, ref, vmax, ("staged", n, delta), dtype)
        assert np.abs(lse.cpu().numpy() - ref_lse).max() < 1e-4, (n, delta)
        # the same rows appended and attended in one call
        out = m.pool.append_attend([s, t], cu, to_dev(q, dtype), to_dev(kn, dtype), to_dev(vn, dtype), sh.scale)
        _check(out, ref, vmax, ("fused", n, delta), dtype)
        for b, x in enumerate((s, t)):
            m.model.append(x, kn[cu[b]:cu[b + 1]], vn[cu[b]:cu[b + 1]])
            m.check_gather(x)
        assert m.pool.length(t) == nt + delta
        m.pool.close()


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 64), (12, 4, 128)])
def test_general_kernels_walk_chains_and_queues(hq, hkv, d):
    """More units than workgroups: planned chains and the run-time queue of the stream kernel, chains of the block kernel,
    next to empty entries; the scores keep outgrowing the reference maximum."""
    sh = wl.Shape(hq, hkv, d, "bf16")
    rng = np.random.default_rng(3)
    n_slots = 600
    m = Mirror(sh, n_slots, n_slots * 260, granule=16, seed=d)
    slots = [m.acquire() for _ in range(n_slots)]
    hist = rng.integers(1, 200, size=n_slots).tolist()
    m.append(slots, hist)
    deltas = rng.integers(0, 4, size=n_slots).tolist()
    for i in rng.choice(n_slots, 12, replace=False):
        deltas[i] = int(rng.integers(30, 90))
    total = sum(deltas)
    q, kn, vn = m.draw(total, hq), m.draw(total, hkv), m.draw(total, hkv)
    kn = wl.round_to_bf16(kn + 4.0 * np.sign(q[:, :: hq // hkv]))  # later keys score far higher
    for queue in (1, 0):
        dk.set_tuning(m.pool.handle, "stream_queue", queue)
        cu = np.concatenate([[0], np.cumsum(deltas)]).astype(np.int32)
        out = m.pool.attend(slots, cu, to_dev(q, "bf16"), sh.scale, to_dev(kn, "bf16"), to_dev(vn, "bf16"))
        ref, _ = oracle.delta_attend_batch(q, [m.cache(s) for s in slots], kn, vn, cu, sh.scale)
        assert dk.last_plan(m.pool.handle)["route"] == "general"
        _check(out, ref, max(np.abs(vn).max(), 5.0), queue)
    m.pool.close()


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 64), (12, 4, 128)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_scores_whose_partial_sums_over_depth_cancel(hq, hkv, d, sign):
    """The last 16 channels take back what the 16 before them give (24 x 24 x 16, exact in fp32): a score read before its last
    product has arrived is off by a thousand log2 units, and a row's reference maximum with it, upwards or downwards."""
    sh = wl.Shape(hq, hkv, d, "bf16")
    delta, n = 150, 800
    m = Mirror(sh, 1, n + delta + 512, granule=32, seed=d)
    s = m.acquire()
    k, v = m.draw(n, hkv), m.draw(n, hkv)
    q, kn, vn = m.draw(delta, hq), m.draw(delta, hkv), m.draw(delta, hkv)
    for x in (k, kn):
        x[..., d - 32:] = 24.0
    q[..., d - 32:d - 16], q[..., d - 16:] = sign * 24.0, sign * -24.0
    m.append([s], [n], k, v)
    dk.set_tuning(m.pool.handle, "small_units", 0)  # (the block kernel)
    out = m.pool.attend([s], [0, delta], to_dev(q, "bf16"), sh.scale, to_dev(kn, "bf16"), to_dev(vn, "bf16"))
    plan = dk.last_plan(m.pool.handle)
    assert plan["route"] == "general" and plan["stream_items"] == 0 and plan["row_items"] > 0, plan
    ref, _ = oracle.delta_attend(q, k, v, kn, vn, sh.scale)
    _check(out, ref, max(np.abs(v).max(), np.abs(vn).max()), sign)
    m.pool.close()


# descriptors: in the kernel arguments of either kernel, only of the scalar one (in one mode, in both), of neither
@pytest.mark.parametrize("hq,hkv,d,dtype,sessions,scalar", [
    (32, 8, 64, "bf16", 24, ()), (32, 8, 64, "bf16", 32, ("staged",)), (32, 8, 64, "bf16", 40, ("staged", "fused", "appended")),
    (24, 8, 128, "bf16", 40, ("staged", "fused", "appended")), (6, 2, 128, "bf16", 56, ("fused", "appended")),
    (32, 8, 64, "bf16", 100, ("staged", "fused", "appended")), (4, 1, 64, "f32", 24, ()), (4, 1, 64, "f32", 40, ("staged", "fused", "appended")),
    (4, 1, 64, "f32", 64, ()), (8, 8, 128, "f32", 100, ("staged", "fused", "appended")),
])
def test_many_short_sessions(hq, hkv, d, dtype, sessions, scalar):
    """Batches on both sides of the rule that leaves many short sessions to the scalar kernel: results of either kernel, in
    every mode, with entries that have nothing new."""
    sh = wl.Shape(hq, hkv, d, dtype)
    rng = np.random.default_rng(sessions)
    m = Mirror(sh, sessions, sessions * 96, granule=16, seed=d + hq)
    slots = [m.acquire() for _ in range(sessions)]
    m.append(slots, rng.integers(1, 21, size=sessions).tolist())
    deltas = rng.integers(1, 3, size=sessions)
    deltas[::7] = 0
    cu = np.concatenate([[0], np.cumsum(deltas)])
    q, kn, vn = (m.draw(int(cu[-1]), h) for h in (hq, hkv, hkv))
    refs = [oracle.delta_attend(q[cu[b]:cu[b + 1]], *m.cache(s), kn[cu[b]:cu[b + 1]], vn[cu[b]:cu[b + 1]], sh.scale)
            for b, s in enumerate(slots) if deltas[b]]
    ref, ref_lse = (np.concatenate([r[i] for r in refs]) for i in (0, 1))
    vmax = max([np.abs(vn).max()] + [np.abs(m.cache(s)[1]).max() for s in slots])
    qd, kd, vd = (to_dev(x, dtype) for x in (q, kn, vn))
    h, past = m.pool.handle, [m.pool.length(s) for s in slots]
    matrix = "general" if dtype == "bf16" else "f32"
    for units, to_scalar in ((256, scalar), (0, ())):
        dk.set_tuning(h, "small_units", units)
        lse = torch.empty((int(cu[-1]), hq), dtype=torch.float32, device="cuda")
        for mode in ("staged", "fused", "appended"):
            if mode == "fused":
                out = m.pool.append_attend(slots, cu, qd, kd, vd, sh.scale, lse=lse)
            else:
                out = m.pool.attend(slots, cu, qd, sh.scale, *((kd, vd) if mode == "staged" else ()), lse=lse)
            assert dk.last_plan(h)["route"] == ("scalar" if mode in to_scalar else matrix), (mode, dk.last_plan(h))
            _check(out, ref, vmax, (mode, units), dtype)
            assert np.abs(lse.cpu().numpy() - ref_lse).max() < 1e-4, (mode, units)
        m.pool.trim_batch(slots, past)
    m.pool.close()


def test_calls_that_only_have_room_for_the_reference_kernel_still_run():
    """No room for partials, or rows at an address that is no multiple of 16: the result is the reference kernel's."""
    sh = wl.Shape(6, 2, 128, "bf16")
    m = Mirror(sh, 1, 8192, seed=9)
    s = m.acquire()
    m.append([s], [6000])
    q, kn, vn = (to_dev(m.draw(3, h), "bf16") for h in (6, 2, 2))
    h = m.pool.handle
    need = dk.attend_workspace_bytes(h, [s], [0, 3], True)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    general, short, odd, ref = (torch.empty_like(q) for _ in range(4))
    dk.delta_attend(h, [s], [0, 3], q, general, sh.scale, kn, vn, workspace=ws)
    dk.delta_attend(h, [s], [0, 3], q, short, sh.scale, kn, vn, workspace=ws[:4096])
    shifted = torch.empty(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view_as(q).copy_(q)
    dk.delta_attend(h, [s], [0, 3], shifted, odd, sh.scale, kn, vn, workspace=ws)
    dk.set_attend_variant(h, 1)
    assert dk.attend_workspace_bytes(h, [s], [0, 3], True) <= 4096 < need
    dk.delta_attend(h, [s], [0, 3], q, ref, sh.scale, kn, vn, workspace=ws[:4096])
    assert torch.equal(short, ref) and torch.equal(odd, ref)
    assert (general.float() - ref.float()).abs().max().item() < 2e-2
    m.pool.close()


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 2, 64, "bf16"), (6, 2, 128, "bf16"), (4, 1, 64, "f32"), (6, 2, 128, "f32")])
@pytest.mark.parametrize("n,delta", [(100, 8), (40, 70), (5000, 5)])
def test_values_a_row_may_not_see_never_reach_it(hq, hkv, d, dtype, n, delta):
    """Infinities and NaN in V at some of the new tokens: rows before them stay finite and right, rows from them on carry
    them on, exactly as the reference kernel has it."""
    sh = wl.Shape(hq, hkv, d, dtype)
    m = Mirror(sh, 1, n + 512, seed=4)
    s = m.acquire()
    m.append([s], [n])
    q, kn, vn = (to_dev(m.draw(delta, x), dtype) for x in (hq, hkv, hkv))
    vn[delta // 2, 0, 3] = float("inf")
    vn[delta // 2 + 1, hkv - 1, 5] = float("nan")
    vn[delta - 1, 0, d - 1] = float("-inf")
    kn[delta - 1, 0, 7] = float("nan")
    out = m.pool.attend([s], [0, delta], q, sh.scale, kn, vn)
    dk.set_attend_variant(m.pool.handle, 1)
    ref = m.pool.attend([s], [0, delta], q, sh.scale, kn, vn)
    assert torch.equal(torch.isfinite(out), torch.isfinite(ref)) and torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(out[torch.isinf(out)], ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    assert ok[: delta // 2].all()
    assert (out[ok].float() - ref[ok].float()).abs().max().item() <= (2.0 ** -6 if dtype == "bf16" else 2.0 ** -17)
    m.pool.close()


def _time_us(call, reps=5):
    call()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        call()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / reps * 1e3


@pytest.mark.parametrize("hq,hkv,d,dtype", [(32, 8, 64, "bf16"), (24, 8, 128, "bf16"), (5, 1, 128, "bf16"), (8, 2, 64, "f32"), (8, 2, 128, "f32")])
@pytest.mark.parametrize("delta", [1, 9, 200, 600])
def test_infinities_in_a_sessions_history_are_carried_on_at_no_great_cost(hq, hkv, d, dtype, delta):
    """Non-finite values that every row sees: all rows are done again, over the keys they see, with the reference kernel's
    results, the same bits on every call, and in no more than twice the reference kernel's time (it walked them row by row
    once, 15 times as long as that kernel)."""
    sh = wl.Shape(hq, hkv, d, dtype)
    n = 2000
    m = Mirror(sh, 1, n + 1024, seed=6)
    s = m.acquire()
    k, v = (to_dev(m.draw(n, hkv), dtype) for _ in range(2))
    v[5] = float("inf")
    v[700, hkv - 1, 1::2] = float("nan")
    v[1500, 0, 2::4] = float("-inf")
    m.pool.append([s], [0, n], k, v)
    q, kn, vn = (to_dev(m.draw(delta, x), dtype) for x in (hq, hkv, hkv))
    vn[delta // 2, 0, 3] = float("nan")
    out = torch.empty_like(q)
    call = lambda: m.pool.attend([s], [0, delta], q, sh.scale, kn, vn, out=out)  # noqa: E731
    call()
    first = out.clone()
    assert dk.last_plan(m.pool.handle)["route"] != "scalar"
    whole = torch.int16 if dtype == "bf16" else torch.int32
    for _ in range(8):
        out.zero_()
        call()
        assert torch.equal(out.view(whole), first.view(whole))
    us = _time_us(call)
    dk.set_attend_variant(m.pool.handle, 1)
    call()
    assert torch.equal(torch.isnan(out), torch.isnan(first)) and torch.equal(torch.isinf(out), torch.isinf(first))
    assert torch.equal(out[torch.isinf(out)], first[torch.isinf(first)])
    ok = torch.isfinite(out)
    if ok.any():
        assert (out[ok].float() - first[ok].float()).abs().max().item() <= (2.0 ** -6 if dtype == "bf16" else 2.0 ** -17)
    scalar_us = _time_us(call)
    print(f"[non-finite] {hq}/{hkv}/{d} {dtype} delta {delta}: {us:.0f} us, scalar kernel {scalar_us:.0f} us")
    assert us <= 2.0 * scalar_us + 50.0
    m.pool.close()


def test_rows_of_very_many_kv_heads():
    """2^16 KV heads of 128: a staged row is 2^24 bytes from the next, past the matrix kernels' 24-bit row offsets."""
    h, d, n, delta = 1 << 16, 128, 2, 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(24)
    rows = lambda t: torch.randn((t, h, d), generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    pool = DevicePool(1, 16, h, h, d, "bf16", granule_cells=16)
    s = pool.acquire()
    k, v, q, kn, vn = rows(n), rows(n), rows(delta), rows(delta), rows(delta)
    pool.append([s], [0, n], k, v)
    out = pool.attend([s], [0, delta], q, d ** -0.5, kn, vn)
    assert dk.last_plan(pool.handle)["route"] == "scalar"
    pick = torch.tensor([0, 1, h // 2, h - 1], device="cuda")
    ks, vs = (torch.cat(x)[:, pick].float() for x in ((k, kn), (v, vn)))
    score = (q[:, pick].float()[:, None] * ks[None]).sum(-1) * d ** -0.5  # [token, key, head]
    hidden = torch.arange(n + delta, device="cuda")[None] > n + torch.arange(delta, device="cuda")[:, None]
    p = torch.softmax(score.masked_fill(hidden[..., None], float("-inf")), dim=1)
    ref = (p[..., None] * vs[None]).sum(1)
    # (fp32 sums; the result stored as bf16)
    assert ((out[:, pick].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all()
    pool.close()
