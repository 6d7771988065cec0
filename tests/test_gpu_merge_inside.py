"""Small decoding batches, whose split rows the streaming kernel merges itself: the same bits on every call, on pools that run
at the same time on two streams, and in replays of a captured call (which merges by a kernel of its own)."""
import numpy as np
import pytest
import torch

from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk

pytestmark = pytest.mark.gpu


class Session:
    def __init__(self, hq, hkv, d, hist, delta, seed):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        self.rows = lambda n, h: torch.randn((n, h, d), generator=gen, device="cuda", dtype=torch.bfloat16)
        self.pool = DevicePool(len(hist), sum(hist) + 512 * len(hist) + 512, hq, hkv, d, "bf16")
        self.slots = [self.pool.acquire() for _ in hist]
        cu = np.concatenate([[0], np.cumsum(hist)]).astype(np.int32)
        self.pool.append(self.slots, cu, self.rows(sum(hist), hkv), self.rows(sum(hist), hkv))
        total = delta * len(hist)
        self.cu = np.arange(0, total + 1, delta, dtype=np.int32)
        self.q = [self.rows(total, hq) for _ in range(2)]
        self.k, self.v = self.rows(total, hkv), self.rows(total, hkv)
        self.scale = d ** -0.5
        self.lse = torch.empty((total, hq), dtype=torch.float32, device="cuda")
        self.pool.ensure_workspace(self.slots, self.cu, True)

    def attend(self, i, out=None):
        return self.pool.attend(self.slots, self.cu, self.q[i], self.scale, self.k, self.v, out=out, lse=self.lse)

    def reference(self, i):
        dk.set_attend_variant(self.pool.handle, 1)
        out = self.attend(i)
        lse = self.lse.clone()
        dk.set_attend_variant(self.pool.handle, 0)
        return out, lse


# rows per KV head 1..8, keys from just enough to be cut to a full complement of units, one to several sessions
CASES = [(32, 8, 128, [3000], 1), (8, 8, 128, [1500], 1), (32, 8, 128, [900, 6000, 2500], 2), (16, 1, 128, [20000], 1),
         (32, 8, 64, [3000], 1), (14, 2, 64, [5000, 700], 1), (24, 8, 128, [4000], 2), (8, 1, 128, [30000], 1)]


@pytest.mark.parametrize("hq,hkv,d,hist,delta", CASES)
def test_every_call_gives_the_same_bits(hq, hkv, d, hist, delta):
    s = Session(hq, hkv, d, hist, delta, 1)
    want = [s.attend(0).clone(), s.attend(1).clone()]
    for i in (0, 1):
        ref, lse = s.reference(i)
        s.attend(i)
        # rounding of the weights (2^-9 each over hundreds of keys) and of the stored results (2^-7 of the value between two)
        bound = 2.0 ** -7 * ref.float().abs() + 2.0 ** -6 * ref.float().square().mean().sqrt()
        assert ((want[i].float() - ref.float()).abs() <= bound).all()
        assert (s.lse - lse).abs().max().item() < 1e-3
    outs = [torch.empty_like(want[0]) for _ in range(40)]
    for rep in range(4):
        for j, o in enumerate(outs):
            s.attend(j & 1, o)
        torch.cuda.synchronize()
        assert all(torch.equal(o, want[j & 1]) for j, o in enumerate(outs)), rep
    s.pool.close()


def test_two_pools_on_two_streams():
    a, b = Session(32, 8, 128, [3000], 1, 2), Session(32, 8, 128, [5000], 1, 3)
    want = [a.attend(0).clone(), b.attend(0).clone()]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[torch.empty_like(want[i]) for _ in range(60)] for i in (0, 1)]
    for j in range(60):
        for i, s in enumerate((a, b)):
            with torch.cuda.stream(streams[i]):
                s.attend(0, outs[i][j])
    torch.cuda.synchronize()
    for i in (0, 1):
        assert all(torch.equal(o, want[i]) for o in outs[i])
    a.pool.close()
    b.pool.close()


def test_captured_calls_replay():
    s = Session(32, 8, 128, [3000], 1, 4)
    eager = s.attend(0).clone()
    out = torch.empty_like(eager)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s.attend(0, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        s.attend(0, out)
    results = []
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        results.append(out.clone())
        assert torch.equal(s.attend(0), eager)  # the pool goes on working between replays
        torch.cuda.synchronize()
    # the captured call merges in another order of additions: one bf16 step at the most, and always the same
    assert all(torch.equal(r, results[0]) for r in results)
    bound = 2.0 ** -7 * eager.float().abs() + 2.0 ** -9 * eager.float().square().mean().sqrt()
    assert ((results[0].float() - eager.float()).abs() <= bound).all()
    s.pool.close()
