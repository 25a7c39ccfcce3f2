"""Predictions in flight together: the scratch that the calls share per GPU is theirs alone
while they run, whatever streams, outputs and graphs they use."""
import numpy as np
import pytest

from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def _rows(n, d, rng):
    x = np.abs(rng.standard_normal((n, d)))
    return x / np.sqrt((x * x).sum(axis=1))[:, None]


class Request:
    """A prediction with a handle and an output of its own."""

    def __init__(self, n_configs, d, M, seed, out=None):
        import torch

        from paper_2207_03803_amd import gap

        rng = np.random.default_rng(seed)
        counts = rng.integers(1, 60, n_configs)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
        self.X, self.offsets = to_dev(_rows(int(offsets[-1]), d, rng)), to_dev(offsets)
        self.XM, self.c = to_dev(_rows(M, d, rng)), to_dev(rng.standard_normal(M))
        self.out = torch.empty(n_configs, dtype=torch.float64, device="cuda")
        self.params = gap.params(d, 2)

    def enqueue(self, stream=None, out=None):
        from paper_2207_03803_amd import gap

        h = gap.Handle(self.params, stream=stream)
        h.set_model(self.XM)
        h.predict(self.X, self.offsets, self.c, self.out if out is None else out)
        return h

    def alone(self):
        import torch

        h = self.enqueue()
        torch.cuda.synchronize()
        h.close()
        return self.out.clone()


def _requests(n):
    rng = np.random.default_rng(17)
    return [Request(int(rng.integers(1, 400)), int(rng.integers(5, 80)), int(rng.integers(20, 900)), 100 + i)
            for i in range(n)]


def test_many_requests_in_flight_give_what_each_gives_alone():
    import torch

    reqs = _requests(48)
    expect = [r.alone() for r in reqs]
    streams = [torch.cuda.Stream() for _ in range(8)]
    for rep in range(3):
        for r in reqs:
            r.out.fill_(float("nan"))
        torch.cuda.synchronize()
        handles = [r.enqueue(streams[i % 8]) for i, r in enumerate(reqs)]
        torch.cuda.synchronize()
        for h in handles:
            h.close()
        for i, (r, e) in enumerate(zip(reqs, expect)):
            assert torch.equal(r.out, e), (rep, i)


def test_an_output_written_from_outside_does_not_reach_other_requests():
    """A call's state does not lie in its output: an output that other work overwrites all the
    time with numbers of every size (each also a plausible index as bits) spoils itself
    only, and as often as one likes."""
    import torch

    reqs = _requests(6)
    expect = [r.alone() for r in reqs]
    a, b, scribbler = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    bits = torch.tensor([0, 1, 31, 32, 40, 1 << 20, -1, 1 << 62], dtype=torch.int64, device="cuda").view(torch.float64)
    shared = torch.zeros(400, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for rep in range(20):
        handles = []
        for i, r in enumerate(reqs):
            out = shared[:r.out.numel()] if i < 3 else None
            handles.append(r.enqueue(a if i % 2 else b, out))
            with torch.cuda.stream(scribbler):
                shared.copy_(bits.repeat(50))
        torch.cuda.synchronize()
        for h in handles:
            h.close()
        for i in range(3, 6):
            assert torch.equal(reqs[i].out, expect[i]), (rep, i)
    for r, e in zip(reqs, expect):
        assert torch.equal(r.alone(), e)


def test_captured_predictions_replay_beside_others():
    import torch

    reqs = _requests(6)
    expect = [r.alone() for r in reqs]
    graphs, keep = [], []
    for r in reqs[:3]:
        s = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            keep.append(r.enqueue(s))
        graphs.append((g, s))
    for rep in range(4):
        for r in reqs:
            r.out.fill_(float("nan"))
        torch.cuda.synchronize()
        handles = []
        for (g, s), r in zip(graphs, reqs[3:]):
            with torch.cuda.stream(s):
                g.replay()
            handles.append(r.enqueue(torch.cuda.current_stream()))
        torch.cuda.synchronize()
        for h in handles:
            h.close()
        for i, (r, e) in enumerate(zip(reqs, expect)):
            assert torch.equal(r.out, e), (rep, i)
    for h in keep:
        h.close()
