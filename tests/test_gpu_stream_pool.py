"""Partitions share the library's streams between mini-batches: partitions that
are inside a mini-batch together, from one thread or several, and captures give
the bits of a partition on its own."""
import threading

import numpy as np
import pytest

import synth
from parity import to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CFG = synth.PartitionConfig("pool", layers=2, d_model=128, d_ff=256, heads=2, seq=64, batch=8, micro=4, dtype="bf16")


class Run:
    """One partition, driven call by call."""

    def __init__(self, seed):
        from paper_1811_06965_amd.runtime import Partition
        self.case = synth.make_case(CFG, seed, perturb=True)
        self.part = Partition(CFG)
        self.part.load_params(self.case["layers"], self.case["head"])
        self.inp = self.part.device_inputs(self.case)
        self.y, self.dx = torch.empty_like(self.inp["x"]), torch.empty_like(self.inp["x"])
        torch.cuda.synchronize()

    def _chunks(self, t):
        return [c.data_ptr() for c in t.chunk(CFG.micro)]

    def forwards(self, st):
        from paper_1811_06965_amd import gp
        for m, (x, y) in enumerate(zip(self._chunks(self.inp["x"]), self._chunks(self.y))):
            gp.gp_forward_microbatch(self.part.h, m, x, None, y, st)

    def backwards(self, st):
        from paper_1811_06965_amd import gp
        dy, dx = self._chunks(self.inp["dy"]), self._chunks(self.dx)
        for m in range(CFG.micro - 1, -1, -1):
            gp.gp_backward_microbatch_remat(self.part.h, m, dy[m], dx[m], None, st)

    def update(self, st, lr=1e-3):
        from paper_1811_06965_amd import gp
        gp.gp_accumulate_and_step(self.part.h, lr, False, st)

    def result(self):
        torch.cuda.synchronize()
        layers, _ = self.part.params()
        return [to_np(self.y), to_np(self.dx)] + [p[k] for p in layers for k in sorted(p)]

    def steps(self, n, st):
        for _ in range(n):
            self.forwards(st)
            self.backwards(st)
            self.update(st)


def _alone(seed, n):
    r = Run(seed)
    r.steps(n, torch.cuda.current_stream().cuda_stream)
    out = r.result()
    r.part.close()
    return out


def _same(a, b):
    assert len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def test_interleaved_mini_batches():
    st = torch.cuda.current_stream().cuda_stream
    a, b = Run(1), Run(2)
    for _ in range(2):
        a.forwards(st)
        b.forwards(st)
        a.backwards(st)
        b.backwards(st)
        b.update(st)
        a.update(st)
    ra, rb = a.result(), b.result()
    a.part.close()
    b.part.close()
    _same(ra, _alone(1, 2))
    _same(rb, _alone(2, 2))


def test_threads_with_their_own_partitions():
    runs = [Run(s) for s in (1, 2, 3)]
    streams = [torch.cuda.Stream() for _ in runs]
    errors = []

    def go(r, st):
        try:
            r.steps(3, st.cuda_stream)
            st.synchronize()
        except Exception as e:  # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=go, args=x) for x in zip(runs, streams)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    got = [r.result() for r in runs]
    for r in runs:
        r.part.close()
    for s, g in zip((1, 2, 3), got):
        _same(g, _alone(s, 3))


def test_capture_while_another_partition_is_inside_a_mini_batch():
    st = torch.cuda.current_stream().cuda_stream
    a, b = Run(1), Run(2)
    a.forwards(st)  # holds the idle pair
    torch.cuda.synchronize()
    g = b.part.capture_step(b.inp["x"], None, b.inp["dy"], lr=1e-3, dx=b.dx, want_y=True, y=b.y)
    a.backwards(st)
    g.replay()
    a.update(st)
    a.steps(1, st)  # eager work on the pairs between the replays
    g.replay()
    torch.cuda.synchronize()
    g.replay()
    ra, rb = a.result(), b.result()
    del g
    a.part.close()
    b.part.close()
    _same(ra, _alone(1, 2))
    _same(rb, _alone(2, 3))


def test_noalloc_forwards_while_another_partition_is_inside_a_mini_batch():
    """The other partition holds the idle pair of streams: the no-allocation
    forwards take none (they would have to create one), the backward does."""
    from paper_1811_06965_amd import gp
    st = torch.cuda.current_stream().cuda_stream
    a, b = Run(1), Run(2)
    a.forwards(st)
    for m, (x, y) in enumerate(zip(b._chunks(b.inp["x"]), b._chunks(b.y))):
        gp.gp_forward_microbatch_noalloc(b.part.h, m, x, None, y, st)
    b.backwards(st)
    a.backwards(st)
    a.update(st)
    b.update(st)
    ra, rb = a.result(), b.result()
    a.part.close()
    b.part.close()
    _same(ra, _alone(1, 1))
    _same(rb, _alone(2, 1))


def test_partitions_in_turn_on_streams_of_their_own():
    runs = [Run(s) for s in (1, 2)]
    streams = [torch.cuda.Stream() for _ in runs]
    for _ in range(3):
        for r, st in zip(runs, streams):
            r.steps(1, st.cuda_stream)
    got = [r.result() for r in runs]
    runs[0].part.close()  # its pair goes, the other partition's stays
    runs[1].steps(1, streams[0].cuda_stream)
    last = runs[1].result()
    runs[1].part.close()
    for s, g in zip((1, 2), got):
        _same(g, _alone(s, 3))
    _same(last, _alone(2, 4))
