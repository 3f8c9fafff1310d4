"""Outputs that the binding allocates for a context on a stream of its own."""

import numpy as np
import pytest

import paper_1208_0277_amd as sccg
import sccg_gen
from tests.gpu_util import device_workload

pytestmark = pytest.mark.gpu


def test_outputs_belong_to_the_contexts_stream():
    """Dropped outputs of a call that may still be running are not handed out
    to another stream's allocations."""
    import torch
    wl = sccg_gen.pairs(1)
    work = device_workload(wl.A, wl.B, wl.pa, wl.pb)
    torch.cuda.synchronize()
    c = sccg.Context(0, stream=torch.cuda.Stream())
    so = torch.tensor([0, wl.n_pairs], dtype=torch.int64, device="cuda")
    off = torch.tensor([0, wl.A.n], dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    try:
        I, U = c.area_pairs(*work)
        kept = [I, U, *c.jaccard_sets(so, I, U), *c.join_sets(work[0], work[1], off, off, cap=4 * wl.n_pairs),
                c.relate_pairs(*work, I), c.validate_polys(work[0])]
        held = {t.untyped_storage().data_ptr() for t in kept}
        sizes = [(t.untyped_storage().nbytes(), t.dtype) for t in kept]
        del kept, I, U
        fresh = [torch.empty(n // torch.empty(0, dtype=d).element_size(), dtype=d, device="cuda") for n, d in sizes]
        assert not held & {t.untyped_storage().data_ptr() for t in fresh}
        c.sync()
    finally:
        c.close()
    assert np.diff(wl.A.off).min() > 0


def test_outputs_read_on_the_current_stream_and_dropped():
    """Dropped outputs that work queued on the caller's stream still reads are
    not handed to the context's next call."""
    import torch
    wl = sccg_gen.pairs(1)
    work = device_workload(wl.A, wl.B, wl.pa, wl.pb)
    other = device_workload(wl.A, wl.B, wl.pa, np.roll(wl.pb, 1))
    so = torch.tensor([0, wl.n_pairs], dtype=torch.int64, device="cuda")
    off = torch.tensor([0, wl.A.n], dtype=torch.int64, device="cuda")
    x = torch.rand(8192, 8192, device="cuda")
    y = torch.empty_like(x)
    c = sccg.Context(0, stream=torch.cuda.Stream())

    def calls(w):
        I, U = c.area_pairs(*w)
        return [I, U, *c.jaccard_sets(so, I, U), c.relate_pairs(*w, I), c.validate_polys(w[0])]

    def join(w):  # waits for its stream, which may share a hardware queue with the readers
        return [*c.join_sets(w[0], w[1], off, off, cap=4 * wl.n_pairs)]

    try:
        calls(other), join(other)
        torch.cuda.synchronize()
        outs = calls(work) + join(work)
        c.sync()
        want = [t.cpu() for t in outs]
        reader = torch.cuda.Event()
        torch.cuda.synchronize()
        for _ in range(20):  # some hundred milliseconds that the readers wait behind
            torch.mm(x, x, out=y)
        got = [t.clone() for t in outs]
        reader.record()
        held = {t.untyped_storage().data_ptr() for t in outs}
        del outs
        again = calls(other)
        assert not reader.query(), "the readers had run before the calls: nothing was tested"
        again += join(other)
        assert not held & {t.untyped_storage().data_ptr() for t in again}
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g.cpu(), w)
    finally:
        c.close()


def test_outputs_without_the_raw_stream_getter(monkeypatch):
    """A torch without the private getter of the current stream's handle."""
    import torch
    wl = sccg_gen.pairs(1)
    work = device_workload(wl.A, wl.B, wl.pa, wl.pb)
    torch.cuda.synchronize()
    for stream in (None, torch.cuda.Stream()):
        c = sccg.Context(0, stream=stream) if stream else sccg.Context(0)
        try:
            want = [t.cpu() for t in c.area_pairs(*work)]
            with monkeypatch.context() as m:
                m.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
                got = c.area_pairs(*work)
            c.sync()
            for g, w in zip(got, want):
                assert torch.equal(g.cpu(), w)
        finally:
            c.close()
