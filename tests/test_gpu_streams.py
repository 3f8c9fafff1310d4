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
