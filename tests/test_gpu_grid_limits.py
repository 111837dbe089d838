"""Grids that cannot be launched (rept_tuning.blocks is the caller's): every counting call that takes a
launch shape refuses one with the same status, and the next call counts as before."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [dict(blocks=1 << 30), dict(blocks=1 << 24), dict(blocks=(1 << 32) - 1, threads=64),
                                   dict(blocks=1 << 28, threads=1024, phase_launches=1),
                                   dict(blocks=1 << 29, phase_launches=2)])
def test_grid_too_large(cuda, shape):
    import torch
    from paper_1811_09136_amd import rept
    from paper_1811_09136_amd.batch import Batch, Job
    n, p = 300, rept.Params(3, 7, 11)
    e = synth.er(n, 4000, 5, 6)
    g = rept.Graph(rept.to_device_edges(e, cuda), n)
    tu = rept.tuning(**shape)
    print("[case]", shape, flush=True)
    job = Job(g, p)
    for call in (Batch([job], tu).launch, Batch([job, Job(g, p)], tu).launch, lambda: g.count_eta(p, tuning=tu)):
        with pytest.raises(rept.ReptError) as ei:
            call()
        assert ei.value.code == rept.REPT_EDEVICE
    glob, loc = g.count(p)
    torch.cuda.synchronize()
    og, ol = oracle.rept(e, n, 3, 7, 11)
    assert np.array_equal(glob.cpu().numpy(), og) and np.array_equal(loc.cpu().numpy(), ol)
    g.close()
