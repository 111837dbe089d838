"""A captured batch launch replayed after its workspace is prepared for other jobs: the graph holds the
launch shape, the workspace the jobs, so a replay counts the jobs that the workspace holds by then, also
where the captured jobs had no unit for one of the phases."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _strip(k):
    """k nodes, each joined to the next two: no unit above any wave cap."""
    i = np.arange(k - 2, dtype=np.uint32)
    return np.concatenate([np.stack([i, i + 1], 1), np.stack([i, i + 2], 1), [[k - 2, k - 1]]]).astype(np.uint32)


@pytest.mark.parametrize("phase_launches", [0, 1, 2])
@pytest.mark.parametrize("jobs", [1, 3])
def test_replay_after_prepare(cuda, phase_launches, jobs):
    import torch
    from paper_1811_09136_amd import rept
    from paper_1811_09136_amd.batch import Job
    streams = {"light": (_strip(700), 700), "heavy": (synth.complete(120).astype(np.uint32), 120),
               "none": (np.array([[0, 1]], np.uint32), 2), "both": (synth.er(400, 9000, 3, 4), 400)}
    tu = rept.tuning(wave_cap=16, block_cap=256, b_chunk=64, threads=128, light_tile=8, phase_launches=phase_launches)
    table, want = {}, {}
    for name, (e, n) in streams.items():
        e = synth.shuffled(e, 5, flip_seed=6)
        g = rept.Graph(rept.to_device_edges(e, cuda), n)
        table[name] = [Job(g, rept.Params(3, 7, 11 + k)) for k in range(jobs)]
        want[name] = [oracle.rept(e, n, 3, 7, 11 + k) for k in range(jobs)]
    c_jobs = {name: [j.c_job() for j in js] for name, js in table.items()}
    nb = rept.rept_batch_workspace_size(jobs)
    for first in ("light", "none", "heavy"):
        ws = torch.empty(nb, dtype=torch.uint8, device=cuda)
        s = torch.cuda.current_stream().cuda_stream
        rept.rept_batch_prepare(c_jobs[first], tu, ws.data_ptr(), nb, s)
        rept.rept_batch_launch(ws.data_ptr(), s)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            rept.rept_batch_launch(ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
        for name in (first, "both", "heavy", "light", first, "none", "both", "both"):
            print("[case]", phase_launches, jobs, first, name, flush=True)
            rept.rept_batch_prepare(c_jobs[name], tu, ws.data_ptr(), nb, s)
            for j in table[name]:
                j.out[0].fill_(-1)
                j.out[1].fill_(-1)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for j, (og, ol) in zip(table[name], want[name]):
                assert np.array_equal(j.out[0].cpu().numpy(), og), (first, name)
                assert np.array_equal(j.out[1].cpu().numpy(), ol), (first, name)
