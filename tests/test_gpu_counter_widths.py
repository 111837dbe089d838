"""Pair counts of a unit with more reverse lists than its 16-bit counters may gain between two flushes:
node 0 has the out-list {1, 2, 3} and `lists` reverse pairs from nodes joined to 0 and 1, each closing one
triangle with the edge {0, 1}.  With that edge first in the stream all of them add to its s, with it last
to its L; in between, to both.  Against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lists", [32767, 32769, 70000])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_pair_counts_past_a_round(cuda, lists, where):
    import torch
    from paper_1811_09136_amd import rept
    y = 4 + np.arange(lists, dtype=np.uint32)
    z = 4 + lists + np.arange(lists + 100, dtype=np.uint32)

    def pair(v, x):
        return np.stack([v, np.full(len(v), x, np.uint32)], 1)
    e = np.concatenate([pair(y, 0), pair(y, 1), pair(z[:10], 1), pair(z, 2), pair(z, 3), [[0, 2], [0, 3]]])
    e = synth.shuffled(e.astype(np.uint32), 3, flip_seed=4)
    at = {"first": 0, "middle": len(e) // 2, "last": len(e)}[where]
    e = np.ascontiguousarray(np.concatenate([e[:at], [[0, 1]], e[at:]]).astype(np.uint32))
    n = 4 + 2 * lists + 100
    ed, el, vd, vl = oracle.rept2_eta(e, n, 1, 1, 9)
    if where == "first":
        assert int(ed[0]) >= lists * (lists - 1) // 2
    g = rept.Graph(rept.to_device_edges(e, cuda), n)
    for shape in (dict(), dict(blocks=1), dict(blocks=1, phase_launches=1)):
        print("[case]", lists, where, shape, flush=True)
        glob, loc, eta, eta_v = g.count_eta(rept.Params(1, 1, 9), tuning=rept.tuning(**shape))
        torch.cuda.synchronize()
        assert int(glob[0]) == lists, shape
        assert eta.cpu().numpy().tolist() == [ed.tolist(), el.tolist()], shape
        assert np.array_equal(eta_v.cpu().numpy(), np.stack([vd, vl])), shape
    g.close()
