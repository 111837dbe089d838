"""How the counting kernel cuts its units into tiles, at the sizes where a cut can go wrong, against
the oracle (or, where the oracle's replay would be long, a closed form).  All values are integers and
must be equal.

* light units counted several to a wavefront: a strip of triangles (lists of two entries, so passes
  end at the unit limit of 16), cliques of 9 to 17 nodes (passes end at the 64 table entries), and
  units whose reverse lists are empty;
* a unit with more reverse lists than a wavefront's 16-bit counters may gain between flushes, in one
  part and cut into many;
* more equally large nodes than the hub table holds, and one fewer.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

SHAPES = [dict(), dict(light_tile=1), dict(light_tile=64, blocks=3), dict(wave_cap=8), dict(phase_launches=1),
          dict(blocks=1, phase_launches=2)]


def _strip(k):
    """k nodes, each joined to the next two."""
    i = np.arange(k - 2, dtype=np.uint32)
    return np.concatenate([np.stack([i, i + 1], 1), np.stack([i, i + 2], 1), [[k - 2, k - 1]]]).astype(np.uint32)


def _cliques(sizes):
    at, out = 0, []
    for s in sizes:
        out.append(synth.complete(s) + at)
        at += s
    return np.concatenate(out).astype(np.uint32)


def _spokes(hubs, leaves):
    """`leaves` nodes joined to two neighbouring hubs each, the hubs in a ring and a second ring."""
    y = np.arange(leaves, dtype=np.uint32)
    h = [np.stack([hubs + y, (y + k) % hubs], 1) for k in (0, 1)]
    r = np.arange(hubs, dtype=np.uint32)
    ring = [np.stack([r, (r + k) % hubs], 1) for k in (1, 2)]
    return np.concatenate(h + ring).astype(np.uint32)


GRAPHS = {
    "strip": lambda: _strip(1003),
    "cliques": lambda: _cliques([9, 17, 12, 16, 10, 3, 3, 11] * 9),
    "bipartite-plus": lambda: np.concatenate([synth.complete_bipartite(5, 60), synth.complete(5)]).astype(np.uint32),
    "hubs-33": lambda: _spokes(33, 33 * 140),
    "hubs-32": lambda: _spokes(32, 32 * 140),
    "hubs-31": lambda: _spokes(31, 31 * 140),
}


def _count(cuda, e, n, P, shape):
    import torch
    from paper_1811_09136_amd import rept
    from paper_1811_09136_amd.batch import Batch, Job
    g = rept.Graph(rept.to_device_edges(e, cuda), n)
    j = Job(g, P)
    Batch([j], rept.tuning(**shape)).launch()
    torch.cuda.synchronize()
    out = j.out[0].cpu().numpy(), j.out[1].cpu().numpy()
    g.close()
    return out


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("m,c", [(1, 1), (3, 10), (2, 16)])
def test_tiles_against_oracle(cuda, name, m, c):
    from paper_1811_09136_amd import rept
    e = synth.shuffled(GRAPHS[name](), 5, flip_seed=6)
    n = int(e.max()) + 1
    og, ol = oracle.rept(e, n, m, c, 77)
    for shape in SHAPES:
        print("[case]", name, m, c, shape, flush=True)
        g, l = _count(cuda, e, n, rept.Params(m, c, 77), shape)
        assert np.array_equal(g, og) and np.array_equal(l, ol), shape


@pytest.mark.parametrize("lists", [32767, 32768, 32769, 70000])
def test_unit_with_many_reverse_lists(cuda, lists):
    """Node 0 has out-list {1, 2, 3} and `lists` reverse pairs from nodes joined to 0 and 1: every such
    node closes one triangle with them (m = 1 counts each once)."""
    from paper_1811_09136_amd import rept
    y = 4 + np.arange(lists, dtype=np.uint32)
    z = 4 + lists + np.arange(lists + 100, dtype=np.uint32)
    pair = lambda v, x: np.stack([v, np.full(len(v), x, np.uint32)], 1)
    e = np.concatenate([pair(y, 0), pair(y, 1), pair(z[:10], 1), pair(z, 2), pair(z, 3),
                        [[0, 1], [0, 2], [0, 3]]]).astype(np.uint32)
    e = synth.shuffled(e, 3, flip_seed=4)
    n = 4 + 2 * lists + 100
    for shape in (dict(), dict(blocks=1), dict(blocks=1, phase_launches=1)):
        print("[case]", lists, shape, flush=True)
        g, l = _count(cuda, e, n, rept.Params(1, 1, 9), shape)
        assert int(g[0]) == lists
        want = np.zeros(n, np.int64)
        want[[0, 1]] = lists
        want[y] = 1
        assert np.array_equal(l[0], want), shape


@pytest.mark.parametrize("nodes", [383, 384, 385, 386, 640, 1100])
def test_chunks_under_long_apexes(cuda, nodes):
    """A clique's apexes have every out-degree below `nodes`, and as many lists: chunks of even size
    below 384, shrinking ones from there (m = 1 counts every triangle once)."""
    from paper_1811_09136_amd import rept
    e = synth.shuffled(synth.complete(nodes), 3, flip_seed=4).astype(np.uint32)
    for shape in (dict(), dict(blocks=1), dict(wave_cap=8, blocks=3), dict(threads=128, wave_cap=8)):
        print("[case]", nodes, shape, flush=True)
        g, l = _count(cuda, e, nodes, rept.Params(1, 1, 9), shape)
        assert int(g[0]) == nodes * (nodes - 1) * (nodes - 2) // 6, shape
        assert (l[0] == (nodes - 1) * (nodes - 2) // 2).all(), shape
