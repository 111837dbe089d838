"""Incremental streams on the device: after every appended chunk the counters equal the
oracle's replay of the stream so far (bit for bit), for REPT (all group layouts) and parallel
MASCOT, whether appends count edge by edge or by a windowed recount of the prefix; invalid
chunks are refused and leave the state unchanged.

Each case prints its name and shape before touching the GPU."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _say(*a):
    print("[case]", *a, flush=True)


def _oracle(edges, n, p):
    if p.mascot:
        return oracle.mascot(edges, n, p.m, p.c, p.seed)
    return oracle.rept(edges, n, p.m, p.c, p.seed, per_proc=p.per_proc)


def _check(inc, edges_so_far, n, p):
    import torch
    torch.cuda.synchronize()
    og, ol = _oracle(edges_so_far, n, p)
    assert np.array_equal(inc.counts[0].cpu().numpy(), og)
    assert np.array_equal(inc.counts[1].cpu().numpy(), ol)
    assert inc.num_edges == len(edges_so_far)


def _paths_follow(inc, policy, appends):
    per_edge, recount = inc.paths()
    assert per_edge + recount == appends
    if policy == "per_edge":
        assert recount == 0
    elif policy == "recount":
        assert per_edge == 0


@pytest.mark.parametrize("policy", ["per_edge", "recount"])
@pytest.mark.parametrize("m,c,per_proc,mascot", [(3, 7, False, False), (1, 1, False, False), (10, 40, False, False),
                                                 (4, 4, True, False), (2, 5, False, True), (5, 3, False, False)])
def test_chunks_equal_oracle_prefixes(cuda, m, c, per_proc, mascot, policy):
    from paper_1811_09136_amd import rept
    e = synth.er(300, 3000, 7 + m, 8 + c)
    p = rept.Params(m, c, 40 + m * c, per_proc, mascot)
    _say(f"stream ER n=300 E=3000 m={m} c={c} per_proc={per_proc} mascot={mascot} policy={policy}")
    inc = rept.IncrementalStream(300, 3000, 1200, p, cuda, policy=policy)
    cuts = [0, 1, 8, 9, 1000, 1700, 2900, 3000]
    for a, b in zip(cuts[:-1], cuts[1:]):
        inc.append(rept.to_device_edges(e[a:b], cuda))
        _check(inc, e[:b], 300, p)
    _paths_follow(inc, policy, len(cuts) - 1)
    inc.close()


@pytest.mark.parametrize("policy", ["auto", "per_edge", "recount"])
def test_hub_stream_and_estimates(cuda, policy):
    """A power-law stream with hub lists in uneven chunks; the estimates after each chunk
    equal the oracle's estimates of the prefix (0 ulp)."""
    from paper_1811_09136_amd import rept
    e, n = synth.scaled_chung_lu(200_000, 19)
    p = rept.Params(10, 40, 3)
    _say(f"stream Chung-Lu n={n} E={len(e)} m=10 c=40 policy={policy}")
    inc = rept.IncrementalStream(n, len(e), 90_000, p, cuda, policy=policy)
    for a, b in [(0, 50_000), (50_000, 50_001), (50_001, 140_000), (140_000, 200_000)]:
        inc.append(rept.to_device_edges(e[a:b], cuda))
        og, ol = oracle.rept(e[:b], n, 10, 40, 3)
        th, tv = inc.estimate()
        oth, otv = oracle.estimate(n, 10, 40, og, ol)
        assert th == oth and np.array_equal(tv.view(np.uint64), otv.view(np.uint64))
    _paths_follow(inc, policy, 4)
    inc.close()


def test_equals_count_on_the_whole_stream(cuda):
    """The final counters equal rept_count on the stream built at once."""
    import torch
    from paper_1811_09136_amd import rept
    e, n = synth.scaled_chung_lu(300_000, 23)
    p = rept.Params(10, 15, 8)
    _say(f"stream vs rept_count Chung-Lu n={n} E={len(e)} m=10 c=15")
    inc = rept.IncrementalStream(n, len(e), 100_000, p, cuda, policy="recount")
    for a in range(0, len(e), 100_000):
        inc.append(rept.to_device_edges(e[a:a + 100_000], cuda))
    g = rept.Graph(rept.to_device_edges(e, cuda), n)
    glob, loc = g.count(p)
    torch.cuda.synchronize()
    assert torch.equal(inc.counts[0], glob) and torch.equal(inc.counts[1], loc)
    _paths_follow(inc, "recount", 3)
    g.close()
    inc.close()


def test_invalid_chunks_leave_state_unchanged(cuda):
    from paper_1811_09136_amd import rept
    e = synth.er(100, 800, 3, 4)
    p = rept.Params(2, 3, 5)
    _say("stream invalid chunks")
    inc = rept.IncrementalStream(100, 750, 400, p, cuda)
    inc.append(rept.to_device_edges(e[:300], cuda))
    bad = [(np.array([[5, 5]], np.uint32), rept.REPT_ESELFLOOP),
           (np.array([[1, 100]], np.uint32), rept.REPT_ERANGE),
           (np.vstack([e[300:310], e[300:301][:, ::-1]]).astype(np.uint32), rept.REPT_EDUP),  # twice in a chunk
           (np.vstack([e[300:305], e[10:11]]).astype(np.uint32), rept.REPT_EDUP),  # already appended
           (np.vstack([e[300:305], [[7, 7]], [[1, 1000]]]).astype(np.uint32), rept.REPT_ERANGE),
           (e[300:701], rept.REPT_ENOMEM)]  # longer than max_chunk
    for chunk, code in bad:
        with pytest.raises(rept.ReptError) as ei:
            inc.append(rept.to_device_edges(chunk, cuda))
        assert ei.value.code == code
        _check(inc, e[:300], 100, p)
    inc.append(rept.to_device_edges(e[300:700], cuda))
    _check(inc, e[:700], 100, p)
    with pytest.raises(rept.ReptError) as ei:
        inc.append(rept.to_device_edges(e[700:800], cuda))  # 800 edges > capacity 750
    assert ei.value.code == rept.REPT_ENOMEM
    _check(inc, e[:700], 100, p)
    inc.append(rept.to_device_edges(e[700:750], cuda))
    _check(inc, e[:750], 100, p)
    inc.append(rept.to_device_edges(e[750:750], cuda))  # an empty chunk changes nothing
    _check(inc, e[:750], 100, p)
    inc.close()


@pytest.mark.parametrize("n,head,chunks", [
    (300, 8192, [1, 31, 32, 33, 64, 2047]),      # the pairwise sort: a workgroup's 32 edges, less and more
    (300, 8193, [8192, 8193, 4096, 1]),          # the largest pairwise sort, the smallest radix sort
    (4096, 8193, [10240, 10239, 12289]),         # 12-bit ids (three digits); tiles of 2,048 edges
    (70000, 30001, [9000, 8192]),                # 17-bit ids (four digits), more nodes than edges
    ((1 << 22) + 1, 8193, [20000]),              # 23-bit ids (six digits)
])
def test_chunk_sort_sizes(cuda, n, head, chunks):
    """Chunks at the edges of the sorts' sizes; after each, a repeat of one of its pairs (reversed) and of
    an earlier one is refused at a size of either sort."""
    from paper_1811_09136_amd import rept
    E = head + sum(chunks)
    e = synth.er(min(n, 70000), E, 5, 6)
    if n > 70000:
        e = (e * np.uint32(59)).astype(np.uint32)
    p = rept.Params(2, 5, 11)
    inc = rept.IncrementalStream(n, E + 10000, 20000 if head < 20000 else head, p, cuda, policy="per_edge")
    at = 0
    for w in [head] + chunks:
        _say(f"chunk sort n={n} at={at} W={w}")
        inc.append(rept.to_device_edges(e[at:at + w], cuda))
        at += w
        for k in (2, 8194):
            for pair in (e[at - 1], e[0][::-1]):
                bad = np.vstack([_fresh(n, k, e), [pair]]).astype(np.uint32)
                with pytest.raises(rept.ReptError) as ei:
                    inc.append(rept.to_device_edges(bad, cuda))
                assert ei.value.code == rept.REPT_EDUP
    _check(inc, e[:at], n, p)
    inc.close()


def _fresh(n, k, e):
    """k pairs that are not in the stream e."""
    if n == 300:
        used = {(min(u, v), max(u, v)) for u, v in e.tolist()}
        out = [(u, v) for u in range(n) for v in range(u + 1, n) if (u, v) not in used]
        return np.array(out[:k], np.uint32)
    used = set((np.minimum(e[:, 0], e[:, 1]).astype(np.int64) * n + np.maximum(e[:, 0], e[:, 1])).tolist())
    u = np.arange(4 * k, dtype=np.int64) % (n - 1)
    v = u + 1 + np.arange(4 * k, dtype=np.int64) // (n - 1)
    keep = np.array([x * n + y not in used and y < n for x, y in zip(u, v)])
    return np.stack([u[keep], v[keep]], 1)[:k].astype(np.uint32)


@pytest.mark.parametrize("name", ["sparse", "clique", "hubs"])
@pytest.mark.parametrize("m,c,per_proc", [(1, 1, False), (2, 16, False), (3, 7, True), (1300, 1100, False)])
def test_per_edge_count_shapes(cuda, name, m, c, per_proc):
    """The per-edge count where its stages change: runs with more entries than are staged (a sparse
    stream), queues that fill in every step (a clique), many large nodes (the table of additions), and
    more processors than the LDS histogram holds; per chunk against the oracle."""
    from paper_1811_09136_amd import rept
    if name == "sparse":
        n, e = 30000, synth.er(30000, 24000, 3, 4)
    elif name == "clique":
        n, e = 150, synth.shuffled(synth.complete(150), 3, flip_seed=4).astype(np.uint32)
    else:
        n = 3300
        y = 300 + np.arange(3000, dtype=np.uint32)
        e = np.concatenate([np.stack([y, (y * 7 + k * 11) % 300], 1) for k in range(5)] +
                           [np.stack([np.arange(300), (np.arange(300) + k) % 300], 1) for k in range(1, 40)])
        e = synth.shuffled(e.astype(np.uint32), 5, flip_seed=6)
    p = rept.Params(m, c, 21, per_proc)
    inc = rept.IncrementalStream(n, len(e), len(e), p, cuda, policy="per_edge")
    cuts = [0, len(e) // 3, len(e) // 3 + 1, len(e) // 2, len(e)]
    for a, b in zip(cuts[:-1], cuts[1:]):
        _say(f"per-edge {name} m={m} c={c} per_proc={per_proc} [{a}, {b})")
        inc.append(rept.to_device_edges(np.ascontiguousarray(e[a:b]), cuda))
        _check(inc, e[:b], n, p)
    inc.close()
