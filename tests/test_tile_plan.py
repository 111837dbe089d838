"""How a counting launch cuts its units into tiles (plan_tiles in api.hip) and how the kernel reads a
tile back (tile_part and light_tile_of in count.hip), compiled for the host as they stand: over graphs,
launch shapes and grids up to the largest that a caller can ask for, every unit is counted whole and
exactly once."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_09136_amd", "csrc")

HARNESS = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <map>
#include <vector>
#include "common.h"
//PLAN
#undef __device__
#define __device__
//READ
// a graph of `units` units with keys spread over [2, top], descending, as the build counts them
static rept_graph graph_of_keys(const std::vector<uint32_t>& keys, uint64_t E, uint32_t num_rev) {
    rept_graph g;
    memset(&g, 0, sizeof(g));
    g.E = E;
    g.num_rev = num_rev;
    g.num_apex = (uint32_t)keys.size();
    for (uint32_t i = 0; i < kKeyTab; ++i)
        for (uint32_t k : keys) g.above[i] += k > key_threshold(i);
    return g;
}
int main(int argc, char** argv) {
    const uint32_t units = atoi(argv[1]), top = atoi(argv[2]), lists = atoi(argv[3]), jobs_n = atoi(argv[4]);
    const uint32_t wave_cap = atoi(argv[5]), threads = atoi(argv[6]), light_tile = atoi(argv[7]), split = atoi(argv[8]);
    const uint32_t own_blocks = strtoul(argv[9], nullptr, 10);
    std::vector<uint32_t> keys(units);
    for (uint32_t i = 0; i < units; ++i) keys[i] = 2 + (uint32_t)((uint64_t)(top - 2) * (units - 1 - i) / units);
    const rept_graph g = graph_of_keys(keys, lists, lists / 2);
    BatchHeader h;
    memset(&h, 0, sizeof(h));
    h.njobs = jobs_n;
    h.wave_cap = wave_cap;
    h.threads = threads;
    h.light_tile = light_tile;
    h.split = split;
    h.blocks = own_blocks ? own_blocks : 1024;
    h.light_blocks = own_blocks ? own_blocks : 1280;
    rept_tuning tu;
    memset(&tu, 0, sizeof(tu));
    tu.blocks = own_blocks;
    std::vector<JobDev> jobs(jobs_n);
    for (uint32_t j = 0; j < jobs_n; ++j) {  // the jobs are consecutive ranges of the graph's units
        memset((void*)&jobs[j], 0, sizeof(JobDev));
        jobs[j].unit0 = (uint64_t)units * j / jobs_n;
        jobs[j].unit1 = (uint64_t)units * (j + 1) / jobs_n;
    }
    plan_tiles(&h, jobs.data(), [&](uint32_t) { return &g; }, &tu);
    // every unit's parts: as many as its tiles say, each once
    std::vector<std::map<uint32_t, uint32_t>> seen(units);
    std::vector<uint32_t> parts(units, 0);
    auto job_of = [&](uint32_t t, bool heavy) {
        uint32_t j = jobs_n - 1;
        while (j && (heavy ? jobs[j].heavy_prefix : jobs[j].light_prefix) > t) --j;
        return j;
    };
    uint32_t most = 0;
    for (uint32_t t = 0; t < h.heavy_total; ++t) {
        const JobDev& J = jobs[job_of(t, true)];
        uint32_t first, unit, part;
        const uint32_t k = tile_part(J.hcls, kHeavyClasses, t - J.heavy_prefix, first, unit, part);
        const uint32_t u = J.unit0 + first + unit;
        if (u >= J.unit1 || keys[u] <= wave_cap) return printf("heavy tile %u: unit %u\n", t, u), 1;
        ++seen[u][part];
        parts[u] = 1u << k;
        most = std::max(most, 1u << k);
    }
    uint32_t widest = 0;
    for (uint32_t t = 0; t < h.light_total; ++t) {
        const JobDev& J = jobs[job_of(t, false)];
        uint32_t first, count, part;
        const uint32_t k = light_tile_of(J.lcls, t - J.light_prefix, first, count, part);
        if (!count || (k && count != 1)) return printf("light tile %u: %u units\n", t, count), 1;
        for (uint32_t i = 0; i < count; ++i) {
            const uint32_t u = J.unit0 + J.hcls[0] + first + i;
            if (u >= J.unit1 || keys[u] > wave_cap) return printf("light tile %u: unit %u\n", t, u), 1;
            ++seen[u][part];
            parts[u] = 1u << k;
        }
        widest = std::max(widest, count);
    }
    for (uint32_t u = 0; u < units; ++u)
        if (seen[u].size() != parts[u] || seen[u].rbegin()->first != parts[u] - 1 ||
            std::any_of(seen[u].begin(), seen[u].end(), [](auto& x) { return x.second != 1; }))
            return printf("unit %u (key %u): %zu parts of %u\n", u, keys[u], seen[u].size(), parts[u]), 1;
    if (widest > light_tile) return printf("%u units in a tile\n", widest), 1;
    printf("%u %u %u\n", h.heavy_total, h.light_total, most);
    return 0;
}
"""


def _text(name, first, last):
    """The source from the line that starts with `first` to the end of the function `last`."""
    with open(os.path.join(CSRC, name)) as f:
        src = f.read()
    a = src.index("\n" + first) + 1
    b = re.search(r"\n[^\n/]*\b" + last + r"\(", src[a:]).start() + a
    return src[a:src.index("\n}\n", b) + 3]


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    code = HARNESS.replace("//PLAN", _text("api.hip", "// Units of `g` whose order key", "plan_tiles"))
    code = code.replace("//READ", _text("count.hip", "// Unit and part of tile t", "light_tile_of"))
    (d / "plan.cpp").write_text(code)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{CSRC}", f"-I{ROOT}/include",
                    f"-I{rocm}/include", "-o", str(d / "plan"), str(d / "plan.cpp")], check=True)

    def run(*args):
        r = subprocess.run([str(d / "plan")] + [str(a) for a in args], capture_output=True, text=True)
        assert r.returncode == 0, (r.returncode, r.stdout)
        return tuple(int(x) for x in r.stdout.split())
    return run


@pytest.mark.parametrize("units,top,lists", [(1, 3, 3), (7, 9, 40), (1000, 60, 20_000), (5000, 700, 300_000),
                                             (20_000, 3000, 4_000_000), (300, 600_000, 2_000_000_000)])
@pytest.mark.parametrize("jobs", [1, 3, 64])
def test_every_unit_once(planner, units, top, lists, jobs):
    for wave_cap, threads, light_tile, split in [(64, 256, 8, 1), (256, 1024, 16, 1), (64, 256, 8, 0), (8, 64, 1, 1),
                                                 (200, 512, 64, 0)]:
        for blocks in (0, 1, 3):
            planner(units, top, lists, jobs, wave_cap, threads, light_tile, split, blocks)


@pytest.mark.parametrize("blocks", [1 << 24, 1 << 28, 1 << 29, 1 << 30, (1 << 30) + 1, 1 << 31, (1 << 32) - 1])
def test_any_grid_the_caller_asks_for(planner, blocks):
    """A grid of 2^30 workgroups has 2^32 wavefronts of the light phase: the plan is made (the launch is
    refused), and is as fine as one for the largest grid that can be launched."""
    finest = planner(5000, 700, 300_000, 1, 64, 256, 8, 1, (1 << 24) - 1)
    assert planner(5000, 700, 300_000, 1, 64, 256, 8, 1, blocks) == finest
    planner(5000, 700, 300_000, 2, 64, 1024, 8, 0, blocks)
