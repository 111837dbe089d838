"""When a wavefront of the counting kernel flushes its LDS histogram of global counts, on the CPU: the
kernel's own rule (drain_hits and flush_hist_now, as they stand in count.hip) is compiled for the host
with one lane and a drain that counts nothing.

A launch of more processors than the histogram holds (c > 1024) has none: its counts go to memory one
by one, and the words behind the wavefront's empty histogram belong to others.  They must be neither
read nor cleared, however many candidates the wavefront has drained."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <stdint.h>
#include <stdio.h>
#include <initializer_list>
#include <type_traits>
#define __device__
#define __forceinline__ inline
struct JobDev { uint32_t c; int64_t* global; };
struct JobRegs { const JobDev* jd; uint32_t use_hist; };
struct TeamView {};
struct WaveView { uint32_t* hist; uint32_t hits; };
template <uint32_t GS> struct HitBatch { uint32_t n; };
static uint32_t lane_id() { return 0; }
static void wave_sync() {}
static void add64(int64_t* p, uint64_t v) { *p += (int64_t)v; }
template <bool ETA, bool PACK, uint32_t GS>
void drain_batch(const JobRegs&, const TeamView&, WaveView&, uint32_t, uint32_t, HitBatch<GS>&) {}
//RULE
int main() {
    static uint32_t lds[4096];
    static int64_t global[4096];
    for (uint32_t use : {0u, 1u}) {
        for (uint32_t c : {1000u, 4000u}) {
            if (use && c > 1024) continue;
            for (uint32_t before :
                {0u, kHistFlushHits - 65u, kHistFlushHits - 64u, kHistFlushHits - 1u, kHistFlushHits}) {
                for (auto& x : lds) x = 7;
                for (auto& x : global) x = 0;
                JobDev jd{c, global};
                JobRegs J{&jd, use};
                WaveView V{lds, before};
                HitBatch<1> D{64};
                drain_hits<false, true, 1>(J, TeamView(), V, 0u, 0u, D, std::integral_constant<bool, true>());
                uint32_t cleared = 0, added = 0;
                for (uint32_t p = 0; p < 4096; ++p) {
                    cleared += lds[p] != 7;
                    added += global[p] != 0;
                }
                printf("%u %u %u %u %u %u\n", use, c, before, cleared, added, V.hits);
            }
        }
    }
}
"""


def _function(src, name):
    """The text of a function or template, from its template line (if any) to its closing brace."""
    at = re.search(r"(template <[^\n]*>\n)?__device__ __forceinline__ void " + name + r"\(", src)
    assert at, name
    end = src.index("\n}\n", at.start()) + 3
    return src[at.start():end]


def test_flush_without_a_histogram(tmp_path):
    with open(os.path.join(ROOT, "paper_1811_09136_amd", "csrc", "count.hip")) as f:
        src = f.read()
    limit = re.search(r"constexpr uint32_t kHistFlushHits = [^;]+;", src).group(0)
    rule = "\n".join([_function(src, "flush_hist_now"), limit, _function(src, "drain_hits")])
    (tmp_path / "rule.cpp").write_text(HARNESS.replace("//RULE", rule))
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "rule"), str(tmp_path / "rule.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "rule")], check=True, capture_output=True, text=True).stdout
    rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    assert len(rows) == 15
    for use, c, before, cleared, added, hits in rows:
        due = use == 1 and before + 64 >= 1 << 31
        words = -(-c // 64) if due else 0  # lane 0's share of the c counters
        assert (cleared, added) == (words, words), (use, c, before)
        if use:
            assert hits == (0 if due else before + 64)
