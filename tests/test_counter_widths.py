"""The partial counters of 16 bits (and the sums of 32) on the device path hold what their flushes let
them gain; the bounds are read from the kernel sources (the 32-bit histograms' are in
test_counter_bounds.py):

* a staged entry's local counter (16 bits per group) and its pair counts (s and L, 16 bits each of one
  word) gain at most one per list walked against the entry.  A unit's lists are walked in rounds of
  kRoundLists, the counters flushed after each; units counted together by a wavefront have at most
  8 wave_cap + 7 reverse lists and wave_cap own ones (their order key is at most wave_cap);
* a walked list's counters gain at most one per entry of the table chunk (at most 4096 entries) and are
  flushed with the chunk of lists;
* the incremental count stages item ends as 16 bits from the run's start on, kRun standing for any end
  past the run;
* its table of additions (32-bit sums) is flushed with its histogram, before the items since the last
  flush pass 2^31; an item adds at most one to any counter.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_09136_amd", "csrc")


def _src(name):
    with open(os.path.join(CSRC, name)) as f:
        return f.read()


def _const(src, name):
    m = re.search(r"\b" + name + r" = ([^;,]+)[;,]", src)
    assert m, name
    return eval(m.group(1).replace("u", ""))


def test_rounds_of_lists_fit_16_bits():
    s = _src("count.hip")
    rounds = _const(s, "kRoundLists")
    assert rounds < 2**16
    # the rounds: the W entries' pair counts and local counts are flushed and cleared after each
    assert "lists - es > kRoundLists ? es + kRoundLists : lists" in s
    body = s[s.index("lists - es > kRoundLists"):s.index("es = ee;")]
    assert "T.ewe[g * T.DW + i] = 0;" in body and "T.cntw[J.gp * i + g] = 0;" in body
    assert "1u << (16u * (i & 1u))" in s  # two counters to a word: a carry would reach the neighbour


def test_units_counted_together_fit_16_bits():
    a, c = _src("api.hip"), _src("common.h")
    shift = int(re.search(r"#define REPT_REV_SHIFT (\d+)", c).group(1))
    cap = int(re.search(r"wave_cap < 8 \|\| wave_cap > (\d+)\) return REPT_EINVAL", a).group(1))
    assert ((cap + 1) << shift) - 1 + cap < 2**16


def test_walked_lists_fit_16_bits():
    a, s = _src("api.hip"), _src("count.hip")
    cap = int(re.search(r"block_cap < 64 \|\| block_cap > (\d+)\) return REPT_EINVAL", a).group(1))
    assert cap < 2**16
    assert cap + 1 < 2**_const(s, "kTagShift")  # a table slot's index field holds i + 1
    assert "flush_pair(J, g, pab, v);" in s


def test_incremental_ends_and_sums():
    s = _src("stream.hip")
    run = _const(s, "kRun")
    assert run < 2**16 and "(uint16_t)(e < kRun ? e : kRun)" in s
    assert "if (run > kRun) run = kRun;" in s
    flush = s[s.index("const auto flush = [&] {"):s.index("uint64_t since = 0;")]
    assert "sums.sum[i] = 0u;" in flush and "hist[i] = 0u;" in flush
    assert "if (since + (i1 - i0) > (1ull << 31)) {" in s and 2**31 + run < 2**32
