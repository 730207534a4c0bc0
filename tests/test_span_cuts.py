"""Host check of the span-cut arithmetic shared by the plan kernel and the merge kernel of the attention path.

`csrc/span_cuts.h` depends on nothing of the device.  It is compiled here for the host; for many shapes (pair counts per
request, KV heads, span counts, unit weights) the spans are enumerated the way the plan kernel writes them
(for every unit, the waves whose cut falls into the unit's stretch) and checked against what the streaming
and merge kernels rely on:
  * the spans (each ends where the next one starts) tile the flat sequence: in order, nothing lost, nothing twice;
  * every wave gets its descriptor from exactly one unit, and its span begins inside that unit;
  * the waves that hold pairs of a unit are exactly w_first .. w_last of the merge kernel's formula, so the
    partial slots it reads are the ones that were written (also after the division by four that applies where
    wavefronts hand over inside their workgroup);
  * slot `wave + unit` (and `workgroup + unit`) is unique along the sequence.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER_DIR = os.path.join(ROOT, "paper_2604_09562_amd", "csrc")

SHIM = r"""
#define SS_HOST_DEVICE
#include "span_cuts.h"
using ss::SpanCuts;
using ss::SpanClasses;
// One class, a pair costing one: the layout, and where unit (b, g)'s stretch begins.
static SpanClasses one_class(const int32_t *prefix, int batch, int weight)
{
    SpanClasses c;
    c.cost = 1;
    c.weight = weight;
    for (int k = 0; k < ss::kMaxClasses; ++k) c.end[k] = batch, c.x[k] = prefix[batch];
    return c;
}
static long long unit_start(const SpanClasses &c, const int32_t *prefix, int b, int g, int hkv)
{
    return c.start(b, prefix[b], 0) * hkv + (long long)g * (c.weight_of(0) + prefix[b + 1] - prefix[b]);
}
// For every unit (b, g) in order: the waves the plan kernel would describe from it, with their first pair and
// span (x0, x1).  out[w] = {unit, t0, x0, x1}; count[w] = how many units claimed wave w.
extern "C" void plan_spans(const int32_t *prefix, int batch, int hkv, int weight, long long nw, long long *out, int *count)
{
    const SpanClasses classes = one_class(prefix, batch, weight);
    const SpanCuts c = {classes.total() * hkv, nw};
    for (int b = 0; b < batch; ++b)
        for (int g = 0; g < hkv; ++g) {
            const int n = prefix[b + 1] - prefix[b];
            const long long off = (long long)prefix[b] * hkv + (long long)g * n, ya = unit_start(classes, prefix, b, g, hkv);
            const long long w_lo = c.first_cut_at_or_after(ya), w_hi = c.first_cut_at_or_after(ya + weight + n);
            for (long long w = w_lo; w < w_hi && w < nw; ++w) {
                const int t0 = SpanCuts::first_pair(c.cut(w), ya, weight, 1);
                out[4 * w + 0] = (long long)b * hkv + g;
                out[4 * w + 1] = t0;
                out[4 * w + 2] = off + t0;
                if (w) out[4 * w - 1] = off + t0;   // a span ends where the next one starts
                ++count[w];
            }
        }
    out[4 * nw - 1] = (long long)prefix[batch] * hkv;
}
extern "C" long long choose_spans(long long total, int longest, long long units, long long waves, int classes, int kv8, int *mode, int *whole)
{
    const ss::SpanChoice c = ss::choose_spans(total, longest, units, waves, classes != 0, kv8 != 0);
    *mode = c.mode;
    *whole = c.whole;
    return c.spans;
}
extern "C" void quotients(const long long *a, const long long *b, int n, long long *out)
{
    for (int i = 0; i < n; ++i) out[i] = ss::quotient(a[i], b[i]);
}
extern "C" void merge_waves(const int32_t *prefix, int batch, int hkv, int weight, long long nw, int *first, int *last)
{
    const SpanClasses classes = one_class(prefix, batch, weight);
    const SpanCuts c = {classes.total() * hkv, nw};
    for (int b = 0; b < batch; ++b)
        for (int g = 0; g < hkv; ++g)
            c.unit_spans(unit_start(classes, prefix, b, g, hkv), prefix[b + 1] - prefix[b], weight, 1, first[b * hkv + g], last[b * hkv + g]);
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("span_cuts")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", HEADER_DIR, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def _check(shim, pairs, hkv, weight, nw):
    batch = len(pairs)
    prefix = np.concatenate([[0], np.cumsum(pairs)]).astype(np.int32)
    total = int(prefix[-1]) * hkv
    out = np.full((nw, 4), -1, np.int64)
    count = np.zeros(nw, np.int32)
    p = prefix.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    shim.plan_spans(p, batch, hkv, weight, ctypes.c_longlong(nw), out.ctypes.data_as(ctypes.POINTER(ctypes.c_longlong)),
                    count.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
    label = (list(map(int, pairs)), hkv, weight, nw)
    assert np.all(count == 1), label                       # every wave is described exactly once
    x0, x1 = out[:, 2], out[:, 3]
    assert x0[0] == 0 and x1[-1] == total, label
    assert np.all(x1[:-1] == x0[1:]), label                # contiguous, in order
    assert np.all(x1 >= x0), label
    # the span begins inside the unit that described it (or is empty and sits at that unit's start)
    unit_off = np.array([int(prefix[b]) * hkv + g * int(pairs[b]) for b in range(batch) for g in range(hkv)], np.int64)
    unit_n = np.array([int(pairs[b]) for b in range(batch) for _ in range(hkv)], np.int64)
    u = out[:, 0]
    assert np.all((x0 >= unit_off[u]) & (x0 < unit_off[u] + unit_n[u])), label
    assert np.all(out[:, 1] == x0 - unit_off[u]), label
    # which waves hold pairs of each unit, from the spans themselves
    first = np.zeros(batch * hkv, np.int32)
    last = np.zeros(batch * hkv, np.int32)
    shim.merge_waves(p, batch, hkv, weight, ctypes.c_longlong(nw), first.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)),
                     last.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)))
    slots, wg_slots = set(), set()
    for unit in range(batch * hkv):
        lo, hi = unit_off[unit], unit_off[unit] + unit_n[unit]
        holders = [w for w in range(nw) if max(x0[w], lo) < min(x1[w], hi)]
        assert holders == list(range(first[unit], last[unit] + 1)), (label, unit, holders, int(first[unit]), int(last[unit]))
        for w in holders:
            assert (w + unit) not in slots, (label, unit, w)
            slots.add(w + unit)
        for wg in sorted({w // 4 for w in holders}):
            assert (wg + unit) not in wg_slots, (label, unit, wg)
            wg_slots.add(wg + unit)
        # a unit whose holders share one workgroup is finished inside the streaming kernel: the merge kernel skips it
        assert (first[unit] // 4 == last[unit] // 4) == (len({w // 4 for w in holders}) == 1)


def test_quotient(shim):
    """Floor division at exact multiples and one to either side, up to its limits: dividend below 2^62, quotient below 2^50."""
    rng = np.random.default_rng(3)
    pairs = []
    for _ in range(20000):
        b = int(2 ** rng.uniform(0, 61.9))
        q = int(2 ** rng.uniform(0, min(50.0, 61.99 - np.log2(b)))) if b < 2 ** 61 else 1
        for a in (q * b - 1, q * b, q * b + 1, q * b + b - 1):
            if 0 <= a < 2 ** 62 and a // b < 2 ** 50:
                pairs.append((a, b))
    for b in (1, 2, 3, 2 ** 12 - 1, 2 ** 12, 2 ** 12 + 1):
        for q in (0, 1, 2 ** 50 - 1):
            pairs += [(q * b, b), (q * b + b - 1, b)]
    pairs += [(2 ** 62 - 1, 2 ** 12 + 1), (2 ** 62 - 1, 2 ** 62), (0, 1), (0, 2 ** 62)]
    a, b = (np.array(x, np.int64) for x in zip(*pairs))
    out = np.empty_like(a)
    p64 = ctypes.POINTER(ctypes.c_longlong)
    shim.quotients(a.ctypes.data_as(p64), b.ctypes.data_as(p64), len(a), out.ctypes.data_as(p64))
    assert len(a) > 50000 and np.array_equal(out, a // b)


def test_small_shapes_exhaustively(shim):
    n = 0
    for hkv in (1, 2):
        for weight in (0, 1, 2, 3, 7, 8):
            for pairs in ([1], [5], [1, 1], [1, 4], [3, 1, 2], [2, 2, 2, 2], [1, 9, 1], [6, 1, 1, 1, 5]):
                total = sum(pairs) * hkv
                for nw in range(1, total + 1):          # never more spans than pairs (the plan keeps two pairs or more per wave on average)
                    _check(shim, np.array(pairs), hkv, weight, nw)
                    n += 1
    assert n > 500


def test_random_shapes(shim):
    rng = np.random.default_rng(1)
    for _ in range(300):
        batch = int(rng.integers(1, 40))
        hkv = int(rng.choice([1, 2, 4, 8]))
        kind = rng.integers(0, 3)
        if kind == 0:
            pairs = rng.integers(1, 6, batch)                       # many short units
        elif kind == 1:
            pairs = np.exp(rng.uniform(0, np.log(600), batch)).astype(np.int64) + 1   # ragged
        else:
            pairs = rng.integers(200, 1200, batch)                  # long
        total = int(pairs.sum()) * hkv
        weight = int(rng.choice([0, 1, 2, 3, 8, 17, 32]))           # 2 is the default, 32 the largest the option gives
        nw_max = max(1, total // 2)                                 # the plan kernel's bound: two pairs per span on average
        nw = int(min(nw_max, rng.choice([1, 4, 8, 64, 256, 1024])))
        nw = max(4 * (nw // 4), 1) if nw >= 4 else nw
        _check(shim, pairs, hkv, weight, nw)


def test_bench_workload_shape(shim):
    # 64 requests, contexts uniform on [256, 4096] + 5 new tokens, 8 KV heads, 1024 spans
    rng = np.random.default_rng(2)
    pairs = (rng.integers(256, 4097, 64) + 5 + 31) // 32
    for weight in (2, 8):
        _check(shim, pairs, 8, weight, 1024)


CHAIN, TEAM, ALONE = 0, 1, 2
WAVES = 1024


def choose(shim, total, longest, units, classes, kv8):
    mode, whole = ctypes.c_int(), ctypes.c_int()
    shim.choose_spans.restype = ctypes.c_longlong
    n = shim.choose_spans(ctypes.c_longlong(total), int(longest), ctypes.c_longlong(units), ctypes.c_longlong(WAVES), int(classes),
                          int(kv8), ctypes.byref(mode), ctypes.byref(whole))
    return n, mode.value, whole.value


@pytest.mark.parametrize("classes,kv8", [(False, False), (True, False), (True, True)])
def test_the_merge_adds_few_partials(shim, classes, kv8):
    """Over many shapes: there are never more spans than wavefronts (teams) or, but for whole units, than half as many as pairs; and the
    merge adds a unit's partials one after the other, so that these are at most about 32, or what the longer spans leave on a
    call of long units.  One request, a few equal ones, one long among short ones."""
    seen = set()
    for hkv in (1, 2, 8):
        for batch in (1, 2, 4, 16, 64, 128, 512):
            for n in (1, 2, 4, 5, 8, 9, 16, 17, 31, 33, 64, 125, 250, 500, 1000, 4000):
                for rest in (n, 3):
                    pairs = np.array([n] + [min(rest, n)] * (batch - 1))
                    total, units = int(pairs.sum()) * hkv, batch * hkv
                    nw, mode, whole = choose(shim, total, n, units, classes, kv8)
                    label = (hkv, batch, n, rest, nw, mode, whole)
                    seen.add((mode, whole))
                    most = WAVES if mode != TEAM else WAVES // 4
                    if whole:
                        assert mode == TEAM and nw == units <= most and n <= 16, label
                        continue
                    assert 1 <= nw <= most and (nw == 1 or total >= 2 * nw), label
                    assert mode == TEAM or mode == (ALONE if classes else CHAIN), label
                    if units < 2 * (WAVES // 4) and (classes or total < 2 * WAVES):
                        assert mode == TEAM, label                  # few units, or a chip that is not full
                    if classes and units < 2 * (WAVES // 4):
                        assert mode != ALONE, label                 # (such calls are launched without the code for it)
                    if units * nw > 100000:
                        continue   # (the check walks every unit's spans)
                    _check(shim, pairs, hkv, 2, nw)
                    prefix = np.concatenate([[0], np.cumsum(pairs)]).astype(np.int32)
                    first, last = np.zeros(units, np.int32), np.zeros(units, np.int32)
                    as_int = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
                    shim.merge_waves(as_int(prefix), batch, hkv, 2, ctypes.c_longlong(nw), as_int(first), as_int(last))
                    per = 4 if mode == CHAIN else 1
                    partials = int((last // per - first // per).max()) + 1
                    longer = max(1, min(most, total // (16 if mode == TEAM else 4)))
                    assert partials <= max(34, -(-n * longer // total) // per + 2), (label, partials)
    assert seen == ({(TEAM, 0), (TEAM, 1), (ALONE, 0)} if classes else {(TEAM, 0), (TEAM, 1), (CHAIN, 0)})


@pytest.mark.parametrize("units,mean,longest,classes,kv8,want", [
    (511, 2, 4, True, False, TEAM), (512, 2, 4, True, False, ALONE),                 # two units to a team
    (512, 13, 30, True, False, ALONE), (512, 14, 30, True, False, TEAM),             # 27 pairs per unit to a wavefront
    (1024, 27, 60, True, False, ALONE), (1024, 28, 60, True, False, TEAM), (1024, 28, 60, True, True, ALONE),
    (768, 42, 99, True, True, ALONE), (768, 43, 99, True, True, TEAM),               # 56 with e4m3 caches
    (511, 2, 4, False, False, TEAM), (512, 2, 4, False, False, CHAIN),               # one or two row blocks: many units,
    (64, 31, 40, False, False, TEAM), (64, 32, 40, False, False, CHAIN), (1, 4000, 4000, False, False, TEAM),
    (1, 4096, 4096, False, False, CHAIN)])                                           # or a full chip (spans of four pairs in a long unit)
def test_whose_the_spans_are(shim, units, mean, longest, classes, kv8, want):
    assert choose(shim, units * mean, longest, units, classes, kv8)[1] == want


@pytest.mark.parametrize("classes,few,many", [(True, 8, 16), (False, 4, 8)])
def test_whole_units(shim, classes, few, many):
    """A span per unit for units of a few pairs: of more where they are at least half as many as teams."""
    for units, longest, want in ((1, few, 1), (1, few + 1, 0), (127, few, 1), (127, few + 1, 0), (128, many, 1), (128, many + 1, 0),
                                 (256, many, 1), (257, 2, 0)):
        n, mode, whole = choose(shim, units * 2 + longest - 2, longest, units, classes, False)
        assert (mode, whole) == (TEAM, want) and (not whole or n == units), (units, longest)
