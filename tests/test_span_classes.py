"""Host check of the span cuts with classes (`csrc/span_cuts.h`): requests laid out by class, a pair and the opening of a unit
costing what their class says.  The spans have to tile the flat sequence, and the spans that hold pairs of a unit have to be the
ones the merge kernel's formula names."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HEADER_DIR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_09562_amd", "csrc")

SHIM = r"""
#define SS_HOST_DEVICE
#include "span_cuts.h"
using namespace ss;
// out[w] = {unit, first pair, x0, x1} of every span, as the plan kernel finds them unit by unit; first/last: the merge's formula
extern "C" long long spans(const int32_t *n, const int32_t *cls, int batch, int hkv, const int32_t *cost, const int32_t *weight, long long nw,
                           int32_t *prefix, long long *cprefix, long long *out, int *count, int *first, int *last)
{
    SpanClasses k5;
    k5.cost = k5.weight = 0;
    prefix[0] = 0;
    cprefix[0] = 0;
    for (int i = 0; i < batch; ++i) {
        prefix[i + 1] = prefix[i] + n[i];
        cprefix[i + 1] = cprefix[i] + (long long)n[i] * cost[cls[i]] + weight[cls[i]];
    }
    for (int k = 0; k < kMaxClasses; ++k) {
        k5.end[k] = 0;
        for (int i = 0; i < batch; ++i) k5.end[k] += cls[i] <= k;
        k5.x[k] = prefix[k5.end[k]];
        k5.cost |= (uint64_t)cost[k] << (8 * k);
        k5.weight |= (uint64_t)weight[k] << (12 * k);
    }
    if (k5.total() != cprefix[batch]) return -1;
    const SpanCuts c = {k5.total() * hkv, nw};
    for (int p = 0; p < batch; ++p) {
        const int co = k5.cost_of(cls[p]), we = k5.weight_of(cls[p]);
        if (k5.of(p) != cls[p] || co != cost[cls[p]] || we != weight[cls[p]] || k5.start(p, prefix[p], cls[p]) != cprefix[p]) return -1;
        for (int g = 0; g < hkv; ++g) {
            const long long off = (long long)prefix[p] * hkv + (long long)g * n[p], stretch = we + (long long)n[p] * co,
                            ya = k5.start(p, prefix[p], cls[p]) * hkv + g * stretch;
            for (long long w = c.first_cut_at_or_after(ya); w < c.first_cut_at_or_after(ya + stretch) && w < nw; ++w) {
                const int t0 = SpanCuts::first_pair(c.cut(w), ya, we, co);
                out[4 * w] = (long long)p * hkv + g;
                out[4 * w + 1] = t0;
                out[4 * w + 2] = off + t0;
                if (w) out[4 * w - 1] = off + t0;   // a span ends where the next one starts
                ++count[w];
            }
            c.unit_spans(ya, n[p], we, co, first[p * hkv + g], last[p * hkv + g]);
        }
    }
    out[4 * nw - 1] = (long long)prefix[batch] * hkv;
    return (long long)prefix[batch] * hkv;
}
extern "C" long long team_spans(long long total, int longest, long long most) { return count_team_spans(total, longest, most); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("span_classes")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", HEADER_DIR, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.spans.restype = lib.team_spans.restype = ctypes.c_longlong
    return lib


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


@pytest.mark.parametrize("seed", range(6))
def test_spans_by_class(shim, seed):
    rng = np.random.default_rng(seed)
    for _ in range(60):
        batch, hkv = int(rng.integers(1, 50)), int(rng.choice([1, 2, 8]))
        cls = np.sort(rng.integers(0, 5, batch)).astype(np.int32)
        n = (np.exp(rng.uniform(0, np.log(rng.choice([4, 60, 700])), batch)).astype(np.int32) + 1).astype(np.int32)
        kind = rng.integers(0, 3)
        if kind == 0:   # whole units
            cost, weight = np.zeros(5, np.int32), np.ones(5, np.int32)
        elif kind == 1:
            cost, weight = np.array([10, 9, 9, 8, 8], np.int32), np.array([280, 220, 160, 96, 64], np.int32)
        else:
            cost, weight = rng.integers(1, 17, 5).astype(np.int32), rng.integers(0, 1025, 5).astype(np.int32)
        total = int(n.sum()) * hkv
        nw = int(min(rng.choice([1, 3, 16, 256]), max(1, total // 2))) if kind else batch * hkv
        out, count = np.full((nw, 4), -1, np.int64), np.zeros(nw, np.int32)
        first, last = np.zeros(batch * hkv, np.int32), np.zeros(batch * hkv, np.int32)
        prefix, cprefix = np.zeros(batch + 1, np.int32), np.zeros(batch + 1, np.int64)
        assert shim.spans(_p(n), _p(cls), batch, hkv, _p(cost), _p(weight), ctypes.c_longlong(nw), _p(prefix), _p(cprefix), _p(out),
                          _p(count), _p(first), _p(last)) == total
        assert np.all(count == 1) and np.all(out[:, 1] >= 0)
        x0, x1 = out[:, 2], out[:, 3]
        assert x0[0] == 0 and x1[-1] == total and np.all(x1[:-1] == x0[1:]) and np.all(x1 >= x0)
        off = np.concatenate([[0], np.cumsum(np.repeat(n, hkv))])
        for u in range(batch * hkv):
            holders = [w for w in range(nw) if max(x0[w], off[u]) < min(x1[w], off[u + 1])]
            if kind:
                assert holders == list(range(first[u], last[u] + 1)), (u, holders, first[u], last[u])
            else:   # the merge has to see that every unit lies in one span, which is its own
                assert holders == [u] and first[u] == last[u], (u, holders)


def test_team_spans(shim):
    for total, longest, want in [(1, 1, 1), (8, 8, 4), (64, 64, 32), (66, 66, 4), (700, 4, 256), (625, 625, 39), (100000, 400, 256), (8000, 8000, 256)]:
        assert shim.team_spans(ctypes.c_longlong(total), longest, ctypes.c_longlong(256)) == want, (total, longest)
