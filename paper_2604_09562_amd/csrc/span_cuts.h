// Where the flat sequence of KV tile pairs is cut into the spans of the streaming attention kernel.
//
// The pairs of all (request, KV head) units lie end to end, unit major: request b contributes hkv units of
// n_b pairs each.  Spans are equal in a "weighted" coordinate in which every unit is preceded by `weight`
// virtual pairs (what opening a unit costs a wavefront): unit u = b * hkv + g occupies the stretch
// [ya, ya + weight + n_b), ya = (flat index of its first pair) + weight * u, and wave w starts at the cut
// w * total_w / nw.  A cut inside a unit's virtual part starts the span at the unit's first pair.  The plan
// kernel (which writes the spans) and the merge kernel (which has to know which waves hold a part of a unit)
// both use the functions below; plain integer code with no device dependency, so that a host test can check
// them against each other over many shapes.
#pragma once

#include <stdint.h>

#ifndef SS_HOST_DEVICE
#define SS_HOST_DEVICE __host__ __device__
#endif

namespace ss {

// How many spans, and whether the spans of a workgroup are combined in LDS (`can_chain`: the instance is able to).
//
// A call that does not fill the chip is bound by latency: spans of two pairs, and every wavefront leaves its partial at once
// (the hand-over is a chain of up to four unit ends, 1.2 us each, 3.8 us for the output), as the merge kernel runs anyway: 4 requests
// of 40..600 tokens over 8 KV heads 16.4 -> 11.4 us in the streaming kernel, against spans of four pairs with the hand-over.
// But the merge kernel adds a unit's partials one after the other, so that holds only while they are few.  A whole call, in us,
// with spans of two pairs / the same and the hand-over / four pairs and the hand-over (one request, 8 KV heads, depth 4):
//   1000 tokens (16 spans a unit)  20.5 / 22.2 / 23.9      2000 (31)  24.1 / 23.3 / 24.8      4000 (63)  30.8 / 25.1 / 25.9
//   8000 (125)  41.7 / 28.9 / 28.3      32000 tokens over one KV head (500)  103 / 45.6 / 36.3
// and without a hand-over (three row blocks and more), with spans of two / four pairs:
//   4 requests of 2000, 8 KV heads (31): 29.8 / 28.8 (three row blocks), 32.1 / 32.4 (four, tree)      4000 (63): 34.1 / 30.0
//   60000 tokens over one KV head, five row blocks (937): 184 / 109
// So the hand-over comes in from kMaxLooseSpans spans per unit on, the longer spans from kMaxUnitPartials partials on, both for
// the longest unit.
constexpr int kMinPairsPerSpan = 2, kMinPairsLongUnits = 4;
constexpr int kMaxLooseSpans = 16, kMaxUnitPartials = 32;
constexpr int kSpansPerWg = 4;   // wavefronts of a workgroup

struct SpanCount {
    long long spans;
    int chain;
};
// total: pairs of all units (>= 1); longest: pairs of the longest unit; launch_waves: the most spans there can be.
SS_HOST_DEVICE inline SpanCount count_spans(long long total, int longest, long long launch_waves, bool can_chain)
{
    auto bounded = [&](long long n) { return n < 1 ? 1 : n > launch_waves ? launch_waves : n; };
    SpanCount c;
    c.spans = bounded(total / kMinPairsPerSpan);
    const long long of_longest = longest * c.spans;   // spans of the longest unit, times total
    c.chain = can_chain && (c.spans == launch_waves || of_longest > kMaxLooseSpans * total);
    if (of_longest > (c.chain ? kSpansPerWg : 1) * kMaxUnitPartials * total) c.spans = bounded(total / kMinPairsLongUnits);
    return c;
}

struct SpanCuts {
    const int32_t *prefix;   // [batch + 1] exclusive prefix of the pairs per KV head of the requests
    int batch, hkv, weight;
    long long total;         // pairs of all units
    long long total_w;       // pairs of all units plus `weight` per unit
    long long nw;            // number of spans

    SS_HOST_DEVICE static SpanCuts make(const int32_t *prefix, int batch, int hkv, int weight, long long nw)
    {
        SpanCuts c;
        c.prefix = prefix;
        c.batch = batch;
        c.hkv = hkv;
        c.weight = weight;
        c.total = (long long)prefix[batch] * hkv;
        c.total_w = c.total + (long long)weight * batch * hkv;
        c.nw = nw;
        return c;
    }
    // weighted coordinate of wave w's cut
    SS_HOST_DEVICE long long cut(long long w) const { return w * total_w / nw; }
    // flat index of unit (b, g)'s first pair, and the weighted coordinate where its stretch begins
    SS_HOST_DEVICE long long unit_offset(int b, int g) const
    {
        return (long long)prefix[b] * hkv + (long long)g * (prefix[b + 1] - prefix[b]);
    }
    SS_HOST_DEVICE long long unit_coord(int b, int g) const { return unit_offset(b, g) + (long long)weight * ((long long)b * hkv + g); }
    // the waves whose cut falls into the stretch [ya, ya + weight + n): w_lo <= w < w_hi (w_hi may exceed nw)
    SS_HOST_DEVICE long long first_cut_at_or_after(long long y) const { return (y * nw + total_w - 1) / total_w; }
    // pair of the unit at which a span begins whose cut lies `ya <= cut < ya + weight + n`
    SS_HOST_DEVICE int first_pair(long long cut_y, long long ya) const
    {
        const long long in_unit = cut_y - ya - weight;
        return in_unit > 0 ? (int)in_unit : 0;
    }
    // unit and pair that weighted coordinate y (< total_w) falls on; returns the flat pair index
    SS_HOST_DEVICE long long locate(long long y, int &b, int &g, int &pair) const
    {
        int lo = 0, hi = batch - 1;   // last request whose first unit starts at or before y
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (((long long)prefix[mid] + (long long)weight * mid) * hkv <= y)
                lo = mid;
            else
                hi = mid - 1;
        }
        b = lo;
        const int n = prefix[b + 1] - prefix[b];
        const long long r = y - ((long long)prefix[b] + (long long)weight * b) * hkv;
        g = (int)(r / (n + weight));
        const int in_unit = (int)(r - (long long)g * (n + weight)) - weight;
        pair = in_unit > 0 ? in_unit : 0;
        return (long long)prefix[b] * hkv + (long long)g * n + pair;
    }
    // flat index one past wave w's last pair
    SS_HOST_DEVICE long long span_end(long long w) const
    {
        if (w + 1 >= nw) return total;
        if (weight == 0) return (w + 1) * total / nw;
        int b, g, t;
        return locate(cut(w + 1), b, g, t);
    }
    // The waves that hold pairs of a unit with n >= 1 pairs whose stretch begins at ya: the last wave whose cut
    // lies at or before the unit's first pair ... the last wave whose cut lies at or before its last pair.
    SS_HOST_DEVICE void unit_waves(long long ya, int n, int &w_first, int &w_last) const
    {
        w_first = (int)(((ya + weight + 1) * nw - 1) / total_w);
        w_last = (int)(((ya + weight + n) * nw - 1) / total_w);
    }
};

}  // namespace ss
