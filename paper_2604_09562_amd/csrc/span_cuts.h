// Where the flat sequence of KV tile pairs is cut into the spans of the streaming attention kernel.
//
// The pairs of all (request, KV head) units lie end to end, unit major: the request at place p of the layout contributes
// hkv units of n_p pairs each.  Spans are equal in a weighted coordinate in which every unit is preceded by
// what opening it costs, and a pair is as long as it costs: the unit occupies the stretch
// [ya, ya + weight + n * cost), and span w starts at the cut w * total_w / nw.  A cut inside the opening's part
// starts the span at the unit's first pair; a span ends where the next one starts.  The plan
// kernel (which writes the spans) and the merge kernel (which has to know which spans hold a part of a unit)
// both use the functions below; they depend on nothing of the device, so that a host test can check
// them against each other over many shapes: the same arithmetic, the division of `quotient` included.
#pragma once

#include <stdint.h>

#ifndef SS_HOST_DEVICE
#define SS_HOST_DEVICE __host__ __device__
#endif
#define SS_INLINE __attribute__((always_inline))   // (a call would put the struct into scratch memory)

namespace ss {

// How many spans, and whether the spans of a workgroup are combined in LDS (`can_chain`: the instance is able to).
//
// The spans of a call with one or two row blocks on a full chip are these, a wavefront's each, handed over in LDS.  A call that does not
// fill the chip is served by teams instead (count_team_spans); what is counted here then only says so (fewer spans than
// launched wavefronts) and stands in the plan's record.
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

// Spans of a team kernel, whose four wavefronts take a span's pairs in turn and write one partial: of two pairs as long as the chip
// is not full (then half of the wavefronts have none, but the span is over sooner), of sixteen where a unit would leave more
// than kMaxUnitPartials partials.  A whole call, in us, with a span per wavefront and no team / spans of 8 / 4 / 2 pairs:
//   24 requests of 30..200 tokens, 8 KV heads, three row blocks  24.1 / 31.9 / 26.5 / 23.7     4 of 40..600, four and five  25.7 / 28.9 / 24.6 / 23.6
//   4 of 1000..3000, e4m3  27.8 / 26.5 / 24.7 / 24.7      one of 60000 over one KV head, five row blocks  108 / 53 (spans of 16) / 74 (spans of 8)
constexpr int kMinTeamPairs = 2, kMinTeamPairsLongUnits = 16;
SS_HOST_DEVICE inline long long count_team_spans(long long total, int longest, long long most)
{
    auto bounded = [&](long long n) { return n < 1 ? 1 : n > most ? most : n; };
    const long long n = bounded(total / kMinTeamPairs);
    return longest * n > kMaxUnitPartials * total ? bounded(total / kMinTeamPairsLongUnits) : n;
}

// Requests of different row blocks in one call are laid out class by class (most row blocks first, so that a run of units
// is streamed by the code for just their row blocks), and a pair of a class costs `cost` and opening one of its units `weight`.
constexpr int kMaxClasses = 5;
struct SpanClasses {
    int end[kMaxClasses];    // requests (in layout order) of class 0, classes 0 and 1, ...: the last one is the batch
    int x[kMaxClasses];      // their pairs per KV head
    uint64_t cost, weight;   // of a pair (8 bits a class), of opening a unit (12 bits a class): packed, as arrays indexed by a
                             // variable would live in scratch memory
    SS_HOST_DEVICE SS_INLINE int of(int i) const
    {
        int c = 0;
#pragma unroll
        for (int k = 0; k + 1 < kMaxClasses; ++k) c += i >= end[k];
        return c;
    }
    SS_HOST_DEVICE SS_INLINE int cost_of(int c) const { return (int)(cost >> (8 * c)) & 0xff; }
    SS_HOST_DEVICE SS_INLINE int weight_of(int c) const { return (int)(weight >> (12 * c)) & 0xfff; }
    // What the requests in front of place p cost per KV head: p is of class c, and `pre` pairs lie in front of it.
    SS_HOST_DEVICE SS_INLINE long long start(int p, int pre, int c) const
    {
        long long y = 0;
        int first = 0, x0 = 0;   // requests and pairs in front of class c
#pragma unroll
        for (int k = 0; k + 1 < kMaxClasses; ++k) {
            if (k < c) {
                y += (long long)(x[k] - x0) * cost_of(k) + (long long)(end[k] - first) * weight_of(k);
                first = end[k];
                x0 = x[k];
            }
        }
        return y + (long long)(pre - x0) * cost_of(c) + (long long)(p - first) * weight_of(c);
    }
    SS_HOST_DEVICE SS_INLINE long long total() const { return start(end[kMaxClasses - 1], x[kMaxClasses - 1], kMaxClasses - 1); }
};

// a / b for 0 <= a < 2^62, b >= 1 and a quotient below 2^50: by a division in fp64 and one correction (the integer division is
// about 150 instructions on the GPU).
SS_HOST_DEVICE SS_INLINE inline long long quotient(long long a, long long b)
{
    const long long q = (long long)((double)a / (double)b);   // off by less than one: 2^50 * 3 * 2^-53
    const long long r = a - q * b;
    return q + (r < 0 ? -1 : r >= b ? 1 : 0);
}

struct SpanCuts {
    long long total_w;   // the coordinate's end: what all units cost
    long long nw;        // number of spans

    // weighted coordinate of span w's cut
    SS_HOST_DEVICE SS_INLINE long long cut(long long w) const { return quotient(w * total_w, nw); }
    // the first span whose cut lies at or behind y: those of a unit's stretch [ya, ye) are from this of ya to this of ye
    SS_HOST_DEVICE SS_INLINE long long first_cut_at_or_after(long long y) const { return quotient(y * nw + total_w - 1, total_w); }
    // pair of the unit at which a span begins whose cut lies in the unit's stretch
    SS_HOST_DEVICE SS_INLINE static int first_pair(long long cut_y, long long ya, int weight, int cost)
    {
        const long long in_unit = cut_y - ya - weight;
        return in_unit > 0 ? (int)quotient(in_unit, cost) : 0;
    }
    // The spans that hold pairs of a unit with n >= 1 pairs whose stretch begins at ya: the last one whose cut
    // lies at or before the unit's first pair ... the last one whose cut lies at or before its last pair.
    SS_HOST_DEVICE SS_INLINE void unit_spans(long long ya, int n, int weight, int cost, int &w_first, int &w_last) const
    {
        w_first = (int)quotient((ya + weight + cost) * nw - 1, total_w);
        w_last = (int)quotient((ya + weight + (long long)n * cost) * nw - 1, total_w);
    }
};

}  // namespace ss
