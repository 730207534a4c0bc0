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

// Whose a span is: a wavefront's, its partials handed over inside the workgroup (kernels of one or two row blocks); a workgroup's,
// whose wavefronts take its pairs in turn and leave one partial; a wavefront's by itself (kernels of more row blocks).
enum { kSpanChain = 0, kSpanTeam = 1, kSpanAlone = 2 };

constexpr int kSpansPerWg = 4;   // wavefronts of a workgroup
// The merge adds a unit's partials one after the other: with more than kMaxUnitPartials for the longest unit the spans get longer.
constexpr int kMaxUnitPartials = 32;

struct SpanChoice {
    int mode;
    long long spans;   // of all pairs, cut by cost
    bool whole;        // instead: a span per unit
};

// Wavefronts' spans: of two pairs as long as the chip is not full, of four where a unit would leave too many partials (a hand-over leaves
// one for four spans).
SS_HOST_DEVICE inline long long count_wave_spans(long long total, int longest, long long waves, bool chain)
{
    auto bounded = [&](long long n) { return n < 1 ? 1 : n > waves ? waves : n; };
    const long long n = bounded(total / 2);
    return longest * n > (chain ? kSpansPerWg : 1) * kMaxUnitPartials * total ? bounded(total / 4) : n;
}
// Teams' spans: of two pairs as long as the chip is not full (then half of the wavefronts have none, but the span is over sooner), of
// sixteen where a unit would leave too many partials.  A whole call, in us, with a span per wavefront and no team / spans of 8 / 4 / 2 pairs:
//   24 requests of 30..200 tokens, 8 KV heads, three row blocks  24.1 / 31.9 / 26.5 / 23.7     4 of 40..600, four and five  25.7 / 28.9 / 24.6 / 23.6
//   4 of 1000..3000, e4m3  27.8 / 26.5 / 24.7 / 24.7      one of 60000 over one KV head, five row blocks  108 / 53 (spans of 16) / 74 (spans of 8)
SS_HOST_DEVICE inline long long count_team_spans(long long total, int longest, long long teams)
{
    auto bounded = [&](long long n) { return n < 1 ? 1 : n > teams ? teams : n; };
    const long long n = bounded(total / 2);
    return longest * n > kMaxUnitPartials * total ? bounded(total / 16) : n;
}

// total: pairs of all units (>= 1); longest: pairs of the longest unit; waves: the most wavefronts' spans there can be; classes: a
// kernel of more than two row blocks; kv8: e4m3 caches.
//
// Teams or wavefronts.  A team opens every unit of its span with all four wavefronts and ends it with an exchange: with many units to a
// team that is most of its time, where four wavefronts by themselves open and end four units at once.  With few long units the teams are
// ahead: a quarter of the partials, and the chip's ends closer together.  A whole call, in us, teams / wavefronts by themselves,
// 8 KV heads:
//   three row blocks, bf16, 256 requests of 48 tokens  70 / 42     64 of 200  38 / 34     64 of 400  45 / 43     64 of 800  62 / 63     128 of 1600  178 / 186
//   five row blocks, e4m3   256 of 48  95 / 57     64 of 800  64 / 62     64 of 1600  85 / 85     96 of 512..8192  224 / 232
// So from two units to a team on, and while a unit's pairs on average are not more than kAlonePairs times the units to a wavefront.
// With one or two row blocks the exchange is small and wavefronts hand over: they serve a full chip (64 requests of 256..4096
// tokens: 106 us, and 112 in teams), and calls of many short units (64 of 100 tokens: 24.6, and 26.8 in teams).
//
// Whole units.  A team walks four pairs at once and a chip that is not full has teams to spare, so units up to a few rounds of it get a
// team each: no unit waits behind another's in one span, none is split (before, cuts of equal cost gave one team two units and
// the next none).  A whole call, in us, cuts by cost / whole units: 4 requests of 28..40 tokens, 8 KV heads, three row blocks 23.9 / 18.0,
// five 28.6 / 20.8; 100 of 30..60 over one, five 31.0 / 21.8; two of 20..100 over two, three 23.0 / 18.0; longest unit of 11 pairs, one request 18.4
// / 19.6, 16 requests 22.9 / 20.8, 31 requests 30.0 / 22.7; of 22 pairs level.  With one or two row blocks splitting costs less: 4 requests of
// up to 8 pairs 16.0 / 16.6, 31 of them 23.1 / 19.1.
constexpr int kAlonePairs = 27, kAlonePairsKv8 = 56, kWholePairs = 8;
SS_HOST_DEVICE inline SpanChoice choose_spans(long long total, int longest, long long units, long long waves, bool classes, bool kv8)
{
    const long long teams = waves / kSpansPerWg;
    SpanChoice c;
    c.whole = false;
    if (classes) {
        const bool alone = units >= 2 * teams && (double)total * (double)waves <= (double)(kv8 ? kAlonePairsKv8 : kAlonePairs) * (double)units * (double)units;
        c.mode = alone ? kSpanAlone : kSpanTeam;
        c.spans = count_wave_spans(total, longest, waves, false);
    } else {
        c.spans = count_wave_spans(total, longest, waves, true);
        c.mode = c.spans == waves || units >= 2 * teams ? kSpanChain : kSpanTeam;
    }
    if (c.mode == kSpanTeam) {
        c.spans = count_team_spans(total, longest, teams);
        if (units <= teams && longest <= kWholePairs * (2 * units >= teams ? 2 : 1) / (classes ? 1 : 2)) {
            c.whole = true;
            c.spans = units;
        }
    }
    return c;
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

    // weighted coordinate of span w's cut  (a span per unit of the coordinate: no division, a third of a short call's plan)
    SS_HOST_DEVICE SS_INLINE long long cut(long long w) const { return nw == total_w ? w : quotient(w * total_w, nw); }
    // the first span whose cut lies at or behind y: those of a unit's stretch [ya, ye) are from this of ya to this of ye
    SS_HOST_DEVICE SS_INLINE long long first_cut_at_or_after(long long y) const { return nw == total_w ? y : quotient(y * nw + total_w - 1, total_w); }
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
