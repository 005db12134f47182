// Several layers in one launch, one behind the other through the window positions: a layer's workgroup takes position p as soon
// as the layer below has left it in memory, so that the launch takes about as long as its longest layer and not as all of
// them.  For grids that leave most of the chip idle (plan.cpp): every workgroup has one series tile, or a quarter of one, and
// one residue class, and its positions rise in every layer (in the reverse pass they fall).
//
// A workgroup counts its complete positions in a word of its own.  Data that another workgroup reads is written through to
// memory and read past the caches (buf_store_shared, buf_load_shared), and a position is counted after a wait for its
// stores and a barrier behind the waits of all waves that store: whoever sees the count sees the data.
//
// Every wait ends.  Workgroups take their places by ticket, in the order in which the layers run: whoever waits, waits for lower
// tickets only, which have been drawn by workgroups that are running, and the lowest one of those that have not ended waits
// for nobody.  That does not depend on the order of dispatch, nor on how many workgroups the chip holds.  (A wait that goes on
// for seconds all the same, because calls overlap on one workspace, is given up, once for all that this wave reads from then on,
// which is NaN: loss and forecasts show it, in the reverse pass the gradients.)
//
// What it costs: words of several workgroups in one cache line, and all lanes storing the same one, made every position wait
// (512 hourly series, the first two layers: 4800 us); a line each and one lane that stores: 350 us (as two launches 440 us).
// Fewer positions between a store and its count change less than 1 %; pauses between two looks: at kWidePollSleep.  Places dealt so that a tile's workgroups share an XCD, as in the launches of one layer, are slower (517 us), also with
// data handed on in whole cache lines (534 us): what is written through by one workgroup and read past the caches by another
// is better not in the same L2.
#pragma once

#include "device_utils.h"
#include "esrnn_internal.h"

namespace esrnn {

namespace {

constexpr int kPollSleep = 4;       // (times 64 clocks)
// in 16-series layers, whose eight waves all look, four to sixteen words each: first two layers of 512 hourly series 368 - 378 us with 4,
// 356 with 20, 351 - 360 with 40, 360 with 120; of 501 monthly ones and for forecasts of 333 hourly ones level.  (In 4-series layers, one
// wave of four words, 40 costs 7 quarterly series 3 us of 41.)
constexpr int kWidePollSleep = 40;
constexpr int kMostLooks = 1 << 22; // (seconds)

// Memory operations of this wave are complete, but for the last N.
template <int N>
__device__ __forceinline__ void stores_complete_but()
{
    static_assert(N < 64, "");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | 0x70 | 0xf00 | (N >> 4) << 14);      // vmcnt(N), the other counters at their most
    asm volatile("" ::: "memory");
}

struct Progress {
    unsigned *mine = nullptr;           // this workgroup's word: complete positions times the dilation
    const unsigned *below = nullptr;    // words of the workgroups whose output this one reads: [quarter][class]
    int words = 1, d = 1;               // how many (at most 64); dilation of that layer

    // by one lane of the wave that is told to, without a branch between the requests around it: the resource ends behind the
    // word, and what the other lanes store lies outside
    __device__ __forceinline__ void publish(int value, bool told) const
    {
        buf_store_shared(make_rsrc(mine, 4), told ? 4 * (threadIdx.x & 63) : 4, 0, __builtin_bit_cast(float, value));
    }
};

// The places of a launch, as the workgroups draw them.
struct Places {
    int layers, NB;
    int d[kTogetherMost];               // classes of every layer
    int quarters[kTogetherMost];        // workgroups of a series tile and class: 4 for a 4-series layer, else 1
    int first[kTogetherMost + 1];       // first place of every layer, and the number of all
    unsigned *words;                    // the ticket, and a word per place, a cache line each
};
struct Place {
    int layer, bt, q, chain;
};
__device__ __forceinline__ Place draw_place(const Places &t, unsigned *slot)
{
    if (threadIdx.x == 0) *slot = atomicAdd(t.words, 1u);
    __syncthreads();
    // (unsigned: in a workspace whose words were not cleared a ticket is any number, and every place has to be in the launch)
    const int ticket = (int)min((unsigned)__builtin_amdgcn_readfirstlane((int)*slot), (unsigned)t.first[t.layers] - 1u);
    int l = 0;
    while (ticket >= t.first[l + 1]) ++l;
    const int groups = t.NB * t.quarters[l], x = ticket - t.first[l], chain = x / groups, y = x - chain * groups;
    if (t.quarters[l] == 1) return {l, y, 0, chain};
    // the quarters of a tile eight apart
    const int full = t.NB & ~7, rest = y - 4 * full, m = rest < 0 ? 8 : t.NB & 7, z = rest < 0 ? y & 31 : rest;
    return {l, (rest < 0 ? (y >> 5) * 8 : full) + z % m, z / m, chain};
}
// a layer's words: [series tile][quarter][class]
__device__ __forceinline__ unsigned *word_at(const Places &t, int layer, int bt, int q, int chain)
{
    return t.words + kWordStride * (1 + t.first[layer] + (bt * t.quarters[layer] + q) * t.d[layer] + chain);
}
// of a workgroup that reads what layer `before` leaves (-1: none)
__device__ __forceinline__ Progress progress_of(const Places &t, const Place &p, int before)
{
    Progress g;
    g.mine = word_at(t, p.layer, p.bt, p.q, p.chain);
    if (before < 0) return g;
    // (a quarter reads the same quarter, or all there are)
    const bool same = t.quarters[p.layer] == t.quarters[before];
    g.below = word_at(t, before, p.bt, same ? p.q : 0, 0);
    g.d = t.d[before];
    g.words = same ? g.d : g.d * t.quarters[before];
    return g;
}

// What a layer of a launch does for the others: kAlone, nothing; kFirst, its positions are counted; kLater, it also waits for the
// layer before it; kLast, it waits only.
enum { kAlone, kFirst, kLater, kLast };

// What a wave knows of the layer before its own (the one below, in the reverse pass the one above).
struct Below {
    const Progress &g;
    unsigned word, first;               // this lane's word, and the first position of its class
    int last;                           // and its last one, of so many positions (where they fall)
    int have = 0;
    bool lost = false;
    __device__ Below(const Progress &progress, int positions = 0) : g(progress)
    {
        word = min((int)(threadIdx.x & 63), g.words - 1);
        first = word % (unsigned)g.d;
        last = (int)first < positions ? (int)first + (positions - 1 - (int)first) / g.d * g.d : -1;
    }
    __device__ __forceinline__ void look() { have = __builtin_bit_cast(int, buf_load_shared(make_rsrc(g.below), 4 * kWordStride * word, 0)); }
    // until position p is complete in every class of the layer below
    template <int pause = kPollSleep>
    __device__ __forceinline__ void wait(int p)
    {
        for (int i = lost ? kMostLooks : 0; __ballot((int)first + have > p) != ~0ull; ++i) {
            asm volatile("" ::: "memory");
            if (i == kMostLooks) { lost = true; break; }
            __builtin_amdgcn_s_sleep(pause);
            look();
        }
        asm volatile("" ::: "memory");
    }
    // The same where positions fall from the last one to 0: every class from its own last position.  (The first comparison stands
    // outside the loop.  In its head, which is reached from a look as well, it waits for everything that is under way: with a
    // wait every position that was 0.77 us of each.  Forward layers wait once in several positions, and the drain costs them nothing:
    // the first two layers for forecasts of 333 hourly series 292 us, and 308 us without it.)
    __device__ __forceinline__ void wait_falling(int p)
    {
        if (!g.below) return;
        bool complete = __ballot(last - have < p) == ~0ull;
        for (int i = lost ? kMostLooks : 0; !complete; ++i) {
            asm volatile("" ::: "memory");
            if (i == kMostLooks) { lost = true; break; }
            __builtin_amdgcn_s_sleep(kPollSleep);
            look();
            complete = __ballot(last - have < p) == ~0ull;
        }
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ float checked(float v) const { return lost ? __builtin_nanf("") : v; }
};

}  // namespace

}  // namespace esrnn
