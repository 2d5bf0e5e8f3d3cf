// What the workgroups of an ordering in one launch (k_small_frame) say to each other, apart from how they sort: no HIP in here, so that a
// test can run it on the CPU under every order of its loads and stores.
//
// A tile's word is the call's number << 16 | its pairs, and stays so until the next call.  One more word, the state, says how the
// call ended: the number << 16 | what was decided, and whoever decides first has decided for all.  The totals' workgroup decides
// SMALL_PUBLISHED once it has seen every tile's word, and stores the totals only if that stands; a tile whose looks at the tiles before it
// have ended decides SMALL_GIVEN_UP, and leaves its pairs out only if that stands.  Where SMALL_PUBLISHED stands instead, all words have
// been seen, so its next look finds them: totals that arrive are those of an ordering with every tile in place.
//
// Memory: pair(i), the words 2 i and 2 i + 1; state(); swap(was, now), the state before it, which is `now` behind it if it was `was`;
// rest(), between two looks.  Words and state are past all caches, each is loaded before what depends on it is, and a workgroup's
// barrier stands between its looks and its decision, and between that and its next look: no fence is needed besides.
#pragma once
#include <stdint.h>

namespace fs {

constexpr int SMALL_MAX_TILES = 1024;
constexpr int SMALL_THREADS = 256;
constexpr int SMALL_TILES_PER = SMALL_MAX_TILES / SMALL_THREADS;
static_assert(SMALL_TILES_PER == 4, "two loads of two words for each thread");

constexpr uint32_t SMALL_PUBLISHED = 1, SMALL_GIVEN_UP = 2;

// Thread t looks after tiles 2 t, 2 t + 1, 512 + 2 t and 512 + 2 t + 1.
__device__ __forceinline__ int small_tile(int t, int q) { return (q >> 1) * 2 * SMALL_THREADS + 2 * t + (q & 1); }

// What those of thread t's tiles that are below `end` have said in this call (0 for the others); false when one of them says nothing
// in `polls` looks.
template <typename Memory>
__device__ __forceinline__ bool small_look(Memory mem, int t, int end, uint32_t call, int polls, uint32_t (&c)[SMALL_TILES_PER])
{
    for (int k = 0; k < polls; k++) {
        unsigned long long w[SMALL_TILES_PER / 2] = {};
#pragma unroll
        for (int h = 0; h < SMALL_TILES_PER / 2; h++)
            if (small_tile(t, 2 * h) < end) w[h] = mem.pair(h * SMALL_THREADS + t);
        bool all = true;
#pragma unroll
        for (int q = 0; q < SMALL_TILES_PER; q++) {
            const uint32_t word = (uint32_t)(w[q >> 1] >> 32 * (q & 1));
            const bool mine = small_tile(t, q) < end;
            all = all & (!mine | (word >> 16 == call));
            c[q] = mine ? word & 0xffffu : 0u;
        }
        if (all) return true;
        mem.rest();
    }
    return false;
}

// What has been decided: `mine`, or what another workgroup of this call has decided before.  was: the state as it was loaded at any
// time in this launch.  (It changes once in a call: the loop ends behind its second swap.)
template <typename Memory>
__device__ __forceinline__ uint32_t small_decide(Memory mem, uint32_t call, uint32_t was, uint32_t mine)
{
    while (was >> 16 != call) {
        const uint32_t found = mem.swap(was, call << 16 | mine);
        if (found == was) return mine;
        was = found;
    }
    return was & 0xffffu;
}

}  // namespace fs
