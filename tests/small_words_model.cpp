// small_words.hpp under every order of its loads and stores, on the CPU: the workgroups of a small frame's ordering as coroutines that
// stop ahead of each of them.  Tile 0 speaks late, tile 1 has spoken, tile 2 looks at those two, and threads 0 and 1 of the totals'
// workgroup look at tiles 0, 1 and 2.  Arguments: looks of tile 2, looks of the totals' threads, and 1 for the rule that does not do: a
// tile that gives up takes its word back.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <vector>

#define __device__
#define __forceinline__ inline
#include "small_words.hpp"

using namespace fs;

static constexpr uint32_t CALL = 7;
enum Actor { FIRST, LAST, LOOK0, LOOK1, ACTORS };

static uint32_t said[SMALL_MAX_TILES + 1];
static ucontext_t here, actor[ACTORS];
static char stack[ACTORS][32768];
static bool ended[ACTORS];
static int running;

static void stop() { swapcontext(&actor[running], &here); }

struct Memory {
    unsigned long long pair(int i) const
    {
        stop();
        return said[2 * i] | (unsigned long long)said[2 * i + 1] << 32;
    }
    uint32_t state() const { stop(); return said[SMALL_MAX_TILES]; }
    uint32_t swap(uint32_t was, uint32_t now) const
    {
        stop();
        const uint32_t found = said[SMALL_MAX_TILES];
        if (found == was) said[SMALL_MAX_TILES] = now;
        return found;
    }
    void rest() const {}
};

static int looks_tile, looks_totals, take_back, looked;
static bool placed, late, published, silent;
static uint32_t state_before;

static void say(int tile, uint32_t word)
{
    stop();
    said[tile] = word;
}

static void last_tile()
{
    uint32_t c[SMALL_TILES_PER];
    say(2, CALL << 16 | 5);
    if (small_look(Memory{}, 0, 2, CALL, looks_tile, c)) { placed = true; return; }
    late = true;
    if (take_back) say(2, 0);
    else if (small_decide(Memory{}, CALL, Memory{}.state(), SMALL_GIVEN_UP) == SMALL_PUBLISHED)
        placed = small_look(Memory{}, 0, 2, CALL, looks_tile, c);
}

static void totals(int thread)
{
    uint32_t c[SMALL_TILES_PER];
    if (!small_look(Memory{}, thread, 3, CALL, looks_totals, c)) silent = true;
    if (++looked < 2 || silent) return;   // (the workgroup's barrier)
    published = take_back || small_decide(Memory{}, CALL, state_before, SMALL_PUBLISHED) == SMALL_PUBLISHED;
}

static void run(int who)
{
    if (who == FIRST) say(0, CALL << 16 | 3);
    else if (who == LAST) last_tile();
    else totals(who - LOOK0);
    ended[who] = true;
    stop();
}

int main(int, char** argv)
{
    looks_tile = atoi(argv[1]);
    looks_totals = atoi(argv[2]);
    take_back = atoi(argv[3]);
    long schedules = 0, wrong = 0, whole = 0, given_up = 0, placed_late = 0;
    std::vector<int> choice, choices;   // of this schedule at every step: which of the actors that have not ended, of how many
    do {
        memset(said, 0, sizeof(said));
        said[1] = CALL << 16 | 4;
        state_before = said[SMALL_MAX_TILES] = (CALL - 1) << 16 | SMALL_PUBLISHED;
        looked = 0;
        placed = late = published = silent = false;
        for (int k = 0; k < ACTORS; k++) {
            ended[k] = false;
            getcontext(&actor[k]);
            actor[k].uc_stack = {stack[k], 0, sizeof(stack[k])};
            makecontext(&actor[k], (void (*)())run, 1, k);
            running = k;
            swapcontext(&here, &actor[k]);   // (to its first load or store)
        }
        for (size_t step = 0;; step++) {
            int ready[ACTORS], count = 0;
            for (int k = 0; k < ACTORS; k++)
                if (!ended[k]) ready[count++] = k;
            if (count == 0) break;
            if (step == choice.size()) { choice.push_back(0); choices.push_back(count); }
            running = ready[choice[step]];
            swapcontext(&here, &actor[running]);
        }
        schedules++;
        wrong += published && !placed;
        whole += published && placed;
        given_up += !published;
        placed_late += late && placed;
        while (!choice.empty() && choice.back() + 1 == choices.back()) { choice.pop_back(); choices.pop_back(); }
        if (!choice.empty()) choice.back()++;
    } while (!choice.empty());
    printf("%ld %ld %ld %ld %ld\n", schedules, wrong, whole, given_up, placed_late);
}
