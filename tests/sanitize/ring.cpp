// The ring of sign tiles of the persistent kernel for three and four tokens, played on the host with the kernel's own accounting
// (csrc/rb_flow.h): a loading wavefront that asks for the tiles of every stage, eight that wait for them, use them and give them back,
// in any order of turns.  No tile is overwritten that a wavefront still waits for, and everyone comes to the end, also where wavefronts have given up a
// wait and run ahead of what has been asked for.  Built and run by tests/test_sanitizers.py.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "rb_flow.h"

using namespace rb::flow;

constexpr int TILES = 96, HELD = 3;

struct Segment { int P, CT; };

// gives_up[w]: the stage from which on wavefront w no longer waits for tiles
static const char *play(const std::vector<Segment> &stages, const int (&gives_up)[CWAVES], uint32_t first, unsigned seed)
{
    std::mt19937 rng(seed);
    uint32_t total = first, issued = first, landed = first, used = first;
    std::vector<uint32_t> starts;
    for (const Segment &s : stages) { starts.push_back(total); total += (uint32_t)(s.P * s.CT); }
    uint32_t needs[CWAVES];
    int stage[CWAVES] = {}, row[CWAVES] = {}, piece[CWAVES] = {}, arrived = 0;
    bool waits_for_all[CWAVES] = {};
    for (uint32_t &n : needs) n = first;
    const int n_stages = (int)stages.size();
    int at = 0, done_of_stage = 0;                             // the loading wavefront's place
    while (at < n_stages && stages[at].P * stages[at].CT == 0) ++at;
    for (long step = 0; step < 4000000; ++step) {
        bool all = at == n_stages;
        for (int w = 0; w < CWAVES; ++w) all = all && stage[w] == n_stages;
        if (all) return nullptr;
        const int who = (int)(rng() % (CWAVES + 1));
        if (who == CWAVES) {
            if (at == n_stages) { landed = issued; continue; }
            const int count = stages[at].P * stages[at].CT, m = count - done_of_stage < 4 ? count - done_of_stage : 4;
            if (!ring_has_room(issued, (uint32_t)m, used, TILES)) {
                landed = issued;
                int32_t least = (int32_t)(needs[0] - issued);
                for (int w = 1; w < CWAVES; ++w) { const int32_t u = (int32_t)(needs[w] - issued); least = u < least ? u : least; }
                used = issued + (uint32_t)least;
                if (!ring_has_room(issued, (uint32_t)m, used, TILES)) continue;
            }
            // the tiles that these take the place of
            for (int w = 0; w < CWAVES; ++w)
                if (stage[w] < n_stages && stage[w] < gives_up[w] && (int32_t)(issued + (uint32_t)m - TILES - needs[w]) > 0) return "a tile was overwritten that was still needed";
            issued += (uint32_t)m;
            done_of_stage += m;
            if (done_of_stage == count) { do { ++at; } while (at < n_stages && stages[at].P * stages[at].CT == 0); done_of_stage = 0; }
            continue;
        }
        const int w = who;
        if (stage[w] == n_stages) continue;
        const Segment &s = stages[stage[w]];
        if (waits_for_all[w]) {                                // the sums of all eight
            if (arrived < CWAVES * (stage[w] + 1)) continue;
            waits_for_all[w] = false;
            ++stage[w];
            row[w] = piece[w] = 0;
            continue;
        }
        const int c0 = run_begin(w, s.CT), n = run_begin(w + 1, s.CT) - c0;
        if (row[w] == s.P || n * s.P == 0) {
            if (s.P > 0) needs[w] = starts[stage[w]] + (uint32_t)(s.P * s.CT);
            ++arrived;
            waits_for_all[w] = true;
            continue;
        }
        const int m = n - piece[w] < HELD ? n - piece[w] : HELD;
        const uint32_t wanted = starts[stage[w]] + (uint32_t)(row[w] * s.CT + c0 + piece[w] + m);
        if (row[w] == 0 && piece[w] == 0 && n > HELD) needs[w] = starts[stage[w]] + (uint32_t)c0;
        if (stage[w] < gives_up[w] && (int32_t)(landed - wanted) < 0) continue;
        piece[w] += m;
        if (piece[w] == n) {
            piece[w] = 0;
            ++row[w];
            needs[w] = starts[stage[w]] + (uint32_t)(row[w] * s.CT + (row[w] < s.P ? c0 : 0));
        } else {
            needs[w] = wanted;
        }
    }
    return "someone waits for ever";
}

int main()
{
    std::mt19937 rng(1);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    for (int trial = 0; trial < 600; ++trial) {
        std::vector<Segment> stages;
        for (int n = pick(1, 12); n > 0; --n) stages.push_back(Segment{pick(0, 8), pick(0, 5) ? pick(1, 48) : pick(97, 256)});
        int gives_up[CWAVES];
        const int kind = pick(0, 3), from = pick(0, (int)stages.size());
        for (int &g : gives_up) g = kind == 0 ? 1000 : kind == 1 ? from : kind == 2 ? pick(0, (int)stages.size()) : (pick(0, 1) ? from : 1000);
        const uint32_t first = trial % 2 ? 0u : 0xffffff00u;   // (the counts may wrap)
        if (const char *what = play(stages, gives_up, first, (unsigned)trial)) {
            std::printf("trial %d, kind %d from stage %d of %d: %s\n", trial, kind, from, (int)stages.size(), what);
            return 1;
        }
    }
    std::printf("ring of sign tiles: everyone came to the end\n");
    return 0;
}
