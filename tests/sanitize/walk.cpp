// The passes that the host asks for in the initialisation (csrc/rb_walk.h), played against updates of given numbers of iterations.  Built and run by
// tests/test_sanitizers.py.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "rb_walk.h"

using namespace rb::derive;

static int play(const char *what, int K, const std::vector<int> &iterations)
{
    int needed = 0, asked = 0, looks = 0, n = K * (FIRST_LOOK + 1);
    for (int i : iterations) needed += i + 1;                  // (and the pass after them)
    for (;;) {
        asked += n;
        ++looks;
        if (asked >= needed) break;
        int finished = 0, before = 0;
        while (before + iterations[finished] + 1 <= asked) before += iterations[finished++] + 1;
        n = passes_to_ask(asked, asked - before, finished, (int)iterations.size() - finished);
        if (n < 1 || n > MOST_PASSES) { std::printf("%s: %d passes asked for\n", what, n); return 1; }
    }
    // Looks: one for every two passes or more (two over the mean) until an eighth of all is more, from 24 passes on one for every ninth that they grow, and
    // one for every MOST_PASSES less an eighth.  Passes too many are all of the last request: a quarter, or for each update left FIRST_LOOK + 2 where it takes two.
    const int n_updates = (int)iterations.size(), extra_allowed = needed / 4 + FIRST_LOOK * n_updates;
    const int looks_allowed = 12 + (int)std::ceil(std::log(std::max(1.0, needed / 24.0)) / std::log(9.0 / 8.0)) + needed / (MOST_PASSES - MOST_PASSES / 8);
    std::printf("%s: %d passes needed, %d asked for, %d looks\n", what, needed, asked, looks);
    if (looks > looks_allowed || asked - needed > extra_allowed) { std::printf("%s: too many\n", what); return 1; }
    return 0;
}

int main()
{
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    int bad = 0;
    for (int K = 1; K <= 3; ++K)
        for (int T : {1, 2, 5, 20, 200}) {
            const size_t n = (size_t)K * T;
            for (int each : {1, 2, 4, 5, 8, 30, 200}) bad += play("all alike", K, std::vector<int>(n, each));
            std::vector<int> one(n, 4);
            one[0] = 200;
            bad += play("a slow one first", K, one);
            std::vector<int> middle(n, 4);
            middle[n / 2] = 200;
            bad += play("a slow one later", K, middle);
            std::vector<int> any(n);
            for (int &i : any) i = pick(0, 9) ? pick(2, 6) : pick(20, 200);
            bad += play("any", K, any);
        }
    if (bad) return 1;
    std::printf("passes asked for in measure\n");
    return 0;
}
