// What the wavefronts of the few-token kernel read of a layer's input scales and sign tiles, done on the
// host with the kernel's own arithmetic (csrc/rb_layout.h) under the address sanitizer: blocks of exactly
// the size of the layer, every width up to 4224 columns, every number of wavefronts that a wider
// op of the same launch may bring.  Built and run by tests/test_sanitizers.py.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "rb_layout.h"

using namespace rb;

static int one_layer(int K, int in, int waves)
{
    const int n = units_of(in), run = n / waves, rest = n % waves;
    uint16_t *h = (uint16_t *)std::malloc((size_t)K * in * 2);
    for (int i = 0; i < K * in; ++i) h[i] = (uint16_t)i;
    std::vector<int> seen(n, 0);
    int bad = 0;
    for (int wave = 0; wave < waves; ++wave) {
        const UnitRun r = unit_run(wave, run, rest);
        auto request = [&](int u) {
            if (u < 0 || u >= n || u / 2 >= col_tiles(in)) ++bad;             // (the sign tile that holds the unit)
            for (int lane = 0; lane < 64; ++lane) {
                const int ch = lane & 15, row4 = lane >> 4;
                if (row4 >= K) continue;
                uint16_t v[8];
                std::memcpy(v, h + u * UNIT_COLS + ((uint32_t)row4 * (uint32_t)in + chunk_scales_at(u, ch, in)), 16);
                if (chunk_exists(u, ch, in) && v[0] != (uint16_t)(row4 * in + u * UNIT_COLS + 8 * ch)) ++bad;
            }
        };
        request(first_request(r, in));
        if (r.begin < r.end && first_request(r, in) != r.begin) ++bad;
        for (int u = r.begin; u < r.end; ++u) {
            if (u < n) ++seen[u];
            if (u + 1 < r.end) request(u + 1);
        }
    }
    for (int u = 0; u < n; ++u) bad += seen[u] != 1;
    std::free(h);
    return bad;
}

int main()
{
    for (int K = 2; K <= 3; ++K)
        for (int in = 32; in <= 4224; in += 32)
            for (int waves = 1; waves <= 16; ++waves)
                if (const int bad = one_layer(K, in, waves)) {
                    std::printf("K=%d in=%d wavefronts=%d: %d wrong\n", K, in, waves, bad);
                    return 1;
                }
    std::printf("few-token requests: all in bounds\n");
    return 0;
}
