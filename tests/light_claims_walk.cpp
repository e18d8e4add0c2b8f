// Walks the claim protocol of the light PP tiles (csrc/light_claims.hpp) on the host:
//   light_claims_walk GRID WAVES PER FROM TO STEP SEED
// takes every item of n = FROM, FROM + STEP, ... <= TO light tiles with GRID workgroups of
// WAVES waves in random orders of the waves and prints the first n at which an item is not
// taken exactly once.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2512_12629_amd/csrc/light_claims.hpp"

namespace {

uint64_t state = 1;
uint32_t draw(uint32_t below) {     // xorshift64*
    state ^= state >> 12;
    state ^= state << 25;
    state ^= state >> 27;
    return (uint32_t)((state * 2685821657736338717ull) >> 33) % below;
}

// order 0: waves at random; 1: each runs to its end before the next begins, in random
// order (workgroups that reach the light tiles late); 2: whole groups late
bool walk(int grid, int waves, int n, int per, int order, int &missed, int &repeated) {
    std::vector<cube2::LightClaims> w;
    for (int b = 0; b < grid; ++b)
        for (int i = 0; i < waves; ++i) w.emplace_back(grid, b, i, waves, n, per, true);
    std::vector<int> live(w.size());
    for (size_t i = 0; i < w.size(); ++i) live[i] = (int)i;
    for (size_t i = w.size(); i > 1; --i) std::swap(live[i - 1], live[draw((uint32_t)i)]);
    const int late = (int)draw(8);
    int counter[8] = {};
    std::vector<int> taken((size_t)n * per, 0);
    bool bounds = true;
    auto claim = [&](int g) { return counter[g]++; };
    auto first = [](int v) { return v; };
    auto step = [&](int i) {
        int place = 0, part = 0;
        if (!w[i].take(place, part, claim, first)) return false;
        if (place < 0 || place >= n || part < 0 || part >= per) return bounds = false;
        ++taken[(size_t)place * per + part];
        return true;
    };
    if (order == 1) {
        for (int i : live)
            while (step(i)) {}
    } else {
        for (int pass = order == 2 ? 0 : 1; pass < 2; ++pass) {
            std::vector<int> now;
            for (int i : live)
                if (order != 2 || ((i / waves) % 8 == late) == (pass == 1)) now.push_back(i);
            while (!now.empty()) {
                const uint32_t k = draw((uint32_t)now.size());
                if (!step(now[k])) {
                    now[k] = now.back();
                    now.pop_back();
                }
            }
        }
    }
    missed = repeated = 0;
    for (int t : taken) {
        missed += t == 0;
        repeated += t > 1;
    }
    return bounds && missed == 0 && repeated == 0;
}

}  // namespace

int main(int argc, char **argv) {
    if (argc != 8) return 2;
    const int grid = atoi(argv[1]), waves = atoi(argv[2]), per = atoi(argv[3]), from = atoi(argv[4]),
              to = atoi(argv[5]), step = atoi(argv[6]);
    state = 88172645463325252ull + (uint64_t)atoi(argv[7]);
    for (int n = from; n <= to; n += step)
        for (int order = 0; order < 3; ++order) {
            int missed, repeated;
            if (!walk(grid, waves, n, per, order, missed, repeated)) {
                std::printf("%d tiles, order %d: of %d items %d left out, %d taken again\n", n, order,
                            n * per, missed, repeated);
                return 1;
            }
        }
    return 0;
}
