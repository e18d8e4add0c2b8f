// light_claims.hpp -- which items of the light PP tiles a wave takes.
//
// The items are `per` parts of each of n tiles.  Workgroups b = g (mod 8) run on one
// XCD and own every 8th tile of the order, from the g-th on: group g's share.  A wave's
// first chunk of items is its number among its group's waves, the last workgroups' first
// (the first ones to start have the heavy tiles); the next ones come from
// the group's counter, or, where there are at most 4 items per wave, at fixed strides.
// When a group's share is taken, its waves go on with the next group's.  The shares
// differ by a tile where n is not a multiple of 8, and the groups' waves where the grid
// is not; what a claim stands for (`fixed`, `chunk`) therefore comes from the launch
// alone, the same for every group: with each group's own, a wave that went on to another
// group left items out (chunks of 2 here and 3 there: 228 of 13808 items of 3452 tiles) or
// took a group's items again that were handed out at strides (2304 of 9232, 2308 tiles).
//
// Plain C++ (constexpr functions are callable on the device): the tests walk it on the
// host.
#pragma once

namespace cube2 {

struct LightClaims {
    int grid, waves, n, per;   // workgroups, waves of each, tiles, items per tile
    int ng, g;                 // groups, the group whose items are being taken
    bool fixed;                // strides instead of counters
    int chunk;                 // items per claim
    int nitems, nw;            // the group's items and waves
    int next;                  // the wave's next chunk (valid in its first lane)
    int item = 0, end = 0;     // the rest of its present one
    int done = 0;              // groups found exhausted

    constexpr LightClaims(int grid_, int block, int wave, int waves_, int n_, int per_, bool counters)
        : grid(grid_), waves(waves_), n(n_), per(per_), ng(grid_ >= 8 ? 8 : 1), g(block % ng),
          fixed(false), chunk(1), nitems(0), nw(0), next(0) {
        // of any group: the most items and the fewest waves
        const int most = (n + ng - 1) / ng * per, few = grid / ng * waves, each = most / (2 * few);
        fixed = most <= 4 * few || !counters;
        chunk = fixed ? 1 : (each < 4 ? each : 4);
        enter();
        // numbered by pairs of waves, the last workgroup's pair first
        const int blocks = nw / waves, pair = wave / 2 * 2;
        next = pair * blocks + (blocks - 1 - block / ng) * (pair + 1 < waves ? 2 : 1) + wave % 2;
    }

    constexpr void enter() {
        nitems = (n > g ? (n - g + ng - 1) / ng : 0) * per;
        nw = (grid - g + ng - 1) / ng * waves;
    }

    // The wave's next item: its tile's place in the order and its part of the tile; false
    // when none is left.  claim(g) adds one to group g's counter and returns what it held
    // (in the wave's first lane); first(v) is v of the wave's first lane.
    template <class Claim, class First>
    constexpr bool take(int &place, int &part, Claim claim, First first) {
        while (item >= end) {
            const int c = first(next);
            if (c >= (nitems + chunk - 1) / chunk) {
                if (fixed || ++done == ng) return false;
                g = g + 1 < ng ? g + 1 : 0;
                enter();
                next = nw + claim(g);   // after the chunks that the group's own waves began with
                continue;
            }
            item = c * chunk;
            end = item + chunk < nitems ? item + chunk : nitems;
            next = fixed ? c + nw : nw + claim(g);
        }
        place = item / per * ng + g;
        part = item % per;
        ++item;
        return true;
    }
};

}  // namespace cube2
