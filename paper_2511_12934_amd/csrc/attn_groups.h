// How many workgroups serve each request of a batch in the attention kernel that keeps K/V resident: host arithmetic alone.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace aif {

// The cost of a group in key tiles: a tile walks its request's key tiles in every head and costs about GROUP_TILE more
// (rows, stores); the keys and values come once (64 x 10^4 x 500 keys: 66 us of loop, 15 of ends, 5 of loading).
constexpr int GROUP_TILE = 4, GROUP_LOAD = 6;
constexpr int GROUP_MAX_CU = 512;
// min_tiles of a batch: a tile a SIMD gives a small batch every compute unit; a tile a wave makes the fewest groups.
constexpr int GROUP_MIN_TILES = 4, GROUP_FEWEST_TILES = 12;

// Requests of tiles[i] > 0 candidate tiles over keys[i] key tiles, n <= n_cu <= GROUP_MAX_CU of them: groups[i] workgroups for
// each, at most n_cu in all, so that the costliest group costs as little as that allows (to 1 in 64).  No request gets more
// than one for every min_tiles tiles begun.  Returns their number.
// What bounds it: a division a request and probe of the search, on the host and before the call's first launch.  256 requests
// of 75 to 300 candidates over 100 keys, one call waited for: 102.4 us with groups of one size, 110.3 with a bisection in whole
// numbers (ten probes, 18 us on another processor), 101.1 with four to five probes in floats over arrays (1.0 to 1.4 us there; what
// rounding does to a count here does it to the count that is used, so the bound holds).
inline int plan_group_counts(int n, const int32_t *tiles, const int32_t *keys, int n_cu, int min_tiles, int32_t *groups)
{
    float cost[GROUP_MAX_CU], load[GROUP_MAX_CU], most[GROUP_MAX_CU];
    double all = 0, loads = 0;
    for (int i = 0; i < n; ++i) {
        cost[i] = (float)tiles[i] * (keys[i] + GROUP_TILE);
        load[i] = GROUP_LOAD * keys[i];
        most[i] = (tiles[i] + min_tiles - 1) / min_tiles;
        all += cost[i];
        loads += load[i];
    }
    // enough groups of request i that none costs more than w: cost / (w - load), rounded up
    auto count = [&](float w) {
        int sum = 0;
        for (int i = 0; i < n; ++i) {
            const float room = std::max(w - load[i], 1.0f);
            const int g = (int)std::min(cost[i] / room, most[i]);
            groups[i] = g + (g < most[i] && g * room < cost[i] ? 1 : 0);
            sum += groups[i];
        }
        return sum;
    };
    // Between a cost that is too little and one that is enough: every probe goes where count() would fall to n_cu if the tiles
    // cost / (w - load) fell as 1 / w and the rounding up stayed half a group a request, but not past the middle of what is left.
    double lo = std::floor((all + loads) / n_cu), hi = 0, w = std::max(lo, 1.0), tried = -1;
    int sum = 0;
    for (;;) {
        const int c = count(tried = w);
        const double next = std::floor(w * (c - 0.5 * n) / (n_cu - 0.5 * n));
        if (c <= n_cu) {
            hi = w;
            sum = c;
            if (c == n_cu || hi - lo <= 1 + hi / 64) break;
            w = std::max(next, std::floor((lo + hi) / 2));
            w = std::min(w, hi - 1);
        } else {
            lo = w;
            if (hi == 0)
                w = std::max(next, lo + 1 + std::floor(lo / 64));
            else {
                if (hi - lo <= 1 + hi / 64) break;
                w = std::max(std::min(next, std::floor((lo + hi) / 2)), lo + 1);
            }
        }
    }
    return tried == hi ? sum : count(hi);
}

// How many groups of four tiles a batch of the user network may take before it is cut into groups of twelve at least.  Its
// candidates are the users' own histories: the groups all load their keys and values at the same time and do little else, so from
// 5/8 of the units on (all of them for heads of 32, half the bytes) loading more often costs more than shorter groups save.
// Users of 125 to 500 items, calls back to back, us, groups of twelve / of four (on 256 units):
// 128 -> 64: 32 users (111 groups of four) 35.2 / 33.8; 44 (153) 36.4 / 36.0; 52 (180) 37.5 / 37.5; 64 (221) 39.1 / 39.9; 84 (290, cut
// to 256) 41.3 / 42.8; 48 -> 32: 64 (221) 27.4 / 26.9; 80 (277) 28.6 / 28.3; 90 (312) 29.4 / 30.0.
// (Not by the line: 92 to 120 users of 128 -> 64 take 1 to 4 % less in fours, whose groups have grown to five or six tiles there;
// shorter histories at as many groups take 2 to 4 % more.  Scoring gains up to a group a unit: its tiles do more each.)
inline int user_fine_groups(int n_cu, int d_head) { return d_head == 32 ? n_cu : 5 * n_cu / 8; }

// min_tiles for a batch whose groups of min_tiles are wanted as long as they are at most most_fine.
inline int groups_min_tiles(int n, const int32_t *tiles, int min_tiles, int64_t most_fine)
{
    int64_t fine = 0;
    for (int i = 0; i < n; ++i) fine += (tiles[i] + min_tiles - 1) / min_tiles;
    return fine <= most_fine ? min_tiles : std::max(min_tiles, GROUP_FEWEST_TILES);
}

}  // namespace aif
