// Which particles of a leaf each of its work items holds (tree layouts; host and
// device).
#pragma once

#include <cstdint>

// First particle of item t of the nt = ceil(ni / 16) items of a leaf of ni
// particles: even runs, none over 16 (t = nt: ni). In 64 bits: a leaf may hold any
// number of particles (where too many have a radius too wide for half of it), and ni
// times nt passes 2^31 from 185,000 on.
constexpr int item_first(int ni, int nt, int t)
{
    return (int)((int64_t)ni * t / nt);
}

// The same for nt <= 4, without the division (exact for products below 2^15).
constexpr int item_first_small(int ni, int nt, int t)
{
    const int x = ni * t;
    return nt == 1 ? x : nt == 2 ? x >> 1 : nt == 3 ? (x * 21846) >> 16 : x >> 2;
}
