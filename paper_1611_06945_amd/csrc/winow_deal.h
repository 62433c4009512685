// How the row-of-planes Winograd kernel deals its tiles to workgroups (plain C++, host and device).
#pragma once

namespace convfwd {

// Workgroups of a launch: 256, one per CU, or two for each tile of the fullest XCD, so that every XCD can halve its tiles where they are few.
// Two for each tile of the launch are not enough: an XCD's tiles may be an eighth rounded up and its workgroups an eighth rounded down
// (of the numbers below 128 only multiples of eight are halved throughout).
constexpr int winow_grid(int tiles) { return tiles > 120 ? 256 : 16 * ((tiles + 7) / 8); }

struct WinowShare {
    int first, count;  // tiles of the XCD
    int wgs;           // ... and its workgroups
    int full;          // tiles ahead of the last round
    bool halved;       // the last round has tiles for no more than half of the workgroups, its tiles are halved
    int units;         // whole tiles, then halves of the last ones; workgroup i takes i, i + wgs, ...
};

constexpr WinowShare winow_share(int tiles, int grid, int xcd)
{
    WinowShare s{};
    const int rem = tiles & 7, more = xcd < rem ? 1 : 0;
    s.first = xcd * (tiles >> 3) + (more ? xcd : rem);
    s.count = (tiles >> 3) + more;
    s.wgs = (grid >> 3) + (xcd < (grid & 7) ? 1 : 0);
    s.full = s.count - s.count % s.wgs;
    s.halved = 2 * (s.count - s.full) <= s.wgs;
    s.units = s.halved ? 2 * s.count - s.full : s.count;
    return s;
}

}  // namespace convfwd
