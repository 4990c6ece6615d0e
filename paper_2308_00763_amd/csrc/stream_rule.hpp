// When pass A streams (a workgroup keeps a table of pixel cells over its run of
// tiles) instead of taking one tile per workgroup.  Host code, plain C++.
#pragma once

#include <math.h>
#include <stdint.h>

namespace pf {

constexpr int kCells = 2048;       // cells of a streaming workgroup's table
constexpr int kPrefRows = 64;      // LDS row-prefix table: window rows
constexpr int kWinMaxW = 128;      // widest frame window staged in LDS
constexpr int kStreamTiles = 4096;  // fewest tiles that stream

// A filter's part in the rule: whether a table is expected to hold its tiles'
// cells, the tiles from which it pays alone, and what one more run of tiles (a
// batch member's) costs, in tiles.
struct StreamRule {
    bool fits;
    int32_t tiles;
    double run;
};

// The expected table.  A tile's cloud has the transition's deviation and that
// of the particles resampled before it; the likelihood falls by `contrast`
// over a move of the disk off itself, 2 / (pi r) of it per pixel, so those lie
// about pi r / (2 contrast) from the best position.  1024 normal draws span 6.5
// deviations, the table has a margin of one more on each side (some of which
// it can do without), and a few pixels.  Where it does not fit, every tile
// pays for the attempt and takes its sums at a lower occupancy (2^24 FP16
// particles, us a step one-tile | streaming: r = 5 and deviations (7, 5) 114 | 148,
// (10, 8) 335 | 437; r = 3, (20, 9) 437 | 462; a batch of radii 3, 8, 12 under a
// flat likelihood 1816 | 2408).  Tiles that certainly reach over more rows than
// the window holds take their sums from the frame either way, better with the
// fewer workgroups per CU (2^22 particles, r = 16, (2, 6): 5630 | 4360).
//
// Where it fits, the table costs each workgroup's run some tiles' gain, by its
// cells and by how its sums are formed.  Measured from 2^22 to 2^24 particles, the
// break-even in multiples of 2^20 by radius and deviations (FP16; FP32 as much or
// a little more):
//            (1, 1)  (3, 3)  (5, 2)  (5, 4)     one-tile | streaming at 2^22, (5, 2)
//     r = 3    3.1     4.7     4.9     6.0         42.5 | 43.7 us
//     r = 5    3.5     4.9     4.8     5.6         41.9 | 42.8
//     r = 6    2.8     4.5     4.7     6.3         45.8 | 47.7
//     r = 8    3.0     4.0     3.2     4.1         47.1 | 44.7
//     r = 12   2.6     4.1     3.8     5.5         59.0 | 57.6
//     r = 16   2.5     3.6     3.2                 69.0 | 62.0
// FP32 with diagnostics loses at every size (2^24 particles 257 | 269 us).
inline StreamRule stream_rule(bool f32, bool f64, bool diagnostics, int r, double contrast, double sigma_x,
                              double sigma_y)
{
    StreamRule s{false, INT32_MAX, 0.0};
    if (f64 || (f32 && diagnostics) || !(contrast > 0)) return s;
    const double d = 3.14159265358979 * r / (2.0 * contrast), post = 3.0 * d * d;
    const double dx = sqrt(sigma_x * sigma_x + post), dy = sqrt(sigma_y * sigma_y + post);
    const double w = 8.5 * dx + 5.0, h = 8.5 * dy + 5.0;
    s.fits = w * h <= (r == 8 ? kCells + 256 : kCells) && w + 2 * r + 1 <= kWinMaxW && h + 2 * r - 2 <= kPrefRows + 3;
    if (s.fits) {
        const double k = w * h * 1e-3;
        const double m = r >= 10 ? 0.2 + 2.3 * k + 16.0 / r : r == 8 ? 2.9 + 0.9 * k : 3.4 + 1.6 * k;
        s.tiles = (int32_t)fmax(kStreamTiles, 1024.0 * m);
        s.run = r >= 10 ? 1.0 : r == 8 ? 2.0 : 2.2;
    } else if (6.5 * sigma_y + 3.0 + 2 * r - 2 >= kPrefRows + 8 && contrast >= 1.0) {
        s.tiles = kStreamTiles;
    }
    return s;
}

// A batch's pass A takes all its tiles one way, by the sum over its stepped
// members: the tiles whose table fits have to outweigh the others, what the
// workgroups' runs cost and a run per member.  (FP16, r = 5, us a step one-tile |
// streaming, by tiles of each member: 8192 tiles 1: 82 | 101, 4: 74 | 74, 8: 73 | 69;
// 32768 tiles 2: 288 | 289, 4: 273 | 245, 64: 251 | 199; r = 12, 16384 tiles 1: 212 |
// 237, 2: 194 | 177.)
struct StreamSum {
    double fit = 0, other = 0, alone = 0, runs = 0;
    void add(const StreamRule& s, int tiles)
    {
        if (s.fits) {
            fit += tiles;
            alone += (double)tiles * s.tiles;
            runs += s.run;
        } else {
            other += tiles;
        }
    }
    bool streams() const { return fit + other >= kStreamTiles && fit > 0 && fit - other >= alone / fit + runs; }
};

}  // namespace pf
