// Launch shape of the Metropolis colour kernels (host side).
#pragma once

#include <stdint.h>

namespace cvf {

// Target number of wavefronts of a Metropolis colour launch.
#ifndef CVF_MET_WAVES
#define CVF_MET_WAVES 4096
#endif
// Smallest L % 4 == 2 lattice whose shape is made for quads.
#ifndef CVF_MET_RAGGED_MIN
#define CVF_MET_RAGGED_MIN 1024
#endif

struct MetShape {
    uint32_t quad;         // 1: 4-column quads (L % 4 == 0), 2: quads, L % 4 == 2, 0: column pairs
    uint32_t rows;         // rows per wavefront (1, or even, 2..32)
    uint32_t row_blocks;   // grid.y: four wavefronts per workgroup stack vertically
};

// Row blocks: lanes own 4-column quads (the last one ragged in mode 2) or
// column pairs (mode 0), 64 per wavefront; each wavefront walks `rows` rows of
// its column group.  The row count aims the grid at CVF_MET_WAVES wavefronts
// (at L = 4096: 16 rows, 1024 workgroups, all resident at once).
inline MetShape met_shape_mode(uint32_t L, uint32_t quad)
{
    MetShape m;
    m.quad = quad;
    const uint32_t per_lane = m.quad ? 4 : 2;
    const uint32_t groups = ((L + per_lane - 1) / per_lane + 63) / 64;
    const uint32_t target = CVF_MET_WAVES;
    const uint32_t waves_per_group = groups >= target ? 1 : target / groups;
    uint32_t rows = (L + waves_per_group - 1) / waves_per_group;
    rows = (rows + 1) & ~1u;
    if (rows < 2) rows = 2;
    if (rows > 32) rows = 32;
    m.rows = rows;
    m.row_blocks = ((L + rows - 1) / rows + 3) / 4;
    return m;
}

// Row blocks of any lattice, small ones of L % 4 == 2 in column pairs.  What a
// launch takes is met_launch.
inline MetShape met_shape(uint32_t L)
{
    const uint32_t quad = (L % 4 == 0) ? 1 : (L >= CVF_MET_RAGGED_MIN ? 2 : 0);
    return met_shape_mode(L, quad);
}

// Largest side whose lattice is moved one row of quads per wavefront instead of
// in row blocks: up to there the launch is bound by a wavefront's latency,
// not by issue (us per sweep, one row / shape above: L = 256 8.9 / 10.3,
// L = 1024 11.6 / 13.1, L = 1600 18.9 / 21.4, L = 1900 23.7 / 25.9, L = 2044
// 25.2 / 26.3, L = 2046 26.5 / 30.8, L = 2048 24.6 / 24.5, L = 2400 34.0 / 33.0,
// L = 4096 79.1 / 72.9; sides that are no multiple of 16 would still gain up to
// 2200, L = 2050 29.3 / 36.6).
#ifndef CVF_MET_ONE_ROW_MAX
#define CVF_MET_ONE_ROW_MAX 2046
#endif
inline bool met_one_row(uint32_t L) { return L <= CVF_MET_ONE_ROW_MAX; }

// The shape of a launch: quads, one row or a block of rows per wavefront.
inline MetShape met_launch(uint32_t L)
{
    const uint32_t quad = L % 4 == 0 ? 1 : 2;
    if (met_one_row(L)) return {quad, 1, (L + 3) / 4};
    return met_shape_mode(L, quad);
}

// Whether a sweep's stores are written through L2.  Rows of L % 4 == 2 start
// off a dword boundary, so that a wavefront's stores end inside a line: on
// lattices well beyond the L2s' 32 MB those lines are better merged there than
// sent out in two parts (us per sweep, through / left to L2: L = 2050 37.4 /
// 38.4, L = 3002 57.7 / 61.2, L = 3602 80.0 / 80.3, L = 4094 93.8 / 90.9, L =
// 4098 102.2 / 99.7, L = 8002 327.8 / 318.5, L = 8194 367.5 / 355.9, L = 16382
// 1305 / 1288).  Aligned rows gain or stay the same at every size.
inline bool met_through(uint32_t L) { return L % 4 == 0 || (uint64_t)L * L <= 14000000u; }

}  // namespace cvf
