// lhmm_grid.h -- the cell grids of micro-boxes and of the macro problem (not
// part of the public ABI): plain host arithmetic, in part shared with the kernels.
#ifndef LHMM_GRID_H
#define LHMM_GRID_H

#include <algorithm>
#include <cmath>

__host__ __device__ inline double m3_det(const double* A) {
    return A[0] * (A[4] * A[8] - A[5] * A[7]) - A[1] * (A[3] * A[8] - A[5] * A[6]) +
           A[2] * (A[3] * A[7] - A[4] * A[6]);
}

// perpendicular widths w_a = V / |h_b x h_c|
__host__ __device__ inline void m3_widths(const double* h, double* w) {
    const double V = fabs(m3_det(h));
    for (int a = 0; a < 3; ++a) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        const double ux = h[b], uy = h[3 + b], uz = h[6 + b];
        const double vx = h[c], vy = h[3 + c], vz = h[6 + c];
        const double x = uy * vz - uz * vy, y = uz * vx - ux * vz, z = ux * vy - uy * vx;
        w[a] = V / sqrt(x * x + y * y + z * z);
    }
}

// Cells per direction of a cell with widths w, before the limit of a box's
// capacity: as many as leave each at least the cutoff wide (z: cutoff / zsub),
// at least the 2 sub + 1 of a stencil.  Returns whether the cell is narrow (a
// width below three cutoffs).
__host__ __device__ inline bool cell_counts(const double* w, double rc, int zsub, int* nc) {
    bool narrow = false;
    for (int a = 0; a < 3; ++a) {
        const int sub = a == 2 ? zsub : 1;
        int n = (int)floor(sub * w[a] / rc);
        if (!(w[a] >= 3.0 * rc)) narrow = true;
        if (n < 2 * sub + 1) n = 2 * sub + 1;
        nc[a] = n;
    }
    return narrow;
}

// Do zsub of the n2 cells along the z extent hz span the cutoff?  n2 came from
// the width V / |a x b|, which may round a few ulp above hz: boxes of edge
// (3000 / 3)^(1/3) = 10 - 1 ulp have twenty cells in 13% of their deformed
// shapes.  An exact comparison took those for flat, and the one-lane search
// advanced by one record instead of four: 400 boxes of 1029 particles, 20
// steps, 2134 us against 1682 at the whole edge, and 1736 with this rule.
// A pair 1e-12 short of the cutoff has a weight of 1e-12.
__host__ __device__ inline bool z_cells_span(double hz, int zsub, int n2, double rc) {
    return hz * zsub >= rc * n2 * (1.0 - 1e-12);
}

// Tiles of the macro problem's gx x gy cells: `rows` cells of a column and the
// ring around them, a workgroup each.  About as many as CUs; a tile holds 64
// cells with its ring at most (19 rows), and covers each of a column's cells at
// most once with it, so the largest grids have up to 1060.  Columns run along y,
// or along x (turned) where a long grid would have more columns than CUs: each
// workgroup reads all particles' cells, and of 5000 x 3 cells it takes 15000 in
// columns along y (308 us a step of 1300 particles) and 792 along x (45 us).
constexpr int TILES = 256;
constexpr int TILE_CELLS = 64;

struct CellTiles {
    bool turned;     // cell columns run along x
    int ncol, nrow;  // columns, cells of a column
    int rows, tiles; // cells of a column per tile, tiles per column
};

inline CellTiles cell_tiles(int gx, int gy) {
    CellTiles t;
    t.turned = gx > TILES && gx > gy;
    t.ncol = t.turned ? gy : gx;
    t.nrow = t.turned ? gx : gy;
    const int per_column = std::max(1, TILES / t.ncol);
    t.rows = std::min({(t.nrow + per_column - 1) / per_column, t.nrow - 2, TILE_CELLS / 3 - 2});
    t.tiles = (t.nrow + t.rows - 1) / t.rows;
    return t;
}

#endif
