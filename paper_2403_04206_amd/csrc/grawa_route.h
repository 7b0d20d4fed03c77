// Launch shapes of the center+pull pass (host side).  Plain C++ with no GPU dependency, so that the rules can be
// checked on the CPU for sizes that no test allocates.
#ifndef GRAWA_ROUTE_H
#define GRAWA_ROUTE_H

#include <stdint.h>

// Grid of the row-split form, one block per 256-column cell.  Its blocks have 1024 threads and a launch takes fewer
// than 2^32 threads in x, which one row of blocks would exceed from 2^30 columns on (plans go to 2^32).  So the cells
// are cut into rows of at most 2^18 blocks, all of nearly the same length; fewer than gy blocks at the end hold no
// cell.  Up to 2^18 cells (67 M columns) the grid is one row; the limit is far below 2^22 so that a second row is
// reached at sizes that tests can hold.
#define GRAWA_SPLIT_THREADS 1024
#define GRAWA_SPLIT_ROW_BLOCKS ((int64_t)1 << 18)
static inline void grawa_split_grid(int64_t n_cells, unsigned *gx, unsigned *gy)
{
    const int64_t rows = (n_cells + GRAWA_SPLIT_ROW_BLOCKS - 1) / GRAWA_SPLIT_ROW_BLOCKS;
    *gy = (unsigned)rows;
    *gx = (unsigned)((n_cells + rows - 1) / rows);
}

#endif
