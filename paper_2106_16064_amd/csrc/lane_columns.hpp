// The V dense columns of a lane in the sequential-reduction kernels (host code too, so that it can be tried without a GPU).
//
// Column block `block` covers `cols_per_block` columns (a multiple of V, at most G * V) from block * cols_per_block;
// lane `gl` of a group normally owns [first, first + V) with first = block * cols_per_block + gl * V.  RAGGED (N is
// not a multiple of V, N >= V): the lane whose window would pass N takes the last V columns of the row instead, so
// that every load stays inside the row; `skip` of them also belong to its left neighbour, which computes the same
// sums from the same entries in the same order - the lane keeps them out of what it adds to memory, of the
// scaled form's stores and of what it puts under sums that waves add up: where the last block has fewer than V columns that
// neighbour is in another block, with waves of its own.  Plain stores of finished sums may repeat them: the bits are the same.
#pragma once

#include "host_device.hpp"

namespace dgsp {

struct LaneColumns {
    long long first;    // first column of the window
    int skip;           // leading columns of the window that are the neighbour's (0 < skip < V on one lane at most)
    bool any;           // the lane has columns at all
};
template <int V, bool RAGGED>
DGSP_HOST_DEVICE LaneColumns lane_columns(unsigned block, int cols_per_block, int gl, int N) {
    LaneColumns c;
    c.first = (long long)block * cols_per_block + gl * V;
    c.skip = 0;
    c.any = gl * V < cols_per_block && c.first < N;
    if constexpr (RAGGED) {
        if (c.any && c.first + V > N) { c.skip = (int)(c.first + V - N); c.first = (long long)N - V; }
    }
    return c;
}

}  // namespace dgsp
