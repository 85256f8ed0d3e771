// Rows that several waves hold parts of: who writes, who adds (host code too, so that it can be tried without a GPU).
//
// The waves of a balanced kernel start together, and the sum of a row whose entries lie in several chunks is added up in Y with
// atomics.  Something has to be there to add to.  A launch in front of the kernel that clears these rows takes 5 us, as
// long as many a product; here the waves agree on it among themselves.  A row's word goes from anything else to `call` (somebody
// is writing the row) to `call + 1` (the row holds a sum, add to it).  The wave that the row starts in claims the word before
// it does anything else and writes zeros when it knows its rows; who comes to such a row before that wave has even
// started, because the machine is busy with other launches, writes its own part instead.
//
// Nobody waits for a wave that has not started: a word is `call` only between a claim and the same wave's publish(), and in
// between no wave waits for another workgroup's.  The waves of one workgroup start together, so they may meet at a barrier
// there which all of them reach without waiting for anything else (nb_pr_kernel with hot runs).  Every claim is published, whether
// there turns out to be a row or not, so a wait ends for any contents of the row pointers.
//
// `call` is even and of no other call of the process (next_call_number()), so that the words need no clearing: memory that other
// kernels or other processes have used holds one of the two numbers with a chance of 2^-62 a word.
//
// `Ops` accesses words that all waves see: load(p), store(p, v), exchange(p, v), replace(p, seen, v) - compare and swap
// which leaves what it found in `seen` -, and pause(); put(y, v) stores a float so that all waves find it behind the word's publication.
#pragma once

#include "host_device.hpp"

#include <cmath>

namespace dgsp {

using RowWord = unsigned long long;

// The wave that the row starts in: what it found, for mine_to_clear() and publish_start().
template <typename Ops>
DGSP_HOST_DEVICE RowWord claim_row(RowWord* word, RowWord call) { return Ops::exchange(word, call); }

// Is the row mine to clear?  (Otherwise somebody has come before me.)
DGSP_HOST_DEVICE bool mine_to_clear(RowWord found, RowWord call) { return found != call && found != call + 1; }

// Once the zeros are in memory, or the row is not mine to clear.  Whoever has claimed the row before me publishes it himself.
template <typename Ops>
DGSP_HOST_DEVICE void publish_start(RowWord* word, RowWord call, RowWord found) {
    if (found != call) Ops::store(word, call + 1);
}

// A wave with a part of the row, which has `seen` the word.  True: there is a sum to add to.  False: the part is the first one, to be
// written and then published.
template <typename Ops>
DGSP_HOST_DEVICE bool row_has_sum(RowWord* word, RowWord call, RowWord seen) {
    for (;;) {
        if (seen == call + 1) return true;
        if (seen == call) {
            Ops::pause();
            seen = Ops::load(word);
        } else if (Ops::replace(word, seen, call)) {
            return false;
        }
    }
}
template <typename Ops>
DGSP_HOST_DEVICE bool row_has_sum(RowWord* word, RowWord call) { return row_has_sum<Ops>(word, call, Ops::load(word)); }
template <typename Ops>
DGSP_HOST_DEVICE void publish_part(RowWord* word, RowWord call) { Ops::store(word, call + 1); }

// Zeros, or the old values times beta, for the parts of a row to be added to (claim_row()): V columns of a lane.  The first `skip` are left
// alone: they are another lane's, which may be in another column block and have sums there already (lane_columns()).
template <typename Ops, int V, bool AXPBY>
DGSP_HOST_DEVICE void clear_row(float* y, float beta, int skip = 0) {
    float old[V];
#pragma unroll
    for (int i = 0; i < V; ++i) old[i] = AXPBY && beta != 0.0f ? y[i] : 0.0f;
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (i >= skip) Ops::put(y + i, AXPBY && beta != 0.0f ? beta * old[i] : 0.0f);
}
// The first part of a row (row_has_sum()), times alpha already, on what beta leaves of the old values; `skip` as above.
template <typename Ops, int V, bool AXPBY>
DGSP_HOST_DEVICE void write_part(float* y, const float (&v)[V], float beta, int skip = 0) {
    float old[V];
#pragma unroll
    for (int i = 0; i < V; ++i) old[i] = AXPBY && beta != 0.0f ? y[i] : 0.0f;
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (i >= skip) Ops::put(y + i, AXPBY && beta != 0.0f ? fmaf(beta, old[i], v[i]) : v[i]);
}

}  // namespace dgsp
