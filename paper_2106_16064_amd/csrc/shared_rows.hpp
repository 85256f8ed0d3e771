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
// between no wave waits for another.  Every claim is published, whether there turns out to be a row or not, so a wait ends for
// any contents of the row pointers.
//
// `call` is even and no other call's, so that the words need no clearing: memory that other kernels have used holds one of the two
// numbers with a chance of 2^-62 a word.
//
// `Ops` accesses words that all waves see: load(p), store(p, v), exchange(p, v), replace(p, seen, v) - compare and swap
// which leaves what it found in `seen` -, and pause().
#pragma once

#if defined(__HIPCC__)
#define DGSP_SHARED_ROWS_FN __host__ __device__ inline
#else
#define DGSP_SHARED_ROWS_FN inline
#endif

namespace dgsp {

using RowWord = unsigned long long;

// The wave that the row starts in: what it found, for start_row().
template <typename Ops>
DGSP_SHARED_ROWS_FN RowWord claim_row(RowWord* word, RowWord call) { return Ops::exchange(word, call); }

// Is the row mine to clear?  (Otherwise somebody has come before me.)
DGSP_SHARED_ROWS_FN bool mine_to_clear(RowWord found, RowWord call) { return found != call && found != call + 1; }

// Once the zeros are in memory, or the row is not mine to clear.  Whoever has claimed the row before me publishes it himself.
template <typename Ops>
DGSP_SHARED_ROWS_FN void publish_start(RowWord* word, RowWord call, RowWord found) {
    if (found != call) Ops::store(word, call + 1);
}

// A wave with a part of the row.  True: there is a sum to add to.  False: the part is the first one, to be written and then published.
template <typename Ops>
DGSP_SHARED_ROWS_FN bool row_has_sum(RowWord* word, RowWord call) {
    RowWord seen = Ops::load(word);
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
DGSP_SHARED_ROWS_FN void publish_part(RowWord* word, RowWord call) { Ops::store(word, call + 1); }

}  // namespace dgsp
