// How the balanced kernels share out the nnz + M merge-path items (host code too, so that it can be tried without a GPU).
#pragma once

#include "host_device.hpp"

namespace dgsp {

// The even split of the Q quanta into `parts` chunks: chunk c starts at quantum floor(c * Q / parts),
// so chunks differ by at most one quantum and the longer ones are spread over the whole list (put
// first, they would all fall to the first XCDs).  The quotients are formed in fp64: numerators stay
// below 2^53 and a non-integer quotient n / m lies at least 1 / m away from an integer, far more than
// the rounding of one correctly rounded division, so the floors are exact - and much cheaper here
// than 64-bit integer division, which the per-row test of the prepare kernel would pay twice.
struct EvenSplit {
    unsigned Q, parts, shift;     // quanta, chunks, log2 of the quantum
    DGSP_HOST_DEVICE EvenSplit(unsigned items, unsigned parts_, unsigned quantum_log2) {
        const unsigned quantum = 1u << quantum_log2;
        Q = (items >> quantum_log2) + ((items & (quantum - 1)) != 0);
        parts = parts_;
        shift = quantum_log2;
    }
    // first item of chunk c (c may be `parts`: the end of the list, rounded up to a quantum)
    DGSP_HOST_DEVICE unsigned start(unsigned c) const {
        const double n = (double)((unsigned long long)c * Q);
        return (unsigned)(n / (double)parts) << shift;
    }
    // chunk that holds item d: the largest c with floor(c * Q / parts) <= d's quantum
    DGSP_HOST_DEVICE unsigned chunk_of(unsigned d) const {
        const unsigned long long q = d >> shift;
        const double n = (double)((q + 1) * parts - 1);
        return (unsigned)(n / (double)Q);
    }
};

// How a call with a workspace shares out the items (nb_sr_run_kernel).  `chunks` chunks of 2^size_log2 items are dealt to
// `parts` parts, one per XCD that works on a list.  The first chunks of a part are its waves' shares, `run` consecutive ones a
// wave, a single piece; the others are taken one by one by whoever is done, first from the wave's own part.  In the
// workspace: `taken`, a counter for each XCD's queue, kQueuePitch words apart, and `starts`, for each chunk and for the end of the
// list the number of rows that ended before it, which saves the waves their searches.
constexpr unsigned kQueuePitch = 32;
struct ChunkQueues {
    unsigned* taken; int* starts;
    unsigned chunks, size_log2, counters, parts_log2, waves, run, helpers, fewest, fewest_a_row;
    float parts_per_chunk, per_run;                      // 2^parts_log2 / chunks, 1 / run
    // at most 2^23 chunks, 8 parts
    DGSP_HOST_DEVICE unsigned part_from(unsigned part) const { return (chunks * part) >> parts_log2; }
    DGSP_HOST_DEVICE unsigned queue_from(unsigned part) const { return part_from(part) + waves * run; }
    // The host counts with a bound of the entries where it does not know them.  Fewer items: fewer chunks of the same size, and shorter
    // first pieces to the same share - or, where the host would not have chosen queues had it known (`fewest` items, `fewest_a_row`
    // entries a row), equal shares for all waves, as without queues: run = 0, a chunk a wave, even to 64 items (without queues to 32:
    // kRunQuantumLog2).  Arrays twice / four times / eight times as long as the matrix, queues all the same -> equal shares: R-MAT
    // 2^18 x 16 at N = 64 86 / 94 / 100 -> 86 / 89 / 89 us, 2^20 x 6 at N = 50 216 / 224 / 224 -> 205 us, Zipf rows of 16 at N = 64
    // 164 / 173 / 173 -> 165 us, of 10 at N = 100 403 / 423 / 423 -> 415 us, lognormal rows of 20 at N = 100 433 / 438 / 439 -> 440 us;
    // the line is the same as for calls that know the count.
    DGSP_HOST_DEVICE void fit(unsigned items, unsigned rows) {
        const unsigned quanta = EvenSplit(items, 1u, size_log2).Q;
        if (items >= fewest && items - rows >= (unsigned long long)fewest_a_row * rows) {
            if (quanta >= chunks) return;
            run = (unsigned)((float)run * ((float)quanta / (float)chunks));
        } else {
            run = 0u;
        }
        if (run != 0u) {
            chunks = quanta;
            parts_per_chunk = (float)(1u << parts_log2) / (float)chunks;
            per_run = 1.0f / (float)run;
        } else {
            size_log2 = 6u;
            const unsigned all = waves << parts_log2, most = EvenSplit(items, 1u, size_log2).Q;
            chunks = most < all ? most : all;
        }
    }
    // do chunks c1 and c2 >= c1 belong to one piece?  (c2 in a queue, or equal shares: a piece is a chunk; else no multiple of `run`
    // lies behind c1)
    DGSP_HOST_DEVICE bool one_piece(unsigned c1, unsigned c2) const {
        unsigned part = (unsigned)((float)c2 * parts_per_chunk);            // one off at most
        if (part_from(part + 1u) <= c2) ++part;
        else if (part_from(part) > c2) --part;
        const unsigned at = c2 - part_from(part);
        if (at >= waves * run) return c1 == c2;
        unsigned into = at - (unsigned)((float)at * per_run) * run;         // into the piece: at % run
        if ((int)into < 0) into += run;
        else if (into >= run) into -= run;
        return c2 - c1 <= into;
    }
};

}  // namespace dgsp
