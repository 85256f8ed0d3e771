// Tries how the items are shared out without a GPU: chunk_queues_check <name of a check>; exit code 0: it holds.
#include "../paper_2106_16064_amd/csrc/chunk_queues.hpp"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <random>
#include <vector>

namespace {

using dgsp::ChunkQueues;
using dgsp::EvenSplit;

std::mt19937 g_random(11);
unsigned between(unsigned lo, unsigned hi) { return std::uniform_int_distribution<unsigned>(lo, hi)(g_random); }

// Queues over `items` items as the host counts them, with a first piece of about half a share.
ChunkQueues queues_for(unsigned items, unsigned parts_log2, unsigned waves, unsigned size_log2, unsigned fewest, unsigned a_row) {
    ChunkQueues q{};
    q.size_log2 = size_log2;
    q.chunks = EvenSplit(items, 1u, size_log2).Q;
    q.parts_log2 = parts_log2;
    q.waves = waves;
    q.run = (unsigned)((q.chunks >> parts_log2) * 0.55 / waves);
    q.parts_per_chunk = (float)(1u << parts_log2) / (float)q.chunks;
    q.per_run = 1.0f / (float)q.run;
    q.fewest = fewest;
    q.fewest_a_row = a_row;
    return q;
}

// Every chunk's piece, by counting.
std::vector<unsigned> pieces_of(const ChunkQueues& q) {
    std::vector<unsigned> piece(q.chunks);
    unsigned n = 0;
    if (q.run == 0) {
        for (unsigned c = 0; c < q.chunks; ++c) piece[c] = n++;
        return piece;
    }
    for (unsigned part = 0; part < 1u << q.parts_log2; ++part) {
        unsigned c = q.part_from(part);
        for (unsigned w = 0; w < q.waves; ++w, ++n)
            for (unsigned i = 0; i < q.run; ++i) piece[c++] = n;
        for (; c < q.part_from(part + 1); ++c) piece[c] = n++;
    }
    return piece;
}

bool pieces_agree(const ChunkQueues& q) {
    for (unsigned part = 0; part < 1u << q.parts_log2 && q.run != 0; ++part)
        if (q.queue_from(part) > q.part_from(part + 1)) return false;
    const std::vector<unsigned> piece = pieces_of(q);
    const unsigned ahead = std::max(q.run, 1u) + 1;
    for (unsigned c = 0; c < q.chunks; c += q.chunks > 100000 ? between(1, 40) : 1) {
        for (unsigned d = 0; d <= ahead && c + d < q.chunks; d += ahead > 40 ? between(1, ahead / 8) : 1)
            if (q.one_piece(c, c + d) != (piece[c] == piece[c + d])) return false;
        const unsigned far = between(c, q.chunks - 1);
        if (q.one_piece(c, far) != (piece[c] == piece[far])) return false;
    }
    return true;
}

// Chunks that belong together are told by arithmetic in single precision, up to 2^23 of them.
bool pieces() {
    for (int i = 0; i < 120; ++i) {
        const unsigned parts_log2 = between(0, 3), waves = between(1, 512), all = waves << parts_log2;
        const unsigned a_wave = between(4, std::max(5u, std::min(4000u, ((1u << 23) - 1) / all)));
        const unsigned chunks = std::min((1u << 23) - 1, all * a_wave + between(0, all));
        ChunkQueues q = queues_for(chunks * 512u - between(0, 511), parts_log2, waves, 9, 0, 0);
        if (q.run == 0) return false;
        if (!pieces_agree(q)) return printf("%u chunks in 2^%u parts, %u waves\n", q.chunks, parts_log2, waves), false;
    }
    return true;
}

// The host's bound is longer than the matrix: as many chunks as there are, first pieces to the same share; and equal shares
// where a wave's share is below the line, or the rows have too few entries for it.
bool fits() {
    for (int i = 0; i < 600; ++i) {
        const unsigned parts_log2 = between(0, 3), waves = between(64, 512), all = waves << parts_log2;
        const unsigned bound = std::min(2100000000u, all * between(2048, 40000)), fewest = all * 2048u, a_row = i % 2 ? 6 : 8;
        const unsigned items = i % 7 == 0 ? between(1, 200) : (unsigned)((double)bound * between(1, 1000) / 1000.0) + 1u;
        const unsigned rows = std::max(1u, (unsigned)((double)items / between(3, 20)));
        const ChunkQueues before = queues_for(bound, parts_log2, waves, bound / all >= 4096 ? 10 : 9, fewest, a_row);
        ChunkQueues q = before;
        q.fit(items, rows);
        if (q.chunks > before.chunks) return false;                      // the list of first rows has room for no more
        const bool queues = items >= fewest && (items - rows) / rows >= a_row;
        if (!queues && q.run != 0) return printf("queues for %u items, %u rows\n", items, rows), false;
        if (queues && q.run == 0 && before.run * (double)items / bound >= 1.1) return false;
        if (q.run == 0 && (q.chunks > all || q.size_log2 != 6 || (q.chunks < all && q.chunks != (items + 63) / 64))) return false;
        if (EvenSplit(items, q.chunks, q.size_log2).start(q.chunks) < items) return false;
        if (!pieces_agree(q)) return false;
    }
    // the matrix as the host had it: nothing changes
    ChunkQueues q = queues_for(9000000, 3, 512, 9, 8 * 512 * 2048, 6);
    const unsigned chunks = q.chunks, run = q.run;
    q.fit(9000000, 500000);
    return q.chunks == chunks && q.run == run && q.size_log2 == 9;
}

// The even split: chunks in order, each item in the chunk that holds it.
bool even_split() {
    for (int i = 0; i < 3000; ++i) {
        const unsigned items = i % 3 == 0 ? between(1, 5000) : between(1, 4000000000u), parts = between(1, i % 2 ? 5000 : 70);
        const EvenSplit s(items, parts, between(5, 10));
        if (s.start(0) != 0) return false;
        for (unsigned c = 0; c < parts; c += between(1, parts / 64 + 1)) {
            const unsigned long long from = (unsigned long long)c * s.Q / parts << s.shift, to = (unsigned long long)(c + 1) * s.Q / parts << s.shift;
            if (s.start(c) != (unsigned)from) return false;
            if (from == to) continue;                                    // a chunk without items
            for (const unsigned long long d : {from, (from + to) / 2, to - 1})
                if (d < items && s.chunk_of((unsigned)d) != c) return false;
        }
    }
    return true;
}

}  // namespace

int main(int argc, char** argv) {
    const char* name = argc > 1 ? argv[1] : "";
    if (!strcmp(name, "pieces")) return pieces() ? 0 : 1;
    if (!strcmp(name, "fits")) return fits() ? 0 : 1;
    if (!strcmp(name, "even_split")) return even_split() ? 0 : 1;
    fprintf(stderr, "unknown check %s\n", name);
    return 2;
}
