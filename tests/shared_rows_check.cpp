// Drives the agreement on shared rows with threads in place of waves: shared_rows_check <name of a check>; exit code 0: it holds.
#include "../paper_2106_16064_amd/csrc/shared_rows.hpp"

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>

namespace {

using dgsp::RowWord;

struct Words {
    static RowWord load(RowWord* p) { return __atomic_load_n(p, __ATOMIC_SEQ_CST); }
    static void store(RowWord* p, RowWord v) { __atomic_store_n(p, v, __ATOMIC_SEQ_CST); }
    static RowWord exchange(RowWord* p, RowWord v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
    static bool replace(RowWord* p, RowWord& seen, RowWord v) {
        return __atomic_compare_exchange_n(p, &seen, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST);
    }
    static void pause() { std::this_thread::yield(); }
};

struct Row {
    RowWord word;
    std::atomic<long> sum;
};

// the wave that the row starts in: `late` steps after the others
void start(Row& row, RowWord call, int late, long part) {
    for (int i = 0; i < late; ++i) std::this_thread::yield();
    const RowWord found = dgsp::claim_row<Words>(&row.word, call);
    if (dgsp::mine_to_clear(found, call)) row.sum.store(0);
    dgsp::publish_start<Words>(&row.word, call, found);
    if (dgsp::row_has_sum<Words>(&row.word, call)) row.sum.fetch_add(part);
    else std::_Exit(2);                                  // it has just been published
}

void give(Row& row, RowWord call, long part) {
    if (dgsp::row_has_sum<Words>(&row.word, call)) {
        row.sum.fetch_add(part);
    } else {
        row.sum.store(part);
        dgsp::publish_part<Words>(&row.word, call);
    }
}

// Every part once and nothing else, whoever comes first, on words and rows that earlier calls have left behind.
bool every_part_once(int late) {
    constexpr int kParts = 6;
    Row row;
    row.word = 0x123456789abcdefull;
    row.sum = -77;
    for (RowWord call = 1000; call < 1000 + 2 * 1500; call += 2) {
        std::vector<std::thread> waves;
        long expected = 0;
        for (int i = 0; i < kParts; ++i) {
            const long part = 1l << (8 * i);
            expected += part;
            if (i == 0) waves.emplace_back([&row, call, late, part] { start(row, call, late, part); });
            else waves.emplace_back([&row, call, part] { give(row, call, part); });
        }
        for (auto& w : waves) w.join();
        if (row.sum != expected || row.word != call + 1) return false;
        if (call % 3 == 0) { row.word = call + 3 * call; row.sum = 5; }        // somebody else's memory
    }
    return true;
}

// Every order of whole steps for one part and the wave that the row starts in.
bool in_turn() {
    for (int order = 0; order < 2; ++order) {
        Row row;
        row.word = 7;
        row.sum = 1000;
        if (order == 0) { start(row, 40, 0, 3); give(row, 40, 5); }
        else { give(row, 40, 5); start(row, 40, 0, 3); }
        if (row.sum != 8 || row.word != 41) return false;
    }
    return true;
}

// A claim is published whether there is a row to clear or not, except where somebody else holds the word and will.
bool every_claim_ends() {
    for (const RowWord before : {0ull, 41ull, 39ull, ~0ull}) {
        RowWord word = before;
        const RowWord found = dgsp::claim_row<Words>(&word, 40);
        dgsp::publish_start<Words>(&word, 40, found);
        if (word != 41) return false;
    }
    RowWord word = 40;                                   // claimed by a part
    const RowWord found = dgsp::claim_row<Words>(&word, 40);
    dgsp::publish_start<Words>(&word, 40, found);
    if (word != 40 || dgsp::mine_to_clear(found, 40)) return false;
    dgsp::publish_part<Words>(&word, 40);
    return word == 41;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    if (!strcmp(argv[1], "every_part_once")) return every_part_once(0) ? 0 : 1;
    if (!strcmp(argv[1], "the_start_comes_late")) return every_part_once(200) ? 0 : 1;
    if (!strcmp(argv[1], "in_turn")) return in_turn() ? 0 : 1;
    if (!strcmp(argv[1], "every_claim_ends")) return every_claim_ends() ? 0 : 1;
    return 2;
}
