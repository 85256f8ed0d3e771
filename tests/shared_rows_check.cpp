// Drives the agreement on shared rows with threads in place of waves: shared_rows_check <name of a check>; exit code 0: it holds.
#include "../paper_2106_16064_amd/csrc/call_numbers.hpp"
#include "../paper_2106_16064_amd/csrc/lane_columns.hpp"
#include "../paper_2106_16064_amd/csrc/shared_rows.hpp"

#include <algorithm>
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
    static void put(float* p, float v) { *p = v; }
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

// Waves of a workgroup that meet at a barrier between their claims and their publications, as where they fill LDS together.
struct Meeting {
    std::atomic<int> missing;
    explicit Meeting(int waves) : missing(waves) {}
    void meet() {
        for (--missing; missing.load() > 0;) std::this_thread::yield();
    }
};

// A list of chunks, a wave each, whose last row goes on in the next chunk: workgroups that start all at once, or one only when the one
// before it - or behind it - has ended, which is when nobody may wait for waves that have not started.
bool workgroups_that_meet() {
    constexpr int kGroups = 5, kWaves = 3, kChunks = kGroups * kWaves;
    for (RowWord call = 1000; call < 1000 + 2 * 300; call += 2) {
        std::vector<Row> rows(kChunks);
        for (Row& r : rows) { r.word = 7 * call; r.sum = -9; }
        const auto wave = [&](int chunk, Meeting& meeting) {
            Row& mine = rows[chunk];
            const RowWord found = dgsp::claim_row<Words>(&mine.word, call);
            if (dgsp::mine_to_clear(found, call)) mine.sum.store(0);
            meeting.meet();
            dgsp::publish_start<Words>(&mine.word, call, found);
            if (chunk > 0) give(rows[chunk - 1], call, 100);
            give(mine, call, 1);
        };
        const auto group = [&](int g) {
            Meeting meeting(kWaves);
            std::vector<std::thread> waves;
            for (int w = 0; w < kWaves; ++w) waves.emplace_back([&, w] { wave(g * kWaves + w, meeting); });
            for (auto& w : waves) w.join();
        };
        if (call % 6 == 4) {
            std::vector<std::thread> groups;
            for (int g = 0; g < kGroups; ++g) groups.emplace_back([&, g] { group(g); });
            for (auto& g : groups) g.join();
        } else {
            for (int g = 0; g < kGroups; ++g) group(call % 6 == 0 ? g : kGroups - 1 - g);
        }
        for (int c = 0; c < kChunks; ++c)
            if (rows[c].sum != (c + 1 < kChunks ? 101 : 1) || rows[c].word != call + 1) return false;
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

// A row of N columns in column blocks of `per`, each with a word of its own: the wave that the row starts in and one more wave a block.
struct BlockedRow {
    int N, per;
    float beta;
    std::vector<float> y;
    std::vector<RowWord> words;
    static constexpr RowWord kCall = 40;

    BlockedRow(int N, int per, float beta) : N(N), per(per), beta(beta), y(N), words((N + per - 1) / per, 7) {
        for (int n = 0; n < N; ++n) y[n] = beta == 0.0f ? NAN : (float)(8 * n);
    }
    template <typename F>
    void lanes(unsigned block, F&& f) {
        for (int gl = 0; gl * 4 < per; ++gl) {
            const dgsp::LaneColumns c = dgsp::lane_columns<4, true>(block, per, gl, N);
            if (c.any) f(c);
        }
    }
    void start(unsigned block) {
        const RowWord found = dgsp::claim_row<Words>(&words[block], kCall);
        if (dgsp::mine_to_clear(found, kCall))
            lanes(block, [&](const dgsp::LaneColumns& c) { dgsp::clear_row<Words, 4, true>(&y[c.first], beta, c.skip); });
        dgsp::publish_start<Words>(&words[block], kCall, found);
    }
    void give(unsigned block, float part) {
        const bool sum = dgsp::row_has_sum<Words>(&words[block], kCall);
        lanes(block, [&](const dgsp::LaneColumns& c) {
            float v[4];
            for (int i = 0; i < 4; ++i) v[i] = part * (float)(c.first + i + 1);
            if (!sum) dgsp::write_part<Words, 4, true>(&y[c.first], v, beta, c.skip);
            else for (int i = c.skip; i < 4; ++i) y[c.first + i] += v[i];
        });
        if (!sum) dgsp::publish_part<Words>(&words[block], kCall);
    }
    bool whole(float sum) const {
        for (int n = 0; n < N; ++n)
            if (y[n] != (beta == 0.0f ? 0.0f : beta * (float)(8 * n)) + sum * (float)(n + 1)) return false;
        return true;
    }
};

// Every order of the steps of the last two column blocks, the last with one to four columns, with the start first or not.
bool ragged_blocks() {
    for (int N = 9; N <= 16; ++N)
        for (const float beta : {0.0f, 0.5f})
            for (int late = 0; late < 4; ++late) {               // bit b: in block b a part comes before the start
                int order[] = {0, 0, 0, 1, 1, 1};
                do {
                    BlockedRow row(N, 8, beta);
                    int step[2] = {0, 0};
                    for (const int b : order) {
                        const int s = step[b]++;
                        const int what = (late >> b & 1) ? (s == 0 ? 1 : s == 1 ? 0 : 2) : s;
                        if (what == 0) row.start((unsigned)b); else row.give((unsigned)b, what == 1 ? 3.0f : 5.0f);
                    }
                    if (!row.whole(8.0f)) return false;
                } while (std::next_permutation(order, order + 6));
            }
    return true;
}

// Even numbers, one after the other and none twice; without random bytes, too, and nothing is thrown.
bool call_numbers() {
    const RowWord first = dgsp::next_call_number(), second = dgsp::next_call_number();
    if (first % 2 != 0 || second != first + 2) return false;
    if (dgsp::first_call_number([](void* p, size_t n) { memset(p, 0xff, n); return true; }) != ~1ull) return false;
    const auto none = [](void*, size_t) { return false; };
    const RowWord one = dgsp::first_call_number(none), other = dgsp::first_call_number(none);
    return one % 2 == 0 && other % 2 == 0 && one != other && one != first;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    if (!strcmp(argv[1], "every_part_once")) return every_part_once(0) ? 0 : 1;
    if (!strcmp(argv[1], "the_start_comes_late")) return every_part_once(200) ? 0 : 1;
    if (!strcmp(argv[1], "in_turn")) return in_turn() ? 0 : 1;
    if (!strcmp(argv[1], "ragged_blocks")) return ragged_blocks() ? 0 : 1;
    if (!strcmp(argv[1], "call_numbers")) return call_numbers() ? 0 : 1;
    if (!strcmp(argv[1], "workgroups_that_meet")) return workgroups_that_meet() ? 0 : 1;
    if (!strcmp(argv[1], "every_claim_ends")) return every_claim_ends() ? 0 : 1;
    return 2;
}
