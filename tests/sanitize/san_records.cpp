// The shares of slices that several chunks of the MTTKRP record stream hold (csrc/record_shares.hpp): lists made as the
// plan makes them pass, and every single mistake planted in them is found.
#include <cstdio>
#include <random>
#include <vector>

#include "record_shares.hpp"

using namespace cst;

struct Stream {
    std::vector<int64_t> slice_rec;
    std::vector<int32_t> row;
    int64_t q;
    std::vector<RecordShare> list[3];      // by kind; [0] stays empty

    int64_t slices() const { return int64_t(row.size()); }
    bool right() const {                   // what the plan check asks of every slice and of every entry
        for (int64_t s = 0; s < slices(); ++s) {
            const int kind = share_of(slice_rec.data(), s, q);
            if (kind && !share_listed(list[kind].data(), int64_t(list[kind].size()), record_share(slice_rec.data(), s, q, row[size_t(s)])))
                return false;
        }
        for (int kind = 1; kind < 3; ++kind)
            for (int64_t e = 0; e < int64_t(list[kind].size()); ++e)
                if (!share_entry_right(list[kind].data(), e, kind, slice_rec.data(), slices(), slice_rec.back(), q, row.data())) return false;
        return true;
    }
};

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    std::mt19937 rng(7);
    for (int round = 0; round < 300; ++round) {
        Stream t;
        t.q = 16 * (1 + int64_t(rng() % 4));
        const int64_t n = 1 + int64_t(rng() % 40);
        t.slice_rec.push_back(0);
        for (int64_t s = 0; s < n; ++s) {
            // inside a chunk, up to its very end, a few chunks, many
            const int64_t len[] = {1 + int64_t(rng() % 20), t.q - t.slice_rec.back() % t.q, t.q * (1 + int64_t(rng() % 5)),
                                   t.q * (kRecLight - 1 + int64_t(rng() % 3)) + int64_t(rng() % 7)};
            t.slice_rec.push_back(t.slice_rec.back() + len[rng() % 4]);
            t.row.push_back(int32_t(3 * s + int64_t(rng() % 3)));
        }
        for (int64_t s = 0; s < n; ++s) {
            const int kind = share_of(t.slice_rec.data(), s, t.q);
            if (kind) t.list[kind].push_back(record_share(t.slice_rec.data(), s, t.q, t.row[size_t(s)]));
        }
        CHECK(t.right());
        for (int kind = 1; kind < 3; ++kind)
            for (size_t e = 0; e < t.list[kind].size(); ++e) {
                const RecordShare was = t.list[kind][e];
                for (int64_t d : {-2, -1, 1, 2}) {
                    t.list[kind][e].first = was.first + d;
                    CHECK(!t.right());
                }
                for (int64_t far : {int64_t(-1), INT64_MAX, INT64_MIN, int64_t(1) << 40}) {
                    t.list[kind][e].first = far;
                    CHECK(!t.right());
                }
                t.list[kind][e] = was;
                for (int d : {-1, 1}) {
                    t.list[kind][e].count = was.count + d;
                    CHECK(!t.right());
                    t.list[kind][e] = was;
                    t.list[kind][e].row = was.row + d;
                    CHECK(!t.right());
                    t.list[kind][e] = was;
                }
                t.list[kind].erase(t.list[kind].begin() + long(e));                      // left out
                CHECK(!t.right());
                t.list[3 - kind].push_back(was);                                         // in the other list
                CHECK(!t.right());
                t.list[3 - kind].pop_back();
                t.list[kind].insert(t.list[kind].begin() + long(e), 2, was);             // twice
                CHECK(!t.right());
                t.list[kind].erase(t.list[kind].begin() + long(e));
                CHECK(t.right());
            }
    }
    std::printf("san_records: ok\n");
    return 0;
}
