// Driver of tests/test_search_plan.py: the room that search_plan.h gives a batched search, over a grid of calls and of
// indexes.  Prints what is wrong, or "ok".
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "search_plan.h"

using namespace ivftq;

namespace {

std::vector<int32_t> lists(const char* kind, int nlist, int64_t total) {
    std::mt19937_64 rng(nlist);
    std::vector<int32_t> size(nlist);
    for (int l = 0; l < nlist; ++l) {
        const double mean = (double)total / nlist;
        if (kind[0] == 's') size[l] = (int32_t)(mean * (0.7 + 0.6 * (rng() % 1000) / 1000.0));      // spread around the mean
        if (kind[0] == 'h') size[l] = l == nlist / 2 ? (int32_t)(total - nlist) : 1;                // one hot list
        if (kind[0] == 'e') size[l] = l % 3 == 0 ? (int32_t)(3 * mean) : 0;                          // most of them empty
    }
    return size;
}

// Tiles of a pass whose pairs meet list l pairs_of[l] times, as the grouping makes them.
int64_t tiles_of(const std::vector<int32_t>& size, const std::vector<int64_t>& pairs_of, int tq, int part) {
    int64_t t = 0;
    for (size_t l = 0; l < size.size(); ++l)
        if (size[l] > 0) t += (pairs_of[l] + tq - 1) / tq * list_parts(size[l], part);
    return t;
}

// Score rows and per-query arrays: every smaller call (fewer queries, candidates a query or a shorter prefix; streamed where
// the larger one is batched) fits what the larger one was given, and a pass fits its own.
int check_rows() {
    struct Call { bool batched; int64_t nq, row, prefix; SearchRows r; };
    const int64_t nqs[] = {1, 2, 10, 11, 26, 27, 387, 388, 5368, 10'000, 32'768, 100'000};
    const int64_t coarse_rows[] = {16, 1024, 16'384}, limits[] = {1 << 20, 64 << 20, 4ll << 30};
    for (int64_t limit : limits)
        for (int64_t coarse : coarse_rows) {
            std::vector<Call> calls;
            for (int64_t row : {4, 1000, 9988, 10'000, 78'000, 100'004, 3'000'000})
                for (int64_t prefix : {200, 5000, 20'000})
                    for (int64_t nq : nqs)
                        for (bool batched : {false, true}) calls.push_back({batched, nq, row, prefix, search_rows(batched, nq, row, prefix, coarse, limit)});
            for (const Call& a : calls) {
                const SearchRows& r = a.r;
                const bool fits = r.queries >= 1 && r.queries <= a.nq && r.queries <= r.held && r.queries * r.stride <= r.floats &&
                                  (!a.batched || (r.gate_rows >= 1 && r.gate_rows <= r.queries && r.gate_rows * 2 * a.row <= r.floats));
                const bool limited = r.floats * 4 <= std::max(limit, 8 * a.row) && r.held * coarse * 4 <= std::max(limit, 4 * coarse);
                if (!fits || !limited) {
                    std::printf("limit %lld, %lld queries, rows of %lld: a pass does not fit its room\n", (long long)limit, (long long)a.nq, (long long)a.row);
                    return 1;
                }
                // the exact redo of `n` of a pass's queries, launch by launch: as many score rows as there are, and most workgroups at work
                for (int64_t n : {(int64_t)1, r.gate_rows - 1, r.gate_rows, r.gate_rows + 1, r.queries}) {
                    const int64_t window = redo_window(r.queries, r.gate_rows);
                    for (int64_t g0 = 0; a.batched && n <= r.queries && g0 < std::min(n, r.queries); g0 += window) {
                        const int64_t here = std::min(n - g0, window), per = std::max<int64_t>(1, kRedoWorkgroups / here);
                        const int64_t in_turn = std::min(here, kRedoWorkgroups / per);
                        if (in_turn > r.gate_rows || 2 * in_turn * per < kRedoWorkgroups) {
                            std::printf("%lld queries redone in %lld rows: %lld at a time by %lld workgroups each\n", (long long)n, (long long)r.gate_rows,
                                        (long long)in_turn, (long long)per);
                            return 1;
                        }
                    }
                }
                for (const Call& b : calls) {
                    if (b.nq > a.nq || b.row > a.row || b.prefix > a.prefix || (b.batched && !a.batched)) continue;
                    if (b.r.floats > r.floats || b.r.held > r.held) {
                        std::printf("limit %lld: %lld queries with rows of %lld (%s) need more than %lld with %lld (%s): %lld > %lld floats or %lld > %lld rows\n",
                                    (long long)limit, (long long)b.nq, (long long)b.row, b.batched ? "batched" : "streamed", (long long)a.nq,
                                    (long long)a.row, a.batched ? "batched" : "streamed", (long long)b.r.floats, (long long)r.floats,
                                    (long long)b.r.held, (long long)r.held);
                        return 1;
                    }
                }
            }
        }
    std::printf("ok\n");
    return 0;
}

// The tiles of a pass: every one in one queue's order once, and every queue with a workgroup.
int check_queues() {
    for (int resident : {1, 2, 8, 15, 16, 17, 20, 64, 256, 512})
        for (int q = 0; q < kTileQueues; ++q)
            if (queue_servers(tile_workgroups(resident), q) < 1) {
                std::printf("queue %d of a chip that holds %d workgroups is served by none\n", q, resident);
                return 1;
            }
    for (int tiles : {0, 1, 15, 16, 17, 1000, 32768}) {
        std::vector<int> seen(tiles, 0);
        for (int q = 0; q < kTileQueues; ++q)
            for (int j = 0; queue_tile(q, j) < tiles; ++j) ++seen[queue_tile(q, j)];
        for (int t = 0; t < tiles; ++t)
            if (seen[t] != 1) {
                std::printf("tile %d of %d is taken %d times\n", t, tiles, seen[t]);
                return 1;
            }
    }
    return 0;
}

}  // namespace

int main() {
    struct { const char* kind; int nlist; int64_t total; } const indexes[] = {
        {"spread", 4000, 10'000'000}, {"spread", 2000, 10'000'000}, {"spread", 64, 20'000}, {"spread", 16384, 40'000'000},
        {"hot", 4096, 10'000'000}, {"hot", 64, 1'000'000}, {"empty", 1000, 3'000'000}, {"spread", 300, 0}};
    const int nq[] = {1, 2, 3, 50, 51, 63, 64, 65, 127, 128, 129, 195, 196, 387, 388, 500, 1000, 4096, 10'000, 32'767, 32'768};
    const int np[] = {1, 2, 8, 31, 32, 33, 64};
    std::mt19937_64 rng(5);
    for (const auto& ix : indexes) {
        const std::vector<int32_t> size = lists(ix.kind, ix.nlist, ix.total);
        const ListRoom room = list_room(size.data(), ix.nlist), fine = list_room(size.data(), ix.nlist, kPartFine);
        const int64_t few = fine_pairs(ix.total, ix.nlist);
        for (int tq : {kBatchTileNear, kBatchTile}) {
            auto room_of = [&](int64_t q, int64_t pairs) {
                return tq == kBatchTileNear ? tile_room(room, q, pairs, tq) : late_tile_room(room, fine, few, q, pairs);
            };
            for (size_t a = 0; a < std::size(nq); ++a)
                for (size_t b = 0; b < std::size(np); ++b) {
                    const int64_t here = room_of(nq[a], (int64_t)nq[a] * np[b]);
                    const int64_t fewer_q = a ? room_of(nq[a - 1], (int64_t)nq[a - 1] * np[b]) : 0;
                    const int64_t fewer_p = b ? room_of(nq[a], (int64_t)nq[a] * np[b - 1]) : 0;
                    if (here < fewer_q || here < fewer_p) {
                        std::printf("%s nlist=%d tq=%d: %d queries x %d probes have room for %lld tiles, less than a smaller call (%lld, %lld)\n",
                                    ix.kind, ix.nlist, tq, nq[a], np[b], (long long)here, (long long)fewer_q, (long long)fewer_p);
                        return 1;
                    }
                }
        }
        // what calls really make: probes spread evenly, drawn at random, or all meeting in the longest lists
        std::vector<int32_t> order(ix.nlist);
        for (int l = 0; l < ix.nlist; ++l) order[l] = l;
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return size[x] > size[y]; });
        for (int q : nq)
            for (int p : np) {
                const int64_t pairs = (int64_t)q * p;
                if (p > ix.nlist || pairs > 400'000) continue;
                for (int width : {64, 96, 128}) {                   // queries of a tile of the threshold pass, by its form
                const TileShape shape = tile_shape(ix.total, ix.nlist, pairs, width);
                const bool few_tiles = pairs <= few;
                if (shape.part_near < kPartMin || shape.part < (few_tiles ? kPartFine : kPartMin) || shape.part_near % 64 || shape.part % 64) {
                    std::printf("%s nlist=%d: part lengths %d and %d\n", ix.kind, ix.nlist, shape.part_near, shape.part);
                    return 1;
                }
                for (int how = 0; how < 3; ++how) {
                    std::vector<int64_t> meets(ix.nlist, 0);
                    if (how == 0) for (int64_t i = 0; i < pairs; ++i) ++meets[i % ix.nlist];
                    if (how == 1) for (int64_t i = 0; i < pairs; ++i) { const int l = (int)(rng() % ix.nlist); if (meets[l] < q) ++meets[l]; }
                    if (how == 2) for (int i = 0; i < p; ++i) meets[order[i]] = q;
                    for (int near = 0; near < 2; ++near) {
                        const int tq = near ? shape.tq_near : shape.tq;
                        // (the room is counted by the fewest queries that any form takes)
                        const int64_t made = tiles_of(size, meets, tq, near ? shape.part_near : shape.part);
                        const int64_t held = near ? tile_room(room, q, pairs, kBatchTileNear) : late_tile_room(room, fine, few, q, pairs);
                        if (made > held) {
                            std::printf("%s nlist=%d: %d queries x %d probes make %lld tiles of %d, room for %lld\n", ix.kind, ix.nlist, q, p,
                                        (long long)made, tq, (long long)held);
                            return 1;
                        }
                    }
                }
                }
            }
    }
    return check_queues() ? 1 : check_rows();
}
