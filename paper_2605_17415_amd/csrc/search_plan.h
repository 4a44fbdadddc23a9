// How a search is cut into passes and a batched one into tiles, and how much room that takes.  Plain C++, no
// device code.
//
// A recorded graph keeps the addresses of the workspace, which moves only when a call needs more of it.  So what a call is
// given room for must not fall when it has more queries, probes or results: after the largest call no smaller one may
// need more.  The cuts themselves do not have that property (fewer pairs of query and list are cut into more parts each;
// shorter score rows allow longer passes), so the room is a bound that does.
#pragma once
#include <algorithm>
#include <cstdint>

namespace ivftq {

// Passes.  The workspace limit is for the score rows; a pass takes as many queries as it allows, since every pass walks every
// probed list again.  The batched path stores scores of the dense prefix only, rows of `prefix` floats (it stops at the
// first list that brings it to need_max vectors, so it is shorter than that plus the largest list); full-length rows,
// scores and columns, are needed for the queries redone exactly, which have gate_rows rows of the same
// buffer.  The streaming path stores every score.
constexpr int64_t kPassQueries = 32768;
struct SearchRows {
    int64_t stride;        // floats between score rows
    int64_t queries;       // of a pass
    int64_t gate_rows;     // (batched)
    int64_t held;          // rows of the arrays that have one per query of a pass
    int64_t floats;        // of the score buffer
};
// row: floats of a full-length row (every candidate); coarse_row: of a row of coarse scores; limit: bytes
inline SearchRows search_rows(bool batched, int64_t nq, int64_t row, int64_t prefix, int64_t coarse_row, int64_t limit) {
    const int64_t most = std::min(nq, kPassQueries), room = limit / 4;
    auto pass = [&](int64_t floats) { return std::max<int64_t>(1, std::min(most, room / floats)); };
    SearchRows r{};
    r.stride = batched ? std::min(row, prefix) : row;
    r.queries = pass(std::max(r.stride, coarse_row));
    r.gate_rows = std::min(r.queries, pass(2 * row));
    r.held = pass(coarse_row);
    const int64_t one = batched ? 2 * row : row;         // what a query takes when the limit does not cut the call
    r.floats = std::min(most * one, std::max(room, one));
    return r;
}

// Exact redo.  Its workgroups are shared out over the queries that a launch finds, each of which needs a score row until its results are
// selected.  Where the rows are as many as the workgroups, every workgroup has one and one launch looks after all `queries` of a
// pass, however many of them turn out to be redone.  With fewer, workgroups without a row would stand idle as soon as more queries are
// redone than there are rows, so there is a launch for as many queries as there are rows and all workgroups share each of them (40 queries
// redone in two rows, 64 lists of 20,000: 42.5 ms by one launch, 0.98 by launches for two queries each; an empty launch
// takes 2 us).
constexpr int kRedoWorkgroups = 1024;
constexpr int64_t redo_window(int64_t queries, int64_t gate_rows) {
    return gate_rows >= std::min<int64_t>(kRedoWorkgroups, queries) ? queries : gate_rows;
}

// Queries per tile, which is a wavefront's work: of the dense pass, and of the threshold pass the fewest that any form of it takes (which the room is
// counted by: batch_tile of kernels.h says how many a form takes).
constexpr int kBatchTile = 64, kBatchTileNear = 32;
// Lists of more than part_len vectors are cut into nearly equal parts of at most part_len, each a tile of its own.
constexpr int kPartMin = 256, kPartMax = 4096, kPartFine = 64;
struct TileShape { int tq_near, tq, part_near, part; };
constexpr int list_parts(int size, int part_len) { return size > part_len ? (size + part_len - 1) / part_len : 1; }

// Tiles of the batched passes, which 2048 to 3072 resident wavefronts take: enough of them that the last ones to finish matter little, but a
// tile reads its queries and costs reads that follow each other, about 4 us.  The whole call with 16384 and 32768, us: 10,000 queries at
// 10M x 200 1574 and 1503, at 10M x 96 597 and 583, 256 queries at 10M x 200 350 and 357; 65536 were slower than 32768.
constexpr int64_t kTilesWanted = 32768;
inline int part_length(int64_t typical_list, int64_t tiles) {
    const int64_t cuts = std::max<int64_t>(1, kTilesWanted / std::max<int64_t>(1, tiles));
    return (int)std::min<int64_t>(kPartMax, std::max<int64_t>(kPartMin, (typical_list / cuts + 63) / 64 * 64));
}
// Parts of kPartMin leave wavefronts without a tile where lists are few or short and meet few queries, and most of their tiles are one query
// tile high.  So the threshold pass's parts get shorter, down to kPartFine, as long as all tiles find a wavefront at once: the pass, us, with
// parts of 256 and so, 1700 queries x 5 probes of 130 lists of 1050 (48 coordinates, no clusters) 83 and 43, 391 x 43 of 300 of 233 (192) 58 and 36, 1000 x 32
// of 256 of 234 (128, 8 bits) 84 and 56, 500 x 20 of 200 of 300 (256) 73 and 36, 400 x 16 of 300 of 333 (96, clustered) 9.9 and 8.3.  With tiles for a
// wavefront and a few more 200 x 16 of 500 of 500 (200) took 41 instead of 28, 26 so.  (Cut further than that, calls that had as many tiles as
// wavefronts lost: parts of 128 instead of 256 for all, 400 x 64 of 512 of 781 5 to 12 % of the call.)
// (Lists are of different sizes and popularity: three quarters of the wavefronts are aimed at.)
constexpr int64_t kTilesFew = 2048;
// whole: tiles if no list were cut, a list's last one half full; part: as for many tiles
inline int part_late(int64_t typical_list, int64_t whole, int part) {
    const int64_t cuts = kTilesFew * 3 / 4 / std::max<int64_t>(1, whole);
    if (cuts < 2 || cuts <= list_parts((int)typical_list, kPartMin)) return part;
    int fine = (int)std::max<int64_t>(kPartFine, (typical_list / cuts + 32) / 64 * 64);
    while (fine < part && whole * list_parts((int)typical_list, fine) > kTilesFew) fine += 64;
    return std::min(part, fine);
}
inline TileShape tile_shape(int64_t ntotal, int nlist, int64_t pairs, int tq) {
    const int64_t typical = std::max<int64_t>(1, ntotal / nlist), lists = std::max<int64_t>(1, std::min<int64_t>(nlist, pairs));
    const int64_t whole = std::max(lists, pairs / tq + lists / 2);
    return {kBatchTileNear, tq, part_length(typical, lists), part_late(typical, whole, part_length(typical, lists + pairs / tq))};
}
// The most pairs with which calls can have so few tiles, whatever a tile takes: a list that is met, of which few pairs make as many, is a
// tile or more, and so are a tile's queries of pairs.
constexpr int kBatchTileMost = 128;
inline int64_t fine_pairs(int64_t ntotal, int nlist) {
    const int64_t most = kTilesFew / std::max(2, list_parts((int)std::max<int64_t>(1, ntotal / nlist), kPartMin));
    return nlist >= most ? most : most * kBatchTileMost;
}

// The tiles of a pass are dealt out to kTileQueues queues, each served by the workgroups of its number: updates of one counter from all over
// the chip follow each other at about 14 ns.  A launch has as many workgroups as the chip holds (`resident`), and one for every queue
// where that were fewer.
constexpr int kTileQueues = 16;
constexpr int tile_workgroups(int resident) { return std::max(resident, kTileQueues); }
constexpr int queue_servers(int workgroups, int queue) { return (workgroups - queue + kTileQueues - 1) / kTileQueues; }
// the j-th tile of a queue: one of each kTileQueues tiles, another one each time (the parts of a list, of which the last is the
// shortest, follow each other)
constexpr int queue_tile(int queue, int j) { return j * kTileQueues + (queue + 5 * j) % kTileQueues; }

// Entries that hold the tiles of a pass whose tiles take tq queries each, whatever the part length.  A list that meets c
// queries has at most 1 + c / tq tiles for each of its parts; c adds up to `pairs` over the lists and is at most
// `queries` in each.  list_room: what the first tile of every list takes.
struct ListRoom { int64_t all, longest; };
inline ListRoom list_room(const int32_t* size, int nlist, int part_len = kPartMin) {
    ListRoom r{0, 1};
    for (int l = 0; l < nlist; ++l) {
        const int parts = list_parts(size[l], part_len);
        r.all += parts;
        r.longest = std::max<int64_t>(r.longest, parts);
    }
    return r;
}
inline int64_t tile_room(const ListRoom& lists, int64_t queries, int64_t pairs, int tq) {
    return lists.all + std::min(pairs / tq * lists.longest, queries / tq * lists.all);
}
// The threshold pass: of calls with up to few_pairs pairs the parts may be kPartFine, fine the room of such.
inline int64_t late_tile_room(const ListRoom& lists, const ListRoom& fine, int64_t few_pairs, int64_t queries, int64_t pairs) {
    const int64_t q = std::min(queries, few_pairs), p = std::min(pairs, few_pairs);
    return std::max(tile_room(lists, queries, pairs, kBatchTile),
                    std::min(fine.all, p * fine.longest) + std::min(p / kBatchTile * fine.longest, q / kBatchTile * fine.all));
}

}  // namespace ivftq
