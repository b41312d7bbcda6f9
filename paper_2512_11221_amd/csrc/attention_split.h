// How the attention kernel's work is dealt to its workgroups.  Plain integer
// arithmetic, used by the kernel (which keeps the lists in lanes or LDS), by the
// host for the launch, and by a CPU test over arrays.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace asrkf {

#define ASRKF_HD __host__ __device__ __forceinline__

// What a piece costs a workgroup beside its rows (set-up round trips, merge,
// partial), in tiles of one KV head streamed: about 6 us against 0.6 us a tile.
constexpr int kPieceCost = 10;
// Fewest tiles of one KV head worth a workgroup, and the share up to which only
// half of the workgroups are used: with little work the launch is bound by fixed
// latencies, and 256 workgroups start two microseconds later than 128 (one
// sequence of 4093 tokens, 8 KV heads: 14.4 us with 128 workgroups of 8 tiles,
// 15.4 with 256 of 4; of 1500 tokens: 11.9 with 96 of 4, 13.2 with 48 of 8).
constexpr int kMinTiles = 4;
constexpr int kHalfTiles = 8;
// bytes of rows that a wave's tile holds, and of relevance values that it has room for
constexpr int kTileBytes = 8192;
constexpr int kRelRoomBytes = 8192;
constexpr int kAttnWaves = 8;

ASRKF_HD constexpr int tile_tokens(int row_bytes) { return kTileBytes / row_bytes; }
// tiles whose relevance values a workgroup has room for
constexpr int room_tiles(int tile) { return kRelRoomBytes / (tile * 4) * kAttnWaves; }

ASRKF_HD int lesser(int a, int b) { return a < b ? a : b; }
ASRKF_HD int greater(int a, int b) { return a > b ? a : b; }

// Tiles of the (sequence, head group) pairs dealt to the workgroups, from the
// active counts.  Two forms, chosen by what the longest share would be:
//  aligned   every pair is cut into parts of at most `share` tiles, one
//            workgroup each (a workgroup never takes a second piece, which
//            would cost it set-up, merge and partial again);
//  straddled the pairs' tile lists, each preceded by `cost` virtual tiles, are
//            concatenated and cut into equal ranges: when the lengths differ so
//            much, or the pairs are so many, that aligned parts would leave some
//            workgroup more than a piece's cost above the average.
// Batches of up to 64 sequences are planned by every wave for itself, one
// sequence per lane, without a barrier; larger ones by wave 0 into LDS.
struct Split {
    int tile;                       // tokens per tile
    int groups, cost, limit;        // head groups per sequence, piece cost in tiles, workgroups
    int heads;                      // KV heads a workgroup takes together
    bool aligned;
    int share;                      // aligned: tiles per part; straddled: tiles per range (the first
    int extra;                      //   `extra` ranges have one more)
    int live;                       // workgroups with work

    ASRKF_HD void init(int tokens, int n_kv_heads, int heads_per_group, int grid) {
        tile = tokens;
        heads = heads_per_group;
        groups = n_kv_heads / heads_per_group;
        cost = greater(1, kPieceCost / heads_per_group);
        limit = grid;
        extra = 0;
    }
    ASRKF_HD int parts(int tiles) const { return (tiles + share - 1) / share; }
    ASRKF_HD int tiles_of(int n) const { return (n + tile - 1) / tile; }
    // units of a list of n entries: workgroups (aligned), tiles (straddled)
    ASRKF_HD int units_of(int n) const {
        const int tiles = tiles_of(n);
        return n == 0 ? 0 : groups * (aligned ? parts(tiles) : tiles + cost);
    }
    // total: tiles of all sequences, longest: of the longest, filled: sequences with any
    ASRKF_HD void choose(int total, int longest, int filled) {
        const int average = (total * groups + limit - 1) / limit;
        const int most = limit / greater(1, filled * groups);     // parts a pair can have
        share = greater(kMinTiles / lesser(kMinTiles, heads), most > 0 ? (longest + most - 1) / most : 0);
        share = greater(share, lesser(kHalfTiles / lesser(kHalfTiles, heads), 2 * average));
        aligned = most > 0 && share <= greater(average + cost, kHalfTiles);
    }
    // units: of all sequences
    ASRKF_HD void ranges(int units) {
        if (aligned) {
            live = units;
            return;
        }
        live = greater(1, lesser(limit, units / kMinTiles));
        share = units / live;
        extra = units - share * live;
        if (units == 0) live = 0;
    }
    ASRKF_HD int start(int w) const { return w * share + lesser(w, extra); }
    ASRKF_HD int owner(int x) const {                             // the range holding tile x
        const int head = extra * (share + 1);
        return x < head ? x / (share + 1) : extra + (x - head) / share;
    }
    ASRKF_HD void range(int w, int& x, int& x_end) const {
        x = aligned ? w : start(w);
        x_end = aligned ? w + 1 : start(w + 1);
    }
    // The workgroup of index i takes range w: workgroups are dealt to the 8 XCDs
    // round robin, and when every workgroup has work each XCD takes a contiguous
    // block of ranges.  Any one-to-one map gives the same partials.
    ASRKF_HD int range_of(int i) const {
        return live == limit && limit % 8 == 0 ? (i % 8) * (limit / 8) + i / 8 : i;
    }
};

// One workgroup's part of a pair.
struct Piece {
    int b, n;                       // sequence, its active count
    int group;                      // head group
    int t0, t1;                     // tiles
    int n_parts, part, slot;        // workgroups sharing the pair, which of them, partial slot
};

// The next piece of range w from unit x on (x moves past it); false: only
// virtual tiles were left.  Lists: find(x), the sequence that owns unit x;
// offset(b), its first unit; count(b), its active count.
template <typename Lists>
ASRKF_HD bool next_piece(const Split& split, const Lists& lists, int w, int& x, int x_end, Piece& p) {
    while (x < x_end) {
        p.b = lists.find(x);
        const int so = lists.offset(p.b);
        p.n = lists.count(p.b);
        const int tiles = split.tiles_of(p.n);
        if (split.aligned) {
            p.n_parts = split.parts(tiles);
            p.group = (x - so) / p.n_parts;
            p.part = x - so - p.group * p.n_parts;
            p.t0 = p.part * split.share;
            p.t1 = lesser(tiles, p.t0 + split.share);
            p.slot = x;
            ++x;
            return true;
        }
        const int units = tiles + split.cost;     // of one head group
        p.group = (x - so) / units;
        const int first = so + p.group * units + split.cost;      // the pair's first tile
        const int end = lesser(first + tiles, x_end);
        const int from = greater(x, first);
        x = end;
        if (end <= first) continue;               // virtual tiles only
        p.t0 = from - first;
        p.t1 = end - first;
        const int w0 = split.owner(first);
        p.n_parts = split.owner(first + tiles - 1) - w0 + 1;
        p.part = w - w0;
        p.slot = w + p.b * split.groups + p.group;
        return true;
    }
    return false;
}

// How a step's attention is laid out when sequence b lists up to plen[b] + t
// positions: KV heads a workgroup takes together, and how many workgroups to
// launch (at least those with work, at most grid: idle ones delay the others).
inline void attention_layout(const int32_t* plen, int batch, int t, int n_kv_heads, int row_bytes, int grid,
                             int* heads_per_group, int* launch) {
    const int tile = tile_tokens(row_bytes);
    int64_t tiles = 0;
    for (int b = 0; b < batch; ++b) tiles += (plen[b] + tile) / tile;
    // One KV head per piece while every pair can have a workgroup and the pieces are
    // short: a pair's partials and its merge are smallest, and its relevance values
    // are stored once, at the end.  With more pairs a workgroup would walk several
    // short pieces one after the other, each with its own round trips: the waves take
    // as many heads side by side as bring the pairs down to the workgroups, and no
    // more (16 x 100 to 900 tokens, 32 heads: 35.4 us a launch with one head, 31.5
    // with two; 128 x 100 to 500 tokens, 8 heads: 45.0 us with eight, 43.8 with four,
    // 54.8 with one).  With long pieces the relevance values of every head would be
    // stored among the row loads, where they cost ten times their bytes: eight heads,
    // whose values are summed first (64 x 2k to 32k tokens: 684 us with one head, 662
    // with eight).  The softmax reading keeps one value per query head either way and
    // its room holds fewer tiles; the same rule serves it (64 x 2k to 32k tokens: 831
    // us with one head, 808 with eight; 8 x 65k tokens of eight query heads, just on
    // this side of the line: 417 and 455).  The choice rests on the prompts alone, so
    // a step replayed from a graph is dealt like the same step run eagerly; lists that
    // grow long from short prompts stay with the heads chosen for those (64 sequences
    // grown from nothing to 18k tokens: 712 us a launch).
    int hw = 1;
    if (tiles * n_kv_heads > (int64_t)room_tiles(tile) * grid) hw = n_kv_heads < 8 ? n_kv_heads : 8;
    while (hw < 8 && hw < n_kv_heads && (int64_t)batch * n_kv_heads / hw > grid) hw *= 2;
    const int64_t groups = n_kv_heads / hw;
    const int cost = kPieceCost / hw > 1 ? kPieceCost / hw : 1;
    const int least = kMinTiles / (hw < kMinTiles ? hw : kMinTiles);
    int64_t live = 0;
    for (int b = 0; b < batch && live < grid; ++b)
        live += groups * (((plen[b] + t + tile - 1) / tile + cost + least - 1) / least);
    *heads_per_group = hw;
    *launch = live < grid ? (live > 1 ? (int)live : 1) : grid;
}


}  // namespace asrkf
