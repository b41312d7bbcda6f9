// The split of the attention kernel's work (attention_split.h) over plain arrays,
// for the CPU test: every piece of every range, in the kernel's order.
#include "../../paper_2512_11221_amd/csrc/attention_split.h"

#include <vector>

using namespace asrkf;

namespace {

struct Arrays {
    std::vector<int> off;           // [B + 1]
    const int32_t* n;
    int B;

    int find(int x) const {
        int b = 0;
        while (off[b + 1] <= x) ++b;
        return b;
    }
    int offset(int b) const { return off[b]; }
    int count(int b) const { return n[b]; }
};

}  // namespace

extern "C" {

int split_layout(const int32_t* plen, int batch, int t, int n_kv_heads, int row_bytes, int grid, int* launch) {
    int heads = 0;
    attention_layout(plen, batch, t, n_kv_heads, row_bytes, grid, &heads, launch);
    return heads;
}

int split_tile(int row_bytes) { return tile_tokens(row_bytes); }

// The pieces as rows of nine ints (range, then Piece in order), at most cap of
// them; returns their number.  info: live, aligned, groups, cost.
int split_pieces(const int32_t* n_active, int batch, int n_kv_heads, int heads_per_group, int grid, int tile,
                 int32_t* out, int cap, int32_t* info) {
    Split s{};
    s.init(tile, n_kv_heads, heads_per_group, grid);
    int total = 0, longest = 0, filled = 0;
    for (int b = 0; b < batch; ++b) {
        const int tiles = s.tiles_of(n_active[b]);
        total += tiles;
        longest = tiles > longest ? tiles : longest;
        filled += n_active[b] > 0;
    }
    s.choose(total, longest, filled);
    Arrays a{std::vector<int>(batch + 1, 0), n_active, batch};
    for (int b = 0; b < batch; ++b) a.off[b + 1] = a.off[b] + s.units_of(n_active[b]);
    s.ranges(a.off[batch]);
    info[0] = s.live;
    info[1] = s.aligned ? 1 : 0;
    info[2] = s.groups;
    info[3] = s.cost;
    int k = 0;
    for (int i = 0; i < s.live; ++i) {
        const int w = s.range_of(i);
        int x, x_end;
        s.range(w, x, x_end);
        Piece p;
        while (next_piece(s, a, w, x, x_end, p)) {
            if (k < cap) {
                const int row[9] = {w, p.b, p.n, p.group, p.t0, p.t1, p.n_parts, p.part, p.slot};
                for (int c = 0; c < 9; ++c) out[k * 9 + c] = row[c];
            }
            ++k;
        }
    }
    return k;
}

}  // extern "C"
