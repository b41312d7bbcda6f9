// Internal interface between the runtime (runtime.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

namespace asrkf {

// Split-K attention: the tiles of every (sequence, KV head group) pair are dealt
// to the workgroups of a fixed grid, from the active counts on the device
// (attention_split.h).  A pair that several workgroups share leaves one partial
// (m, l, acc) per workgroup, at consecutive slots; the last to arrive folds them.
constexpr int kMaxBatch = 1024;

// A low-relevance detection of the token at state index o in step t: the new
// count c_j (Eq. 3).  W = 0 counts every detection; otherwise a bit mask of
// the detections of the last W steps (bit i = step t - i) gives the count.
__device__ __forceinline__ int detect(int32_t* count, uint64_t* hmask, int32_t* hlast, size_t o,
                                      int t, int W) {
    int c;
    if (W == 0) {
        c = count[o] + 1;
    } else {
        const int gap = t - hlast[o];
        uint64_t m = gap >= 64 ? 0ull : (hmask[o] << gap);
        m |= 1ull;
        if (W < 64) m &= (1ull << W) - 1ull;
        hmask[o] = m;
        hlast[o] = t;
        c = __popcll(m);
    }
    count[o] = c;
    return c;
}

// Whether the token at position pos may be frozen.  wedge = n_t - K: positions
// >= wedge form the window of the K most recent positions (Sec. 3.2), which
// includes the token appended this step.  Algorithm 1 takes the candidates
// outside the window; inside = true takes those inside it instead.
__device__ __forceinline__ bool freeze_candidate(int pos, int wedge, bool inside) {
    return (pos < wedge) != inside;
}

// The K/V cache of a layer: [B][Hkv][pool_rows][D], head-major, so that a
// (sequence, KV head) pair's rows are one contiguous region.
struct AttnArgs {
    const void* kpool;        // layer base
    const void* vpool;
    const void* q;            // [B][Hq][D]
    const void* knew;         // [B][Hkv][D]
    const void* vnew;
    void* kpool_w;            // same as kpool, writable (append)
    void* vpool_w;
    const int32_t* list;      // layer base, [B][cap] ascending positions
    const int32_t* list_row;  // layer base, [B][cap] device row of each listed position
                              // (spill mode only; in resident mode the row is the position)
    const int32_t* n_active;  // layer base, [B]
    float* rel;               // layer base, [B][planes][rel_cap] relevance of the list entries (written):
                              // the first Hkv / heads_per_group planes hold |q.k| summed over a head
                              // group's query heads (Eq. 2); or Hq planes of logits
                              // q.k * log2(e)/sqrt(D) (softmax weights)
    int32_t* t_dev;           // first layer of a step: advanced by one (steps started), else null
    float* part_acc;          // [grid + pairs][heads][D] of the pairs that several workgroups share
    float* part_ml;           // [grid + pairs][heads][2]: (max in log2 units, sum)
    int32_t part_heads;       // query heads that the partials have room for
    int32_t* ticket;          // [B][Hkv] workgroups of a pair that have stored their partial; zero
                              // between launches
    float* out;               // [B][Hq][D]
    float* norm;              // softmax weights: [B][Hq][2] (max, sum) (written), or null
    int32_t B, cap, Hq, Hkv;
    int32_t planes;           // plane stride of a sequence
    int32_t rel_cap;          // entries of a plane (a multiple of 64)
    int32_t grid;             // workgroups the work is dealt to (a launch may have fewer or more)
    int32_t heads_per_group;  // KV heads a workgroup takes together (a power of two dividing Hkv)
    int32_t pool_rows;        // device rows per sequence (cap in resident mode)
    int32_t spill;            // 1: rows come from list_row
    int32_t rel_mode;         // 0: Eq. 2 |q.k|; 1: softmax weights
    float scale_log2;         // log2(e) / sqrt(D)
};

// The score verdicts of a step, from the relevance planes: one flag byte per
// attended position, bit 0 set where s_j < tau (Eq. 2, or the mean softmax
// weight), bit 1 where s_j lies within the debug margin of tau.
struct VerdictArgs {
    const float* rel;         // [layers][B][planes][rel_cap] by list entry, of the layers judged
    const float* norm;        // softmax weights: [layers][B][Hq][2]
    const int32_t* list;      // [states][B][cap]
    const int32_t* n_active;  // [states][B]
    uint8_t* flag;            // [states][B][cap] by position (written)
    float* sum;               // token scope: [B][rel_cap] sums over the layers judged by earlier launches
    int32_t B, cap, rel_cap;
    int32_t planes, used;     // plane stride of a sequence, planes that hold values
    int32_t softmax;
    int32_t states;           // layers judged that have states of their own, or 1 (token scope)
    int32_t layers_summed;    // 1, or the layers judged (token scope: they are summed)
    int32_t add_sum, keep_sum;  // token scope: sum is added / is written instead of the flags
    float tau_sum;            // tau * Hq (* L): compared against the sum
    float margin_sum;         // debug margin * Hq (* L); 0: off
};

// Entropy monitor of a sequence after the last restore (Sec. 3.6).
struct SeqMonitor {
    float entropy, pmax;
    int32_t escalation, level;
};

// Arrays to zero (16-byte aligned, sizes in 32-bit words).
constexpr int kMaxClear = 8;
struct ClearArgs {
    void* p[kMaxClear];
    size_t words[kMaxClear];
    int32_t n;
};

struct CompactArgs {
    int32_t* unfreeze;        // [L][B][cap]
    int32_t* list;            // [L][B][cap]
    int32_t* n_active;        // [L][B]
    const int32_t* plen;      // [B]
    const SeqMonitor* monitor;  // [B] recovery level per sequence (may be null)
    unsigned long long* listed_total;  // running sum of list lengths
    int32_t forced_level;     // -1: read monitor[]; 0: none; 1..3 forced SR/WR/FR
    int32_t count_forced;     // 1: count a forced level (no logits) in recoveries[]
    unsigned long long* recoveries;  // [4], indexed by level 1..3
    const int32_t* t_dev;     // steps started (advanced by each step's first attention launch)
    int32_t t;                // completed step, read from t_dev; lists are built for step t+1
    int32_t max_ctx;          // positions per sequence; a rebuild that would pass it is refused
    int32_t* flags;           // [0] a sequence ran out of device rows (spill mode),
                              // [1] a step would pass max_ctx positions
    int32_t* flag_host;       // spill mode: flags[0] in pinned host memory
    int32_t B, cap, wr_last_N;
    // spill mode only (spill_min_D > 0)
    int32_t spill_min_D;
    int32_t pool_rows;        // device rows per (layer, sequence)
    int32_t* row_of;          // [L][B][cap] device row of a position, -1: host store only
    uint8_t* on_host;         // [L][B][cap] 1: the host store holds the position's rows
    int32_t* list_row;        // [L][B][cap] device row of each listed position
    int32_t* last_row;        // [L][B][cap] the device row a host-only position held last
    int32_t* row_owner;       // [L][B][pool_rows] position whose K/V a row holds, -1: none
    int32_t* hand;            // [L][B] where the next search for free rows starts
    int32_t* pop_buf;         // [L][B][pool_rows] the free rows found for this rebuild
    int32_t* out_pos;         // [L][B][cap] rows to copy to the host store: position ...
    int32_t* out_row;         //   ... and the device row it leaves
    int32_t* n_out;           // [L][B]
    int32_t* in_pos;          // [L][B][cap] rows to copy back: position ...
    int32_t* in_row;          //   ... and the device row it takes
    int32_t* n_in;            // [L][B]
    unsigned long long* xfer; // [0] rows to host, [1] rows from host, [2] device rows released,
                              // [3] rows taken back intact (no copy)
    // the freeze loop of step t runs here, before recovery (not before step 1)
    int32_t freeze;           // 1: apply the step's freeze loop (set on the device: t > 0)
    const uint8_t* flag;      // [L][B][cap] verdicts of step t (VerdictArgs)
    unsigned long long* margin_hits;  // debug margin on: decisions near tau are counted here
    int32_t* count;           // [L][B][cap] (or [B][cap] in token scope): c_j
    uint64_t* hmask;
    int32_t* hlast;
    const int32_t* dur;
    int32_t dur_len, history_W, window_K;
    int32_t cand_inside;      // 1: freeze candidates inside the window, 0: outside
    // segmented rebuild of few, long instances (n_seg > 1)
    int32_t n_seg, seg_len;
    int32_t* seg_count;       // [instances][n_seg] counts ([instances][n_seg + 1][4] in spill mode)
};

// First decode step in spill mode: prompt positions p < P sit in device rows
// p, the other rows are free (the search for free rows starts at row P),
// nothing is on the host.
struct SpillInitArgs {
    int32_t* row_of;
    uint8_t* on_host;
    int32_t* last_row;
    int32_t* row_owner;
    int32_t* hand;
    const int32_t* plen;
    int32_t B, cap, pool_rows;
};

// A prompt's K/V of one (layer, sequence).
struct PrefillArgs {
    const char* k;            // [n][Hkv][row_bytes], any alignment of the element type
    const char* v;
    char* kdst;               // [Hkv][pool_rows][row_bytes]
    char* vdst;
    int32_t* plen;            // the sequence's prompt length, written when set_plen
    int32_t n, Hkv, row_bytes, pool_rows, set_plen;
    int32_t rows;             // rows that the kernel copies: n, or 0 (only the length is set)
};

// Row copies between the device cache and the host store (spill mode).
struct XferArgs {
    char* kpool;              // [L][B][Hkv][pool_rows][row_bytes / Hkv]
    char* vpool;
    char* khost;              // device-visible pointer of the pinned store, [L][B][cap][row_bytes]
    char* vhost;
    const int32_t* pos;       // [L][B][cap] per-instance lists of positions ...
    const int32_t* row;       //   ... and device rows
    const int32_t* count;     // [L][B] list lengths
    int32_t inst0;            // first (layer, sequence) instance of the launch
    int32_t cap, pool_rows, row_bytes;   // row_bytes: one token, every KV head
    int32_t Hkv;
    int32_t to_host;          // 1: device -> host store, 0: host store -> device
};

// Workgroups per sequence in the entropy pass: about 512 in all (measured: at
// batch 64, 8 per sequence take 12.8 us per step against 20.2 us for 32; more
// blocks per sequence wait longer on the sequence's ticket), 4 .. 32 each.
constexpr int kEntropySplitMax = 32;
constexpr int entropy_split(int B) {
    int s = kEntropySplitMax;
    while (s > 4 && s * B > 512) s >>= 1;
    return s;
}

struct EntropyArgs {
    const float* logits;      // [B][V]
    float* partial;           // [B][split][3] block triples (m, S, T)
    int32_t split;            // workgroups per sequence, 4 .. kEntropySplitMax
    int32_t* ticket;          // [B] blocks finished; reset by the last one
    int32_t V, B;
    float theta_H, theta_p;
    int32_t mode;             // 0 AUTO, 1..3 forced, 4 none
    SeqMonitor* monitor;      // [B] (updated)
    unsigned long long* recoveries;  // [4], indexed by level 1..3
    unsigned long long* rr_requests;
};

// start/stop (may be null) are recorded by the kernel's own dispatch.
hipError_t launch_attention(const AttnArgs& a, int dtype_bf16, int head_dim, int group,
                            int grid, hipStream_t s, hipEvent_t start, hipEvent_t stop);
hipError_t attention_occupancy(const AttnArgs& a, int dtype_bf16, int head_dim, int group,
                               int* blocks_per_cu);
hipError_t launch_clear(const ClearArgs& a, hipStream_t s);
hipError_t launch_compact(const CompactArgs& a, int n_instances, hipStream_t s);
// Segments per instance (and their length) for the rebuild; 1 = one workgroup per instance.
int compact_segments(int n_instances, int cap, bool spill, int* seg_len);
hipError_t launch_spill_init(const SpillInitArgs& a, int n_instances, hipStream_t s);
hipError_t launch_xfer(const XferArgs& a, int n_instances, hipStream_t s);
// Whether the attention kernel handles this (dtype, head_dim, q heads per KV head, KV heads).
bool attention_shape_supported(int dtype_bf16, int head_dim, int group, int n_kv_heads);
hipError_t launch_delay(int microseconds, hipStream_t s);
// The step's verdicts and, when e is given, the entropy monitors, in one launch.
hipError_t launch_monitor(const EntropyArgs* e, const VerdictArgs& v, hipStream_t s);
// A prompt's rows into the head-major cache: k, v [n][Hkv][row] -> [Hkv][pool_rows][row].
hipError_t launch_prefill(const PrefillArgs& a, hipStream_t s);

}  // namespace asrkf
