// Active-set GQA flash-decode for gfx950, fused with the relevance products
// and the split combine.
//
// Per launch (one layer, every sequence):
//   Eq. 1  o_h = softmax_j(q_h . k_j / sqrt(D)) v_j over the active list A_t;
//   Eq. 2  the relevance of every j in A_t: per KV head the sum over its
//          query heads of |q_h . k_j| (or, for the reading by attention
//          weight, the logit of every query head), one value per list entry
//          and plane.  The end-of-step verdict sums the planes and compares
//          with tau, so no score crosses workgroups here.
//
// Work decomposition.  The cache is head-major, so a (sequence, KV head) pair
// is one stream of contiguous rows: its active list, cut into tiles of 32
// tokens, is a list of tiles.  The tile lists of all pairs, concatenated (each
// preceded by a few virtual tiles that stand for the fixed cost of a piece),
// are cut into equal contiguous ranges, one per workgroup of a fixed grid,
// computed on the device from the active counts.  A pair with one workgroup is
// finished by it; a pair shared by several leaves one partial (m, l, acc) per
// workgroup, and the workgroup that arrives last (a per-pair ticket) folds
// them in slot order and writes the outputs.  A partial holds one KV head's
// query heads only, so the last one pulls a few KB; with whole-row workgroups
// (every KV head of a token range) it would be the sequence's half megabyte,
// which took a launch of its own.
//
// Why head-major: a plain streaming kernel of this grid moves dense ranges at
// 6.99 TB/s and 35 % gathers at 6.75 TB/s when a wave's load instruction covers
// four whole 256-byte head rows of a head-major cache; 6.82 and 6.52 TB/s for
// whole 2 KiB rows of a token-major cache, 6.29 and 5.85 TB/s for 256-byte rows
// of a token-major cache, and 5.98 and 5.41 TB/s for 64-byte pieces of 16 rows
// (the lane layout of the matrix instruction, hence the LDS tiles below).
//
// Inside a workgroup every wave takes whole tiles (round-robin, a static deal,
// so every run sums in the same order).  A tile's K and V rows travel through
// registers into the wave's own LDS tile, the next tile's rows are requested
// at once, and the arithmetic runs on the matrix cores from LDS: no barrier in
// the loop.  Scores: S^T = K Q^T with the tokens as rows, the query heads
// (repeated) as the 16 columns.  Accumulate: O += P V with P's rows the heads;
// the column layout of S^T is the row layout of P, so the weights stay in their
// lanes.  fp32 rows use the fp32 matrix instruction.  bf16 rows keep fp32
// weights: the repeated columns carry p's leading, middle and trailing 8
// mantissa bits as three bf16 rows (exact: p = hi + mid + lo), summed in fp32
// when the waves are merged.  With eight query heads the sixteen rows hold two
// parts, so a tile takes two passes into the same sums: hi and mid, then 2^-30 p
// and lo.  The 2^-30 p (far below the rounding of hi's sums) is there because the
// second pass may leave no zero in a row whose weight is not zero: an infinite
// value times 0 would turn that row's sum into NaN.  lo in sums of its own took 64
// registers more with rows of 256, and the kernel spilled as many (four layers, 8
// sequences of 16k, one KV head: 230 us a step, 165 with the shared sums).
#include <type_traits>

#include "attention_split.h"
#include "kernels.h"

namespace asrkf {
namespace {

// raw buffer descriptor word 3 for gfx9-class targets (32-bit data, no swizzle)
constexpr int kBufferFlags = 0x00020000;
// cache policy of the K/V row loads: non-temporal.  Each row is read once per
// launch; the streaming probe above reaches 6.07 and 5.83 TB/s without it.
constexpr int kStreamPolicy = 2;
// cache policy of the partials that workgroups exchange: device scope (past the
// XCD's own L2)
constexpr int kAgentScope = 16;
// an offset past every buffer's range (a pair's rows stay below 2 GiB): loads
// there return zeros and stores are dropped, without a memory access, so
// masked lanes cost nothing and the compiler counts every wait exactly
constexpr int kNowhere = (int)0x80000000;

__device__ __forceinline__ int wave_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// value of lane N of the lane's row of 16
template <int N>
__device__ __forceinline__ int row_bcast(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + N, 0xF, 0xF, false);
}

template <int N, typename F>
__device__ __forceinline__ void unroll(F f) {
    if constexpr (N > 0) {
        unroll<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* lds_shortx4;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, kBufferFlags);
}

template <int POLICY>
__device__ __forceinline__ intx4 load16(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POLICY));
}

// A barrier for what the waves share in LDS.  __syncthreads also waits for every
// load and store in flight: the next tile's rows, the relevance stores and the
// append, which nobody in the workgroup reads back.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- the split ----
//
// The split with the lists it deals.  Batches of up to 64 sequences are planned by
// every wave for itself, one sequence per lane, without a barrier; larger ones by
// wave 0 into LDS.
struct Plan : Split {
    // sequence b owns units [off, off + units)
    int n, units, off;              // of the lane's sequence (up to 64 sequences)
    const int32_t* lds;             // [B + 1] offsets, then [B] counts (more than 64)
    int B;

    // the sequence that owns unit x
    __device__ __forceinline__ int find(int x) const {
        if (B <= 64) return __popcll(__ballot((int)(threadIdx.x & 63) < B && off + units <= x));
        int l0 = 0, h0 = B - 1;                                   // last b with lds[b] <= x
        while (l0 < h0) {
            const int mid = (l0 + h0 + 1) >> 1;
            if (wave_uniform(lds[mid]) <= x) l0 = mid; else h0 = mid - 1;
        }
        while (wave_uniform(lds[l0 + 1]) <= x) ++l0;              // past empty lists
        return l0;
    }
    __device__ __forceinline__ int offset(int b) const {
        return B <= 64 ? __builtin_amdgcn_readlane(off, b) : wave_uniform(lds[b]);
    }
    __device__ __forceinline__ int count(int b) const {
        return B <= 64 ? __builtin_amdgcn_readlane(n, b) : wave_uniform(lds[B + 1 + b]);
    }
};

struct PlanInput {
    const int32_t* n_active;
    int B, Hkv, heads_per_group, grid;
};

__device__ __forceinline__ Plan make_plan(const PlanInput& a, int tile, int32_t* lds) {
    Plan p;
    p.init(tile, a.Hkv, a.heads_per_group, a.grid);
    p.B = a.B;
    p.lds = lds;
    const int lane = threadIdx.x & 63;
    int total = 0;
    if (a.B <= 64) {
        p.n = lane < a.B ? a.n_active[lane] : 0;
        const int tiles = p.tiles_of(p.n);
        int sum = tiles, top = tiles;
        if (a.B > 1) {
            for (int o = 1; o < a.B; o <<= 1) {                   // lanes past B hold 0
                sum += __shfl_xor(sum, o);
                top = max(top, __shfl_xor(top, o));
            }
        }
        const int filled = __popcll(__ballot(p.n > 0));
        p.choose(wave_uniform(sum), wave_uniform(top), filled);
        p.units = p.units_of(p.n);
        int incl = p.units;
        if (a.B > 1) {
            for (int o = 1; o < a.B; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
        }
        p.off = incl - p.units;
        total = __builtin_amdgcn_readlane(incl, a.B - 1);
    } else {
        int32_t* off = lds;
        int32_t* cnt = lds + a.B + 1;
        __shared__ int summary[3];
        if (threadIdx.x < 64) {
            constexpr int kBatch = 8;                 // counts loaded together
            const int per = (a.B + 63) / 64;
            const int b0 = min(a.B, lane * per), b1 = min(a.B, b0 + per);
            int sum = 0, top = 0, filled = 0;
            for (int bb = b0; bb < b1; bb += kBatch) {
                int c[kBatch];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) c[k] = a.n_active[min(bb + k, b1 - 1)];
#pragma unroll
                for (int k = 0; k < kBatch; ++k) {
                    if (bb + k >= b1) continue;
                    cnt[bb + k] = c[k];
                    const int tiles = p.tiles_of(c[k]);
                    sum += tiles;
                    top = max(top, tiles);
                    filled += c[k] > 0;
                }
            }
            for (int o = 1; o < 64; o <<= 1) {
                sum += __shfl_xor(sum, o);
                top = max(top, __shfl_xor(top, o));
                filled += __shfl_xor(filled, o);
            }
            p.choose(wave_uniform(sum), wave_uniform(top), wave_uniform(filled));
            int mine = 0;
            for (int bb = b0; bb < b1; ++bb) mine += p.units_of(cnt[bb]);
            int incl = mine;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            int run = incl - mine;
            for (int bb = b0; bb < b1; ++bb) {
                off[bb] = run;
                run += p.units_of(cnt[bb]);
            }
            if (lane == 63) {
                off[a.B] = incl;
                summary[0] = p.share;
                summary[1] = p.aligned ? 1 : 0;
            }
        }
        __syncthreads();
        p.share = wave_uniform(summary[0]);
        p.aligned = wave_uniform(summary[1]) != 0;
        total = wave_uniform(off[a.B]);
    }
    p.ranges(total);
    return p;
}

// ---- tiles ----

template <bool BF16, int D>
struct Row {
    static constexpr int kElem = BF16 ? 2 : 4;
    static constexpr int kBytes = D * kElem;              // one token, one KV head
    static constexpr int kLanes = kBytes / 16;            // lanes per row in a load
    // tokens per tile: 16 KB of K and V rows, in a wave's registers while they travel
    static constexpr int kTile = tile_tokens(kBytes);
    static constexpr int kBlocks = kTile / 16;            // score blocks of 16 tokens
    static constexpr int kLoads = kTile * kLanes / 64;    // load instructions per tile (K or V)
    // LDS row strides: the padding shifts consecutive rows by 4 (K) and 8 (V)
    // banks, so the 16-byte reads of K rows and the transposed reads of V rows
    // meet no bank twice.  A wave's K tile is read before its V tile is written,
    // in the same place.
    static constexpr int kKStride = kBytes + 16;
    static constexpr int kVStride = kBytes + 32;
    static constexpr int kTileLds = kTile * kVStride;
    // room for the relevance values a wave keeps before they are stored
    static constexpr int kRelLds = kRelRoomBytes;
    static constexpr int kWaveLds = kTileLds + kRelLds;
    static constexpr int kWaves = kAttnWaves;
    static constexpr int kQRegs = BF16 ? D / 32 : D / 16; // 16-byte pieces of q per lane
};

// Rows of P: query head h of part p sits in row p * G + h.  With G = 8 the
// sixteen rows hold two parts at a time: two passes.
template <bool BF16, int G>
constexpr bool two_passes() { return BF16 && G == 8; }

// A maximum as the reference of exponents: 2^(x - reference(M)) is 0 for x = -inf,
// also where no score above -inf came yet.  States without such a score are folded
// like the others, with weight 0: their sums are zero, or NaN where a score was,
// which the result has to show.
__device__ __forceinline__ float reference(float M) { return M == -INFINITY ? 0.f : M; }

// (L, o) += wgt * (l, v)
__device__ __forceinline__ void fold(float& L, floatx4& o, float wgt, float l, floatx4 v) {
    L = fmaf(wgt, l, L);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = fmaf(wgt, v[i], o[i]);
}

// Groups of threads that fold a pair's parts, each spanning the outputs of HEADS
// KV heads (four values a thread), and the round trips that the fold takes.
template <int G, int D, int HEADS>
struct Fold {
    static constexpr int kThreads = 64 * kAttnWaves;
    static constexpr int kSpan = HEADS * G * D / 4 < kThreads ? HEADS * G * D / 4 : kThreads;
    static constexpr int kSlotGroups = kThreads / kSpan < 16 ? kThreads / kSpan : 16;
    __device__ static __forceinline__ int trips(int heads, int n_parts, int pass) {
        return (heads * D + kSpan * 4 - 1) / (kSpan * 4) * ((n_parts + kSlotGroups * pass - 1) / (kSlotGroups * pass));
    }
};

// Where a piece's outputs go.
struct Finish {
    float* out;                     // first query head of the piece
    float* norm;                    // its normaliser, or null
    template <int D>
    __device__ __forceinline__ void write(int hh, int d, float M, float L, floatx4 o) const {
        floatx4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = o[i] / L;
        *reinterpret_cast<floatx4*>(out + (size_t)hh * D + d) = r;
        if (norm && d == 0) {
            norm[hh * 2] = M;
            norm[hh * 2 + 1] = L;
        }
    }
};

// a finite value as it is, anything else 0
__device__ __forceinline__ float finite_or_0(float x) { return fabsf(x) < INFINITY ? x : 0.f; }

// a's rows 1, 3 (of 16 lanes) exchanged with b's rows 0, 2, then added:
// rows a0 + a1, b0 + b1, a2 + a3, b2 + b3
__device__ __forceinline__ float add_rows16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// a's upper half exchanged with b's lower half, then added: rows a0 + a2, a1 + a3, b0 + b2, b1 + b3
__device__ __forceinline__ float add_halves(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// the maximum over the lanes of a column (its four rows of 16 lanes)
__device__ __forceinline__ float column_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// A wave's accumulators as [G][kMergeStride] sums in LDS.  Row 4 q4 + i, column
// c16 of block k; the parts of a bf16 weight are added here.  Where a value row
// holds an infinity, the leading part has the result and the others may hold
// 0 * inf, so those count only while they are finite.
template <bool BF16, int D, int G, typename Acc>
__device__ __forceinline__ void store_state(const Acc& acc, float* st, int lane) {
    constexpr int S = D + 4;
    const int c16 = lane & 15, q4 = lane >> 4;
#pragma unroll
    for (int k = 0; k < D / 16; ++k) {
        float* col = st + k * 16 + c16;
        const floatx4 v = acc[k];
        if constexpr (!BF16) {
#pragma unroll
            for (int i = 0; i < (G < 4 ? G : 4); ++i)
                if (q4 * 4 < G) col[(q4 * 4 + i) * S] = v[i];
        } else if constexpr (G == 1) {
            const float x = v[0] + (finite_or_0(v[1]) + finite_or_0(v[2]));
            if (q4 == 0) col[0] = x;
        } else if constexpr (G == 2) {
            const float x0 = q4 == 0 ? v[0] + finite_or_0(v[2]) : finite_or_0(v[0]);
            const float x1 = q4 == 0 ? v[1] + finite_or_0(v[3]) : finite_or_0(v[1]);
            const float x = add_rows16(x0, x1);
            if (q4 < 2) col[q4 * S] = x;
        } else if constexpr (G == 4) {
            float x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = q4 == 0 ? v[i] : q4 < 3 ? finite_or_0(v[i]) : 0.f;
            col[q4 * S] = add_halves(add_rows16(x[0], x[1]), add_rows16(x[2], x[3]));
        } else {
            const int h = (q4 & 1) * 4 + (q4 >> 1);
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float x0 = q4 < 2 ? v[i] : finite_or_0(v[i]);
                const float x1 = q4 < 2 ? v[i + 1] : finite_or_0(v[i + 1]);
                col[(h + i) * S] = add_halves(x0, x1);
            }
        }
    }
}

template <bool BF16, int D>
constexpr int threads_of() { return 64 * Row<BF16, D>::kWaves; }

template <bool BF16, int D, int G>
__global__ void __launch_bounds__((threads_of<BF16, D>()), 2)
attention_kernel(AttnArgs a) {
    using R = Row<BF16, D>;
    constexpr int kWaves = R::kWaves;
    constexpr int kThreads = threads_of<BF16, D>();
    constexpr int kTile = R::kTile;
    constexpr int NBLK = R::kBlocks;
    constexpr int NL = R::kLoads;
    constexpr int NQ = R::kQRegs;
    constexpr int NB = D / 16;                    // column blocks of the accumulators
    constexpr bool kTwice = two_passes<BF16, G>();
    static_assert(G * (D + 4) * 4 <= R::kTileLds, "wave state fits its tile");
    static_assert(64 * 24 <= R::kTileLds, "a wave's folded states fit its tile");

    extern __shared__ __align__(16) char lds[];
    char* tiles = lds;                                            // [kWaves][kWaveLds]
    float* ml_lds = reinterpret_cast<float*>(lds + kWaves * R::kWaveLds);   // [kWaves][2][G]
    int32_t* plan_lds = reinterpret_cast<int32_t*>(ml_lds + kWaves * 2 * G);
    __shared__ int last_arrival;

    // the step's first launch advances the device step counter that the
    // end-of-step rebuild reads (a graph replay of the step then sees its step)
    if (a.t_dev && blockIdx.x == 0 && threadIdx.x == 0) *a.t_dev += 1;
    const int hw = a.heads_per_group;             // KV heads a workgroup takes together
    const int groups = a.Hkv / hw;                // head groups of a sequence

    const int wave = wave_uniform(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int c16 = lane & 15;                    // column (S^T), row of P
    const int q4 = lane >> 4;
    const int piece = (lane % R::kLanes) * 16;    // the lane's 16 bytes of a row
    const int lrow = lane / R::kLanes;            // its row group in a load
    const int wh = wave % hw;                     // the wave's KV head within the group
    const int wt = wave / hw;                     // its turn among the tiles
    const int nwt = kWaves / hw;
    char* kt = tiles + wave * R::kWaveLds;        // the wave's K tile, then its V tile
    char* vt = kt;
    float* rel_kept = reinterpret_cast<float*>(kt + R::kTileLds);  // [tile][wide][kTile]
    // which 8 bits of p the lane's rows of P carry: leading (0), middle (1), trailing (2 and up)
    const uint32_t mask1 = c16 / G >= 1 ? 0xFFFF0000u : 0u;
    const uint32_t mask2 = c16 / G >= 2 ? 0xFFFF0000u : 0u;
    const bool rel_abs = a.rel_mode == 0;

    const Plan plan = make_plan(PlanInput{a.n_active, a.B, a.Hkv, hw, a.grid}, kTile, plan_lds);
    for (int wi = blockIdx.x; wi < plan.live; wi += gridDim.x) {
    const int w = plan.range_of(wi);
    int x, x_end;
    plan.range(w, x, x_end);
    x = wave_uniform(x);
    x_end = wave_uniform(x_end);
    Piece pc;
    while (next_piece(plan, plan, w, x, x_end, pc)) {
        constexpr int kPer = 64 / R::kLanes;
        const int entry = R::kLanes == 8 ? (lane & 7) * 8 + (lane >> 4) * 2 + ((lane >> 3) & 1)
                                         : (lane % NL) * kPer + lrow;
        const int b = wave_uniform(pc.b), nb = wave_uniform(pc.n), gi = wave_uniform(pc.group);
        const int t0 = wave_uniform(pc.t0), t1 = wave_uniform(pc.t1);
        const int n_parts = wave_uniform(pc.n_parts), part = wave_uniform(pc.part), slot = wave_uniform(pc.slot);
        const int pair = b * groups + gi;
        const int g = gi * hw + wh;               // the wave's KV head
        const size_t pool_row0 = ((size_t)b * a.Hkv + g) * a.pool_rows;
        const int pool_bytes = a.pool_rows * R::kBytes;
        const auto rk = buffer((const char*)a.kpool + pool_row0 * R::kBytes, pool_bytes);
        const auto rv = buffer((const char*)a.vpool + pool_row0 * R::kBytes, pool_bytes);
        const int32_t* list_b = (a.spill ? a.list_row : a.list) + (size_t)b * a.cap;
        const auto rl = buffer(list_b, a.cap * 4);
        const int planes = rel_abs ? groups : a.Hq;
        const auto rr = buffer(a.rel + (size_t)b * a.planes * a.rel_cap, planes * a.rel_cap * 4);
        // Load j of a tile takes the tokens j * kPer .. j * kPer + kPer - 1, so that in a
        // dense list one instruction reads 1 KiB in a row.  Lane i of a row of 16 lanes
        // holds the list entry that the row's lanes need in load i (a row broadcast
        // hands it out; where 16 lanes span two tokens, lanes 8 and up hold the second's).
        // The list's last entry is the new token: its row comes from the arguments, not
        // from the cache.
        const int n_cached = nb - 1;
        auto load_rows = [&](int t) __attribute__((always_inline)) {
            return __builtin_amdgcn_raw_buffer_load_b32(rl, t < t1 ? (t * kTile + entry) * 4 : kNowhere, 0, 0);
        };
        auto row_offsets = [&](int t, int rw, int (&off)[NL]) __attribute__((always_inline)) {
            const int lim = t < t1 ? n_cached - t * kTile - lrow : 0;
            unroll<NL>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = decltype(J)::value;
                int row = row_bcast<j>(rw);
                if constexpr (R::kLanes == 8) row = (lane & 8) ? row_bcast<8 + j>(rw) : row;
                off[j] = j * kPer < lim ? row * R::kBytes + piece : kNowhere;
            });
        };
        // The order of the loop's loads is fixed (the list entries of the tile after
        // next, the next tile's K rows, its V rows), and the same ahead of the loop, so
        // that every wait counts exactly what is younger.
        auto load_tile = [&](__amdgpu_buffer_rsrc_t r, const int (&off)[NL], intx4 (&x)[NL])
            __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NL; ++j) x[j] = load16<kStreamPolicy>(r, off[j]);
            __builtin_amdgcn_sched_barrier(0);
        };
        // The relevance values stay in LDS and are stored together, at the piece's end or
        // when the room is full, summed over the workgroup's KV heads: stored tile by
        // tile among the row loads they cost as much as ten times their bytes (a launch
        // over 8 x 32k tokens took 178 instead of 166 us with 8 MB of them).
        const int wide = rel_abs ? 1 : G;         // planes of a KV head
        const bool keeps = c16 < wide;            // lanes that hold a value to keep
        const int chunk = R::kRelLds / (kTile * 4) / wide * nwt;   // tiles the room is for
        const auto store_kept = [&](int c0, int c1) __attribute__((always_inline)) {
            const int per_wave = (c1 - c0 + nwt - 1) / nwt;
            const int n4 = rel_abs ? (c1 - c0) * (kTile / 4) : kWaves * per_wave * wide * (kTile / 4);
            for (int e = threadIdx.x; e < n4; e += kThreads) {
                const int o = e % (kTile / 4), row = e / (kTile / 4);
                floatx4 v = {0.f, 0.f, 0.f, 0.f};
                int at;
                if (rel_abs) {
                    const int turn = row % nwt, idx = row / nwt;
                    for (int h = 0; h < hw; ++h)
                        v += *reinterpret_cast<const floatx4*>(
                            tiles + (h + hw * turn) * R::kWaveLds + R::kTileLds + (idx * kTile + o * 4) * 4);
                    at = gi * a.rel_cap + (c0 + row) * kTile + o * 4;
                } else {
                    const int c = row % wide, idx = row / wide % per_wave, wv = row / wide / per_wave;
                    const int tile = c0 + wv / hw + idx * nwt;
                    v = *reinterpret_cast<const floatx4*>(tiles + wv * R::kWaveLds + R::kTileLds +
                                                          ((idx * wide + c) * kTile + o * 4) * 4);
                    at = ((gi * hw + wv % hw) * G + c) * a.rel_cap + tile * kTile + o * 4;
                    if (tile >= c1) at = kNowhere / 4;
                }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), rr, at * 4, 0, kStreamPolicy);
            }
        };

        int t = t0 + wt;
        int rows = load_rows(t);
        // the query heads of the wave's KV head, as columns (repeated)
        intx4 qf[NQ];
        {
            const auto rq = buffer((const char*)a.q + (size_t)b * a.Hq * R::kBytes, a.Hq * R::kBytes);
            const int qo = (g * G + c16 % G) * R::kBytes + q4 * 16;
#pragma unroll
            for (int s = 0; s < NQ; ++s) qf[s] = load16<0>(rq, qo + s * 64);
        }
        // the new token's rows, for the wave whose tile holds it
        const int t_new = n_cached / kTile;
        const bool owns_new = t_new >= t0 && t_new < t1 && (t_new - t0) % nwt == wt;
        intx4 k_new, v_new;
        int new_row;
        {
            const int span = a.B * a.Hkv * R::kBytes;
            const int no = owns_new && lane < R::kLanes ? (b * a.Hkv + g) * R::kBytes + piece : kNowhere;
            k_new = load16<0>(buffer(a.knew, span), no);
            v_new = load16<0>(buffer(a.vnew, span), no);
            new_row = __builtin_amdgcn_raw_buffer_load_b32(rl, owns_new ? n_cached * 4 : kNowhere, 0, 0);
        }
        intx4 kx[NL], vx[NL];
        int off[NL];
        int next_rows = load_rows(t + nwt);
        row_offsets(t, rows, off);
        load_tile(rk, off, kx);
        load_tile(rv, off, vx);

        float m = -INFINITY, l = 0.f;             // of the lane's column (l: its own tokens)
        floatx4 acc[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) acc[k] = floatx4{0.f, 0.f, 0.f, 0.f};

        int c0 = t0;                              // first tile of the chunk
        for (;;) {
        const int c1 = min(t1, c0 + chunk);
        int kept = 0;
        for (; t < c1; t += nwt) {
            // K: registers -> LDS, then request the next tile's
#pragma unroll
            for (int j = 0; j < NL; ++j)
                *reinterpret_cast<intx4*>(kt + (j * kPer + lrow) * R::kKStride + piece) = kx[j];
            if (t == t_new && lane < R::kLanes)
                *reinterpret_cast<intx4*>(kt + (n_cached % kTile) * R::kKStride + piece) = k_new;
            __builtin_amdgcn_wave_barrier();
            rows = next_rows;
            next_rows = load_rows(t + 2 * nwt);
            row_offsets(t + nwt, rows, off);
            load_tile(rk, off, kx);

            // scores: rows = tokens 4 q4 + i (+ 16), column = the lane's head
            // several shorter chains, added at the end: less rounding, less latency
            constexpr int kChains = BF16 ? 2 : 4;
            floatx4 s[NBLK], sp[NBLK][kChains] = {};
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
#pragma unroll
                for (int blk = 0; blk < NBLK; ++blk) {
                    const intx4 kr = *reinterpret_cast<const intx4*>(kt + (blk * 16 + c16) * R::kKStride +
                                                                     k * 64 + q4 * 16);
                    if constexpr (BF16) {
                        sp[blk][k % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, kr), __builtin_bit_cast(bf16x8, qf[k]), sp[blk][k % 2], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sp[blk][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                __int_as_float(kr[e]), __int_as_float(qf[k][e]), sp[blk][e], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk) {
                s[blk] = sp[blk][0] + sp[blk][1];
                if constexpr (!BF16) s[blk] += sp[blk][2] + sp[blk][3];
            }
            // V: the same, in the same place
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < NL; ++j)
                *reinterpret_cast<intx4*>(vt + (j * kPer + lrow) * R::kVStride + piece) = vx[j];
            if (t == t_new && lane < R::kLanes)
                *reinterpret_cast<intx4*>(vt + (n_cached % kTile) * R::kVStride + piece) = v_new;
            __builtin_amdgcn_wave_barrier();
            load_tile(rv, off, vx);

            float y[NBLK][4];
            const int left = nb - t * kTile - q4 * 4;     // tokens from the lane's first one on
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    y[blk][i] = blk * 16 + i < left ? s[blk][i] * a.scale_log2 : -INFINITY;
            // relevance: the sum of |q.k| over the KV head's query heads (neighbouring
            // columns), or the logits themselves.  Entries past the list's end are
            // kept too (the planes have room, nothing reads them).
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk) {
                floatx4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float r = fabsf(s[blk][i]);
                    if constexpr (G >= 2) r += dpp_mov<0xB1>(r);     // quad_perm [1,0,3,2]
                    if constexpr (G >= 4) r += dpp_mov<0x4E>(r);     // quad_perm [2,3,0,1]
                    if constexpr (G >= 8) r += dpp_mov<0x141>(r);    // row_half_mirror
                    v[i] = rel_abs ? r : y[blk][i];
                }
                if (keeps)
                    *reinterpret_cast<floatx4*>(rel_kept + (kept * wide + c16) * kTile + blk * 16 + q4 * 4) = v;
            }
            ++kept;
            // online softmax
            float top = y[0][0];
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
                for (int i = 0; i < 4; ++i) top = fmaxf(top, y[blk][i]);
            // any new maximum rescales the sums: no weight passes 1, so the sums stay
            // within the tokens' number times the largest value
            if (__any(top > m)) {
                const float mn = fmaxf(m, column_max(top));
                const float sc = m < mn ? __builtin_amdgcn_exp2f(m - mn) : 1.f;
                l *= sc;
                m = mn;
                float row_sc[4];                  // the scale of row 4 q4 + i: head (4 q4 + i) % G
                unroll<4>([&](auto I) __attribute__((always_inline)) {
                    constexpr int i = decltype(I)::value;
                    const int x = row_bcast<i % G>(__float_as_int(sc));
                    if constexpr (G == 8) {
                        const int y = row_bcast<4 + i>(__float_as_int(sc));
                        row_sc[i] = __int_as_float(q4 & 1 ? y : x);
                    } else {
                        row_sc[i] = __int_as_float(x);
                    }
                });
#pragma unroll
                for (int k = 0; k < NB; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[k][i] *= row_sc[i];
            }
            float p[NBLK][4];
            const float mr = reference(m);
#pragma unroll
            for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    p[blk][i] = __builtin_amdgcn_exp2f(y[blk][i] - mr);
                    l += p[blk][i];
                }
            if constexpr (BF16) {
                // the lane's part of every weight, as the rows of P
                int pw[2 * NBLK], pw2[2 * NBLK];
#pragma unroll
                for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {
                        uint32_t u[2], u2[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            float f = p[blk][i + e];
                            if constexpr (kTwice) {
                                const float hi = __uint_as_float(__float_as_uint(f) & 0xFFFF0000u);
                                const float rest = f - hi;
                                const float lo = rest - __uint_as_float(__float_as_uint(rest) & 0xFFFF0000u);
                                u[e] = __float_as_uint(mask1 ? rest : f);
                                u2[e] = __float_as_uint(mask1 ? lo : f * 0x1p-30f);
                            } else {
                                f -= __uint_as_float(__float_as_uint(f) & mask1);
                                f -= __uint_as_float(__float_as_uint(f) & mask2);
                                u[e] = __float_as_uint(f);
                            }
                        }
                        pw[blk * 2 + i / 2] = (int)__builtin_amdgcn_perm(u[1], u[0], 0x07060302u);
                        if constexpr (kTwice) pw2[blk * 2 + i / 2] = (int)__builtin_amdgcn_perm(u2[1], u2[0], 0x07060302u);
                    }
                // V's columns: 4 tokens per transposed read (rows 4 q4 .. 4 q4 + 3 of a block)
                const char* vb = vt + (q4 * 4 + c16 / 4) * R::kVStride + (c16 % 4) * 8;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    auto column = [&](int blk) __attribute__((always_inline)) {
                        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_shortx4)(vb + blk * 16 * R::kVStride + k * 32));
                    };
                    if constexpr (NBLK == 1) {
                        const shortx4 v = column(0);
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                            __builtin_bit_cast(shortx4, intx2{pw[0], pw[1]}), v, acc[k], 0, 0, 0);
                        if constexpr (kTwice)
                            acc[k] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                                __builtin_bit_cast(shortx4, intx2{pw2[0], pw2[1]}), v, acc[k], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int j = 0; j < NBLK; j += 2) {
                            const bf16x8 v = __builtin_bit_cast(
                                bf16x8, __builtin_shufflevector(column(j), column(j + 1), 0, 1, 2, 3, 4, 5, 6, 7));
                            const int* w = pw + 2 * j;
                            acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, intx4{w[0], w[1], w[2], w[3]}), v, acc[k], 0, 0, 0);
                            if constexpr (kTwice) {
                                const int* w2 = pw2 + 2 * j;
                                acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8, intx4{w2[0], w2[1], w2[2], w2[3]}), v, acc[k], 0, 0, 0);
                            }
                        }
                    }
                }
            } else {
                // the tile's sums apart, then added: a chain of one addition per tile
                // instead of per token keeps the rounding error down
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    floatx4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int blk = 0; blk < NBLK; ++blk)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float v = *reinterpret_cast<const float*>(
                                vt + (blk * 16 + q4 * 4 + i) * R::kVStride + (k * 16 + c16) * 4);
                            part = __builtin_amdgcn_mfma_f32_16x16x4f32(p[blk][i], v, part, 0, 0, 0);
                        }
                    acc[k] += part;
                }
            }
        }
        if (c1 == t1) break;
        lds_barrier();
        store_kept(c0, c1);
        lds_barrier();
        c0 = c1;
        }
        if (owns_new && lane < R::kLanes) {       // the append
            const size_t dst = (pool_row0 + new_row) * R::kBytes + piece;
            *reinterpret_cast<intx4*>((char*)a.kpool_w + dst) = k_new;
            *reinterpret_cast<intx4*>((char*)a.vpool_w + dst) = v_new;
        }

        // ---- merge the waves: every wave's state (its head's G x D sums) into its own tile ----
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (lane < G) {
            ml_lds[(wave * 2) * G + lane] = m;
            ml_lds[(wave * 2 + 1) * G + lane] = l;
        }
        store_state<BF16, D, G>(acc, reinterpret_cast<float*>(kt), lane);
        lds_barrier();
        const int heads = hw * G;                 // query heads of the piece
        const size_t slot0 = (size_t)(slot - part) * heads;        // the pair's first partial
        const Finish fin{a.out + ((size_t)b * a.Hq + gi * heads) * D,
                         a.norm ? a.norm + ((size_t)b * a.Hq + gi * heads) * 2 : nullptr};
        // the partials as allocated: (workgroups x 8 KV heads + pairs) query heads, 40 MiB
        // at 256 workgroups, the widest token rows and 1024 sequences
        const auto rp = buffer(a.part_acc, a.part_heads * D * 4), rm = buffer(a.part_ml, a.part_heads * 8);
        // four dims of a head per thread
        for (int e = threadIdx.x * 4; e < heads * D; e += kThreads * 4) {
            const int hh = e / D, d = e % D;
            const int h = hh % G, h_kv = hh / G;
            float mw[kWaves], lw[kWaves];
            floatx4 ow[kWaves];
#pragma unroll
            for (int j = 0; j < kWaves; ++j) {    // every wave has a state, empty ones with m = -inf
                const int wv = min(h_kv + hw * j, kWaves - 1);
                mw[j] = j < nwt ? ml_lds[(wv * 2) * G + h] : -INFINITY;
                lw[j] = ml_lds[(wv * 2 + 1) * G + h];
                ow[j] = *reinterpret_cast<const floatx4*>(tiles + wv * R::kWaveLds + (h * (D + 4) + d) * 4);
            }
            float M = mw[0];
#pragma unroll
            for (int j = 1; j < kWaves; ++j) M = fmaxf(M, mw[j]);
            const float Mr = reference(M);
            float L = 0.f;
            floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < kWaves; ++j) {
                if (j < nwt) fold(L, o, __builtin_amdgcn_exp2f(mw[j] - Mr), lw[j], ow[j]);
            }
            if (n_parts == 1) {
                fin.template write<D>(hh, d, M, L, o);
            } else {
                const size_t slot_h = slot0 + (size_t)part * heads + hh;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, o), rp, (int)(slot_h * D + d) * 4, 0,
                                                       kAgentScope);
                if (d == 0)
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, floatx2{M, L}), rm,
                                                          (int)slot_h * 8, 0, kAgentScope);
            }
        }
        if (n_parts > 1) {
            // the device-scope stores of every thread have completed before the
            // ticket is taken, so no cache-wide write-back is needed
            __builtin_amdgcn_s_waitcnt(0);
            lds_barrier();
            if (threadIdx.x == 0)
                last_arrival = __hip_atomic_fetch_add(a.ticket + pair, 1, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT) == n_parts - 1;
            lds_barrier();
            if (last_arrival) {
                // The pair's partials, read at device scope (they may sit in another
                // XCD's L2).  kSlotGroups groups of threads each fold every
                // kSlotGroups-th slot, all loads of a pass in flight, and the groups'
                // states are folded in order: one or two round trips for the 16 to
                // 32 parts of a lone sequence.  A group spans one KV head's outputs, or
                // eight heads' where that takes fewer round trips (several heads, few
                // parts): with one head's, eight heads in turn took a round trip each (70
                // sequences of 600 tokens, 32 heads of 64: 76.6 us a launch, 67.5 now).
                constexpr int kPass = 4;
                auto fold_parts = [&](auto WIDE) __attribute__((always_inline)) {
                using F = Fold<G, D, decltype(WIDE)::value>;
                constexpr int kFoldThreads = F::kSpan, kSlotGroups = F::kSlotGroups;
                const int grp = threadIdx.x / kFoldThreads;
                // a thread's state, in its wave's tile (the relevance values are still kept)
                auto fold_o = [&](int th) { return reinterpret_cast<floatx4*>(tiles + th / 64 * R::kWaveLds) + th % 64; };
                auto fold_ml = [&](int th) { return reinterpret_cast<float*>(tiles + th / 64 * R::kWaveLds + 1024) + th % 64 * 2; };
                for (int e0 = 0; e0 < heads * D; e0 += kFoldThreads * 4) {
                    const int mine = e0 + threadIdx.x % kFoldThreads * 4;
                    const int e = min(mine, heads * D - 4);          // the others repeat the last
                    const int hh = e / D, d = e % D;
                    float M = -INFINITY, L = 0.f;
                    floatx4 o = {0.f, 0.f, 0.f, 0.f};
                    for (int k = grp; k < n_parts && grp < kSlotGroups; k += kSlotGroups * kPass) {
                        floatx2 pml[kPass];
                        floatx4 po[kPass];
#pragma unroll
                        for (int u = 0; u < kPass; ++u) {
                            const size_t slot_h = slot0 + (size_t)min(k + u * kSlotGroups, n_parts - 1) * heads + hh;
                            pml[u] = __builtin_bit_cast(floatx2, __builtin_amdgcn_raw_buffer_load_b64(
                                rm, (int)slot_h * 8, 0, kAgentScope));
                            po[u] = __builtin_bit_cast(floatx4, load16<kAgentScope>(rp, (int)(slot_h * D + d) * 4));
                        }
                        float Mn = M;
#pragma unroll
                        for (int u = 0; u < kPass; ++u)
                            if (k + u * kSlotGroups < n_parts) Mn = fmaxf(Mn, pml[u][0]);
                        const float Mr = reference(Mn), sc = __builtin_amdgcn_exp2f(M - Mr);
                        L *= sc;
                        o *= sc;
#pragma unroll
                        for (int u = 0; u < kPass; ++u)
                            if (k + u * kSlotGroups < n_parts)
                                fold(L, o, __builtin_amdgcn_exp2f(pml[u][0] - Mr), pml[u][1], po[u]);
                        M = Mn;
                    }
                    if constexpr (kSlotGroups > 1) {
                        lds_barrier();
                        fold_ml(threadIdx.x)[0] = M;
                        fold_ml(threadIdx.x)[1] = L;
                        *fold_o(threadIdx.x) = o;
                        lds_barrier();
                        if (grp == 0) {
                            float Mt = M;
#pragma unroll
                            for (int k = 1; k < kSlotGroups; ++k)
                                Mt = fmaxf(Mt, fold_ml(threadIdx.x + k * kFoldThreads)[0]);
                            const float Mr = reference(Mt), s0 = __builtin_amdgcn_exp2f(M - Mr);
                            L *= s0;
                            o *= s0;
#pragma unroll
                            for (int k = 1; k < kSlotGroups; ++k) {
                                const int src = threadIdx.x + k * kFoldThreads;
                                fold(L, o, __builtin_amdgcn_exp2f(fold_ml(src)[0] - Mr), fold_ml(src)[1], *fold_o(src));
                            }
                            M = Mt;
                        }
                    }
                    if (grp == 0 && mine < heads * D) fin.template write<D>(hh, d, M, L, o);
                }
                };
                if (hw == 1 || Fold<G, D, 1>::trips(heads, n_parts, kPass) <= Fold<G, D, 8>::trips(heads, n_parts, kPass))
                    fold_parts(std::integral_constant<int, 1>{});
                else
                    fold_parts(std::integral_constant<int, 8>{});
                if (threadIdx.x == 0) a.ticket[pair] = 0;      // ready for the next launch
            }
        }
        store_kept(c0, t1);
        lds_barrier();                           // the wave states have been read: tiles may be rewritten
    }
    }
}

template <bool BF16, int D, int G>
size_t lds_bytes(int B) {
    using R = Row<BF16, D>;
    return (size_t)R::kWaves * R::kWaveLds + R::kWaves * 2 * G * 4 + (B > 64 ? (size_t)(2 * B + 1) * 4 : 0);
}

// Timing events, when given, are recorded by the dispatch itself, so they
// bracket the kernel's execution and not the queue work around it.
struct Launch {
    int grid;
    hipStream_t stream;
    hipEvent_t start, stop;
    int* occ;                       // non-null: report occupancy instead
};

template <bool BF16, int D, int G>
hipError_t launch_t(const AttnArgs& a, const Launch& l) {
    const size_t lds = lds_bytes<BF16, D, G>(a.B);
    constexpr int threads = threads_of<BF16, D>();
    auto k = attention_kernel<BF16, D, G>;
    if (l.occ) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(l.occ, k, threads, lds);
    }
    AttnArgs arg = a;
    void* args[] = {&arg};
    return hipExtLaunchKernel(reinterpret_cast<const void*>(k), dim3(l.grid), dim3(threads),
                              args, lds, l.stream, l.start, l.stop, 0);
}

template <bool BF16, int D>
hipError_t launch_g(const AttnArgs& a, int group, const Launch& l) {
    switch (group) {
        case 1: return launch_t<BF16, D, 1>(a, l);
        case 2: return launch_t<BF16, D, 2>(a, l);
        case 4: return launch_t<BF16, D, 4>(a, l);
        case 8: return launch_t<BF16, D, 8>(a, l);
    }
    return hipErrorInvalidValue;
}

hipError_t dispatch(const AttnArgs& a, int dtype_bf16, int head_dim, int group, const Launch& l) {
    if (dtype_bf16) {
        if (head_dim == 128) return launch_g<true, 128>(a, group, l);
        if (head_dim == 64) return launch_g<true, 64>(a, group, l);
        if (head_dim == 256) return launch_g<true, 256>(a, group, l);
    } else {
        if (head_dim == 128) return launch_g<false, 128>(a, group, l);
        if (head_dim == 64) return launch_g<false, 64>(a, group, l);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The head layouts of the interface: token rows (every KV head) of at most
// 8 KiB and at most 64 query heads.
bool attention_shape_supported(int dtype_bf16, int head_dim, int group, int n_kv_heads) {
    if (head_dim != 64 && head_dim != 128 && head_dim != 256) return false;
    if (head_dim == 256 && !dtype_bf16) return false;
    if (group != 1 && group != 2 && group != 4 && group != 8) return false;
    return n_kv_heads * head_dim * (dtype_bf16 ? 2 : 4) <= 8192 && group * n_kv_heads <= 64;
}

hipError_t launch_attention(const AttnArgs& a, int dtype_bf16, int head_dim, int group,
                            int grid, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    return dispatch(a, dtype_bf16, head_dim, group, Launch{grid, s, start, stop, nullptr});
}

hipError_t attention_occupancy(const AttnArgs& a, int dtype_bf16, int head_dim, int group,
                               int* blocks_per_cu) {
    return dispatch(a, dtype_bf16, head_dim, group, Launch{0, nullptr, nullptr, nullptr, blocks_per_cu});
}

}  // namespace asrkf
