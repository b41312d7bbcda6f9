// Row copies between the device KV cache and the pinned host store (spill
// mode; Sec. 3.2 moves frozen tokens' KV off the GPU and back).
//
// The lists of rows to move are made on the device by the end-of-step
// compaction, so the host never learns which tokens move: each launch walks
// the per-(layer, sequence) lists it is given and copies every listed token's
// K row and V row (n_kv_heads * head_dim elements each) one wave per token, 16
// bytes per lane.  The host store is position-indexed and token-major, the
// device cache row-indexed and head-major.  Loads of a token's K and
// V pieces are issued before its stores, so each wave keeps two rows in
// flight over the host link.
//
// The prompt copy (prefill) writes a prompt's rows into the head-major cache.
#include "kernels.h"

namespace asrkf {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / 64;
constexpr int kBlocksPerLaunch = 1024;

__global__ void __launch_bounds__(kThreads)
xfer_kernel(XferArgs a) {
    const int inst = a.inst0 + blockIdx.y;
    const int n = a.count[inst];
    const int lane = threadIdx.x & 63;
    const int w0 = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    const int wstride = gridDim.x * kWavesPerBlock;
    const int32_t* pos = a.pos + (size_t)inst * a.cap;
    const int32_t* row = a.row + (size_t)inst * a.cap;
    const size_t host0 = (size_t)inst * a.cap;
    const int head_bytes = a.row_bytes / a.Hkv;           // powers of two
    const int head_shift = __ffs(head_bytes) - 1;
    const size_t dev0 = (size_t)inst * a.pool_rows * a.Hkv;
    for (int i = w0; i < n; i += wstride) {
        const size_t h = (host0 + (size_t)pos[i]) * a.row_bytes;
        for (int o = lane * 16; o < a.row_bytes; o += 64 * 16) {
            const int g = o >> head_shift;
            const size_t d = ((dev0 + (size_t)g * a.pool_rows) + (size_t)row[i]) * head_bytes + (o - g * head_bytes);
            const uint4 kx = *reinterpret_cast<const uint4*>(a.to_host ? a.kpool + d : a.khost + h + o);
            const uint4 vx = *reinterpret_cast<const uint4*>(a.to_host ? a.vpool + d : a.vhost + h + o);
            *reinterpret_cast<uint4*>(a.to_host ? a.khost + h + o : a.kpool + d) = kx;
            *reinterpret_cast<uint4*>(a.to_host ? a.vhost + h + o : a.vpool + d) = vx;
        }
    }
}

// The rows of a prompt, [n][Hkv][row] -> [Hkv][pool_rows][row], K in the first
// half of the workgroups and V in the second.  A thread moves T-sized pieces
// (16 bytes; smaller ones when an input is not 16-byte aligned), several loads
// in flight; both sides are contiguous over a row, the source over a token.
constexpr int kCopyThreads = 256;
constexpr int kCopyUnroll = 4;

template <typename T>
__global__ void __launch_bounds__(kCopyThreads)
prefill_kernel(PrefillArgs a) {
    const int half = gridDim.x / 2;
    const bool second = (int)blockIdx.x >= half;
    const T* src = reinterpret_cast<const T*>(second ? a.v : a.k);
    T* dst = reinterpret_cast<T*>(second ? a.vdst : a.kdst);
    const unsigned per_row = a.row_bytes / sizeof(T);     // pieces per head row: a power of two
    const unsigned row_shift = __ffs((int)per_row) - 1, head_shift = __ffs(a.Hkv) - 1;
    const unsigned total = (unsigned)a.rows * a.Hkv * per_row; // below 2^31: a sequence's rows are
    const unsigned stride = half * kCopyThreads * kCopyUnroll;
    if (a.set_plen && blockIdx.x == 0 && threadIdx.x == 0) *a.plen = a.n;
    for (unsigned i0 = (second ? blockIdx.x - half : blockIdx.x) * kCopyThreads * kCopyUnroll + threadIdx.x;
         i0 < total; i0 += stride) {
        T x[kCopyUnroll];
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) {
            const unsigned i = i0 + u * kCopyThreads;
            if (i < total) x[u] = __builtin_nontemporal_load(src + i);
        }
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) {
            const unsigned i = i0 + u * kCopyThreads;
            if (i < total) {
                const unsigned e = i & (per_row - 1), row = i >> row_shift;
                const unsigned g = row & (a.Hkv - 1), p = row >> head_shift;
                __builtin_nontemporal_store(x[u], dst + ((size_t)g * a.pool_rows + p) * per_row + e);
            }
        }
    }
}

// Test hook: one wave that waits, without touching memory, until the given
// number of 100 MHz real-time ticks has passed.  It always ends.
__global__ void __launch_bounds__(64) delay_kernel(uint64_t ticks) {
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    while (__builtin_amdgcn_s_memrealtime() - t0 < ticks) __builtin_amdgcn_s_sleep(100);
}

}  // namespace

hipError_t launch_prefill(const PrefillArgs& a, hipStream_t s) {
    if (a.n < 1 || a.row_bytes % 16) return hipErrorInvalidValue;
    const uintptr_t low = reinterpret_cast<uintptr_t>(a.k) | reinterpret_cast<uintptr_t>(a.v);
    const int piece = (low & 15) == 0 ? 16 : (low & 3) == 0 ? 4 : (low & 1) == 0 ? 2 : 1;
    const size_t pieces = (size_t)a.rows * a.Hkv * a.row_bytes / piece;
    constexpr size_t kPerBlock = kCopyThreads * kCopyUnroll;
    size_t half = (pieces + kPerBlock - 1) / kPerBlock;
    if (half < 1) half = 1;
    if (half > 1024) half = 1024;                 // 8 workgroups per CU in all
    const dim3 grid((unsigned)(2 * half)), block(kCopyThreads);
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    if (piece == 16) hipLaunchKernelGGL(prefill_kernel<u4>, grid, block, 0, s, a);
    else if (piece == 4) hipLaunchKernelGGL(prefill_kernel<uint32_t>, grid, block, 0, s, a);
    else if (piece == 2) hipLaunchKernelGGL(prefill_kernel<uint16_t>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(prefill_kernel<uint8_t>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_delay(int microseconds, hipStream_t s) {
    if (microseconds <= 0) return hipSuccess;
    hipLaunchKernelGGL(delay_kernel, dim3(1), dim3(64), 0, s, (uint64_t)microseconds * 100u);
    return hipGetLastError();
}

hipError_t launch_xfer(const XferArgs& a, int n_instances, hipStream_t s) {
    if (n_instances < 1 || a.row_bytes % 16) return hipErrorInvalidValue;
    constexpr int kMaxY = 32768;                  // instances per launch (grid y limit)
    for (int i0 = 0; i0 < n_instances; i0 += kMaxY) {
        XferArgs part = a;
        part.inst0 = a.inst0 + i0;
        const int ni = n_instances - i0 < kMaxY ? n_instances - i0 : kMaxY;
        const int gx = (kBlocksPerLaunch + ni - 1) / ni;
        hipLaunchKernelGGL(xfer_kernel, dim3(gx, ni), dim3(kThreads), 0, s, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace asrkf
