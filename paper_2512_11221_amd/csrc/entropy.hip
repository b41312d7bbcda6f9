// The first launch of a step's end: the entropy monitors with the recovery
// ladder (Sec. 3.6), and the score verdicts that the freeze loop reads.  The
// two are independent and neither fills the device, so they share a launch:
// the first workgroups take the entropy, the others the verdicts.
//
// Entropy.
//
// a.split workgroups per sequence, one pass over the V logits.  Each
// thread forms (m, S, T) with S = sum e^(x-m) and T = sum e^(x-m) (x-m) over
// its logits (all loads of a round in flight together, the round's maximum
// first); the triples are merged across the block and stored.  The last
// block of a sequence to finish (a per-sequence ticket) loads the stored
// triples, one per lane, merges them in a fixed lane tree and forms
//     H = ln S - T / S          (nats, softmax at temperature 1)
//     p_max = 1 / S,
// A logit of -inf has probability 0 and adds nothing; a row with no finite
// logit has no distribution: its entropy is NaN and it triggers nothing.
// Then the kernel updates the sequence's escalation count (one level per consecutive
// spike step, reset by a calm step) and writes the level that the end-of-step
// compaction applies: 1 SR, 2 WR, 3 FR; a count above 3 also records a
// Rewalk Regeneration request.
//
// Verdicts.  The attention launches leave, per attended token (in list order),
// one value per plane: the KV heads' sums of |q.k|, or every query head's
// logit y (softmax reading).  A token's score is
//     H s_j = sum_g rel_gj            (Eq. 2), or
//     H s_j = sum_h 2^(y_hj - M_h) / L_h,
// with (M_h, L_h) the head's softmax normaliser, summed over every layer in
// token scope.  It is compared with tau and the flag byte is stored at the
// token's position.  Four list entries per thread: 16-byte loads of a plane,
// the planes of a group in flight together.
#include "kernels.h"

namespace asrkf {
namespace {

constexpr int kThreads = 256;

struct Triple {
    float m, S, T;
};

__device__ __forceinline__ Triple merge(const Triple& a, const Triple& b) {
    if (b.S == 0.f) return a;
    if (a.S == 0.f) return b;
    constexpr float kLog2e = 1.4426950408889634f;
    const float m = fmaxf(a.m, b.m);
    const float da = a.m - m, db = b.m - m;
    const float ea = __builtin_amdgcn_exp2f(da * kLog2e), eb = __builtin_amdgcn_exp2f(db * kLog2e);
    Triple r;
    r.m = m;
    r.S = ea * a.S + eb * b.S;
    r.T = ea * (a.T + da * a.S) + eb * (b.T + db * b.S);
    return r;
}

// (m, S, T) of a thread's logits: its maximum first, then one pass with
// e = exp(x - m) (as exp2 of pre-scaled differences), no data-dependent branch.
template <int N>
__device__ __forceinline__ Triple triple_of(const float (&x)[N], const bool (&ok)[N]) {
    constexpr float kLog2e = 1.4426950408889634f;
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < N; ++i) m = ok[i] ? fmaxf(m, x[i]) : m;
    // no finite logit: an empty triple (a -inf logit has probability 0)
    if (m == -INFINITY) return Triple{-INFINITY, 0.f, 0.f};
    float S = 0.f, T = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float d = x[i] - m;
        const float e = ok[i] ? __builtin_amdgcn_exp2f(d * kLog2e) : 0.f;
        S += e;
        // a term with e = 0 adds nothing (0 ln 0 = 0), also where d = -inf
        T = fmaf(e, (ok[i] && e > 0.f) ? d : 0.f, T);
    }
    return Triple{m, S, T};
}

constexpr int kVec = 4;             // float4 loads per thread per round

__device__ void entropy_block(const EntropyArgs& a, int sp, int b) {
    __shared__ Triple part[kThreads / 64];
    __shared__ int last;
    const float* x = a.logits + (size_t)b * a.V;
    Triple acc{-INFINITY, 0.f, 0.f};
    // 16-byte loads from the row's first 16-byte boundary on (rows start anywhere when
    // the vocabulary is no multiple of 4); the few logits before and after it go to
    // the first workgroup.  At a vocabulary of 50257 and batch 32 the launch took
    // 15.0 us with one logit per load and takes 10.2 us.
    const int head = min(a.V, (int)((16 - (reinterpret_cast<uintptr_t>(x) & 15)) & 15) / 4);
    const int n4 = (a.V - head) / 4;
    const int tail = a.V - head - 4 * n4;
    const int i0 = (int)((int64_t)sp * n4 / a.split), i1 = (int)((int64_t)(sp + 1) * n4 / a.split);
    // all of a round's loads are issued before any of them is used
    for (int base = i0; base < i1; base += kThreads * kVec) {
        float v[4 * kVec];
        bool ok[4 * kVec];
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
            const int i = base + u * kThreads + threadIdx.x;
            const bool in = i < i1;
            typedef float f4 __attribute__((ext_vector_type(4)));
            const f4 f = in ? __builtin_nontemporal_load(reinterpret_cast<const f4*>(x + head) + i)
                            : f4{0.f, 0.f, 0.f, 0.f};
            v[4 * u] = f.x; v[4 * u + 1] = f.y; v[4 * u + 2] = f.z; v[4 * u + 3] = f.w;
            ok[4 * u] = ok[4 * u + 1] = ok[4 * u + 2] = ok[4 * u + 3] = in;
        }
        acc = merge(acc, triple_of(v, ok));
    }
    if (sp == 0 && head + tail > 0) {
        const int t = threadIdx.x;
        const bool ok[1] = {t < head + tail};
        const float v[1] = {ok[0] ? x[t < head ? t : 4 * n4 + t] : 0.f};
        acc = merge(acc, triple_of(v, ok));
    }
    for (int o = 32; o > 0; o >>= 1) {
        Triple other{__shfl_xor(acc.m, o), __shfl_xor(acc.S, o), __shfl_xor(acc.T, o)};
        acc = merge(acc, other);
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        Triple r = part[0];
        for (int w = 1; w < kThreads / 64; ++w) r = merge(r, part[w]);
        float* dst = a.partial + ((size_t)b * a.split + sp) * 3;
        __hip_atomic_store(dst, r.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dst + 1, r.S, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dst + 2, r.T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // the device-scope stores above have completed before the ticket is taken,
        // so no cache-wide write-back is needed
        __builtin_amdgcn_s_waitcnt(0);
        last = (__hip_atomic_fetch_add(a.ticket + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                == a.split - 1);
    }
    __syncthreads();
    if (!last || threadIdx.x >= 64) return;
    // the blocks' triples, one per lane, read at device scope (they may sit in
    // another XCD's L2); merged in a fixed lane tree, so every run rounds alike
    static_assert(kEntropySplitMax <= 64, "one triple per lane");
    const float* src = a.partial + (size_t)b * a.split * 3;
    const int k = threadIdx.x;
    Triple r{-INFINITY, 0.f, 0.f};
    if (k < a.split) {
        r.m = __hip_atomic_load(src + 3 * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r.S = __hip_atomic_load(src + 3 * k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        r.T = __hip_atomic_load(src + 3 * k + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int o = 1; o < 64; o <<= 1) {
        Triple other{__shfl_xor(r.m, o), __shfl_xor(r.S, o), __shfl_xor(r.T, o)};
        r = (k & o) ? merge(other, r) : merge(r, other);
    }
    if (k != 0) return;
    a.ticket[b] = 0;                           // ready for the next step
    const float H = logf(r.S) - r.T / r.S;
    const float pmax = 1.f / r.S;
    SeqMonitor& mon = a.monitor[b];
    mon.entropy = H;
    mon.pmax = pmax;
    int level = 0;
    if (a.mode == 0) {
        const bool spike = (H > a.theta_H) || (a.theta_p > 0.f && pmax < a.theta_p);
        const int esc = spike ? mon.escalation + 1 : 0;
        mon.escalation = esc;
        level = min(esc, 3);
        if (esc > 3) atomicAdd(a.rr_requests, 1ull);
    } else if (a.mode >= 1 && a.mode <= 3) {
        level = a.mode;
    }
    mon.level = level;
    if (level > 0) atomicAdd(a.recoveries + level, 1ull);
}

constexpr int kEntries = 4 * kThreads;        // list entries per verdict workgroup
constexpr int kPlaneGroup = 4;

// CARRY: a token-scope step whose layers are judged by several launches.
template <bool CARRY>
__device__ void verdict_block(const VerdictArgs& v, int chunk, int inst) {
    const int n = min(v.n_active[inst], v.rel_cap);      // more only where device rows ran out
    const int i0 = chunk * kEntries + 4 * threadIdx.x;
    if (i0 >= n) return;
    const int b = inst % v.B, state = inst / v.B;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (CARRY && v.add_sum) {
        const float4 before = *reinterpret_cast<const float4*>(v.sum + (size_t)b * v.rel_cap + i0);
        s[0] = before.x; s[1] = before.y; s[2] = before.z; s[3] = before.w;
    }
    const int4 pos = *reinterpret_cast<const int4*>(v.list + (size_t)inst * v.cap + i0);
    for (int l = 0; l < v.layers_summed; ++l) {
        const size_t li = (size_t)(state + l) * v.B + b;          // the layer's instance
        const float* rel = v.rel + li * v.planes * v.rel_cap + i0;
        const float* norm = v.norm + li * v.planes * 2;
        for (int p0 = 0; p0 < v.used; p0 += kPlaneGroup) {
            float4 x[kPlaneGroup];
#pragma unroll
            for (int k = 0; k < kPlaneGroup; ++k)
                x[k] = *reinterpret_cast<const float4*>(rel + (size_t)min(p0 + k, v.used - 1) * v.rel_cap);
#pragma unroll
            for (int k = 0; k < kPlaneGroup; ++k) {
                if (p0 + k < v.used) {
                    if (v.softmax) {
                        const float M = norm[2 * (p0 + k)], inv = 1.f / norm[2 * (p0 + k) + 1];
                        s[0] = fmaf(__builtin_amdgcn_exp2f(x[k].x - M), inv, s[0]);
                        s[1] = fmaf(__builtin_amdgcn_exp2f(x[k].y - M), inv, s[1]);
                        s[2] = fmaf(__builtin_amdgcn_exp2f(x[k].z - M), inv, s[2]);
                        s[3] = fmaf(__builtin_amdgcn_exp2f(x[k].w - M), inv, s[3]);
                    } else {
                        s[0] += x[k].x;
                        s[1] += x[k].y;
                        s[2] += x[k].z;
                        s[3] += x[k].w;
                    }
                }
            }
        }
    }
    if (CARRY && v.keep_sum) {
        *reinterpret_cast<float4*>(v.sum + (size_t)b * v.rel_cap + i0) = make_float4(s[0], s[1], s[2], s[3]);
        return;
    }
    uint8_t* flag = v.flag + (size_t)inst * v.cap;
    const int p[4] = {pos.x, pos.y, pos.z, pos.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (i0 + k < n)
            flag[p[k]] = (uint8_t)((s[k] < v.tau_sum ? 1 : 0) | (fabsf(s[k] - v.tau_sum) < v.margin_sum ? 2 : 0));
}

template <bool CARRY>
__global__ void __launch_bounds__(kThreads)
monitor_kernel(EntropyArgs e, VerdictArgs v, int entropy_blocks, int chunks) {
    const int i = blockIdx.x;
    if (i < entropy_blocks) entropy_block(e, i % e.split, i / e.split);
    else verdict_block<CARRY>(v, (i - entropy_blocks) % chunks, (i - entropy_blocks) / chunks);
}

}  // namespace

hipError_t launch_monitor(const EntropyArgs* e, const VerdictArgs& v, hipStream_t s) {
    const int64_t entropy_blocks = e ? (int64_t)e->split * e->B : 0;
    const int64_t chunks = (v.rel_cap + kEntries - 1) / kEntries;
    const int64_t blocks = entropy_blocks + chunks * v.states * v.B;
    if (blocks > (1 << 30)) return hipErrorInvalidValue;   // caches of that size exceed any device
    const auto kernel = v.add_sum || v.keep_sum ? monitor_kernel<true> : monitor_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s,
                       e ? *e : EntropyArgs{}, v, (int)entropy_blocks, (int)chunks);
    return hipGetLastError();
}

}  // namespace asrkf
