// Merge of split-KV partial states into the final output.
//
// Each split s of a query row holds the state of the online-softmax recurrence (Section 4.1.2,
// Eqs. 2-4) after its own run of key tiles: a reference m_s (log2 units of the scaled scores), the
// normaliser l_s and the unnormalised output o_s, both taken against m_s.  Because Eqs. 3-4 only ever
// rescale by e^{m_old - m_new}, states over disjoint key ranges combine the same way:
//     M = max_s m_s,   w_s = 2^(m_s - M),   L = sum_s w_s l_s,   O = (sum_s w_s o_s) / L,
// and O_i = o_i / l_i as at the end of Section 4.1.2; LSE = (M + log2 L) ln 2.  A split that saw no
// key of the row has (m, l) = (-inf, 0), weight 0, and an o that is not looked at; one that saw only scores of -inf or NaN
// has the lowest finite m and l = 0 or NaN (O is NaN if all splits are like that).
//
// Workspace layout (written by sdpa_fwd_kernel<..., KV = true>): o as float [BH][splits][S][D],
// then (m, l) pairs as float [BH][splits][S][2].
//
// Two kernels.  sdpa_merge_kernel: one thread produces 4 consecutive output columns and takes the splits itself; right for up to
// eight splits, and for any split count when the rows are many (a long prefill chunk), where the other threads hide the waiting.
// sdpa_merge_wide_kernel: one workgroup per output row, kMergeLanes threads per column group that
// take every kMergeLanes-th split each and combine through the LDS; for the many splits of a decoding
// step, where rows are few and a walk over 32 splits would be a chain of load latencies longer than
// the attention kernel itself.  Both sum in a fixed order (results do not depend on timing).
//
// Both are bound by latency: a launch, and as many round trips to memory as there are loads that wait for one another.  So all
// loads of a thread are issued before the first use, those of splits that do not exist aimed at the last one, and the empty asm
// after them says so: a load that only a condition needs is moved behind that condition.  And the
// addresses hold no 64-bit division (a launch's grid gives the head, or 32 bits do).  The whole call in us, before that -> now: 8
// heads of 4 rows, 8192 keys D = 128 in 32 splits 12.3 -> 11.6; 4 heads of 64 rows, 4000 keys D = 64 in 3 splits 11.7 -> 10.5, in 16
// 8.5 -> 7.9; 8 heads of 512 rows, 2048 keys D = 64 in 7 splits 19.0 -> 16.9; 128 rows D = 160 in 9 21.0 -> 17.3; 2048 rows in
// 9, where the bytes bound it, level.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsdpa {

// blockDim = (D / 4, 256 / (D / 4)); ONCE: most splits that are taken at once, 0: any number, four at a time.
template <typename T, int ONCE>
__global__ void __launch_bounds__(256)
sdpa_merge_kernel(const float *__restrict__ ws, T *__restrict__ o, float *__restrict__ lse,
                  unsigned rows, unsigned S, int D, int splits)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef T vec4 __attribute__((ext_vector_type(4)));
    constexpr int BATCH = ONCE > 0 ? ONCE : 4;
    const int d4 = threadIdx.x;
    const unsigned r = blockIdx.x * blockDim.y + threadIdx.y;       // bh * S + row
    if (r >= rows) return;
    const unsigned bh = r / S, row = r - bh * S;
    const size_t first = (size_t)bh * splits * S + row;             // split s sits s*S rows further on
    const float *ml = ws + (size_t)rows * splits * D + first * 2, *po = ws + first * D + d4 * 4;

    float M = -INFINITY;
    if constexpr (ONCE == 0)
        for (int s0 = 0; s0 < splits; s0 += 8) {
            float m[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) m[i] = ml[(size_t)(s0 + i < splits ? s0 + i : splits - 1) * S * 2];
#pragma unroll
            for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(m[i]));
#pragma unroll
            for (int i = 0; i < 8; ++i) M = fmaxf(M, m[i]);
        }
    float L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // (four splits at a time: this kernel, us, each load behind a condition / four at a time / eight: 4096 rows of D = 160,
    // 16 splits 17.1 / 9.2 / 9.7; 8192 of D = 128, 8 splits 10.9 / 8.3 / 8.2)
    for (int s0 = 0; s0 < splits; s0 += BATCH) {
        f32x2 st[BATCH];
        f32x4 part[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const size_t p = (size_t)(s0 + i < splits ? s0 + i : splits - 1) * S;
            st[i] = *(const f32x2 *)(ml + p * 2);
            part[i] = *(const f32x4 *)(po + p * D);
        }
#pragma unroll
        for (int i = 0; i < BATCH; ++i) asm volatile("" : "+v"(st[i]), "+v"(part[i]));
        if constexpr (ONCE > 0) {
#pragma unroll
            for (int i = 0; i < BATCH; ++i) M = fmaxf(M, st[i][0]);
        }
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            if (s0 + i >= splits) break;
            // 0 for a split with m = -inf; M itself is -inf only for a row that no key reaches (an empty
            // cache entry, or a causal limit before the first key): all weights 0, O = 0, LSE = -inf
            const float e = __builtin_amdgcn_exp2f(st[i][0] - M), w = M == -INFINITY ? 0.f : e;
            L += w * st[i][1];
            // (a split without keys, l = 0, may have left its o unwritten; a NaN row has l = NaN)
            const f32x4 sum = acc + w * part[i];
            const bool keys = st[i][1] != 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = keys ? sum[c] : acc[c];
        }
        if constexpr (ONCE > 0) break;
    }
    const float inv = M == -INFINITY ? 0.f : 1.0f / L;
    vec4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = (T)(acc[e] * inv);
    *(vec4 *)(o + (size_t)r * D + d4 * 4) = out;
    if (lse != nullptr && d4 == 0)
        lse[r] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * 0.69314718055994530942f : -INFINITY;
#endif
}

constexpr int kMergeLanes = 8;                  // threads that share one column group's splits
constexpr int kMergePerLane = 16;               // most splits per such thread: 8 * 16 = TSDPA_MAX_SPLITS
constexpr int kMergeMaxCols = 40;               // D / 4 at D = 160

// blockDim = (D / 4, kMergeLanes); grid = (S, BH).  PER: splits per thread, at most kMergePerLane.
template <typename T, int PER>
__global__ void __launch_bounds__(kMergeMaxCols * kMergeLanes)
sdpa_merge_wide_kernel(const float *__restrict__ ws, T *__restrict__ o, float *__restrict__ lse, int D, int splits)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef T vec4 __attribute__((ext_vector_type(4)));
    __shared__ f32x4 acc_sh[kMergeLanes][kMergeMaxCols];
    __shared__ f32x2 ml_sh[kMergeLanes];
    const int d4 = threadIdx.x, lane = threadIdx.y;
    const unsigned S = gridDim.x;
    const unsigned r = blockIdx.y * S + blockIdx.x;
    // byte offsets of 32 bits: at most 2048 rows of 128 splits
    const char *ml = (const char *)(ws + (size_t)gridDim.y * S * splits * D), *po = (const char *)ws;
    const unsigned first = blockIdx.y * splits * S + blockIdx.x;       // split s sits s*S rows further on

    // this thread's splits: lane, lane + 8, ...
    f32x2 st[PER];
    f32x4 part[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int s = lane + i * kMergeLanes;
        const unsigned p = first + (s < splits ? s : splits - 1) * S;
        st[i] = *(const f32x2 *)(ml + p * 8u);
        part[i] = *(const f32x4 *)(po + (p * D + d4 * 4) * 4u);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) asm volatile("" : "+v"(st[i]), "+v"(part[i]));
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (lane + i * kMergeLanes >= splits) st[i] = f32x2{-INFINITY, 0.f};
    // combined against their own maximum
    float m_own = -INFINITY;
#pragma unroll
    for (int i = 0; i < PER; ++i) m_own = fmaxf(m_own, st[i][0]);
    float l_own = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        // weight 0 for a split with m = -inf (it saw no key of the row, or does not exist)
        const float w = st[i][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(st[i][0] - m_own);
        l_own += w * st[i][1];
        // (a split without keys, l = 0, may have left its o unwritten; a NaN row has l = NaN)
        const f32x4 sum = acc + w * part[i];
        const bool keys = st[i][1] != 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = keys ? sum[c] : acc[c];
    }
    acc_sh[lane][d4] = acc;
    if (d4 == 0) ml_sh[lane] = f32x2{m_own, l_own};
    __syncthreads();
    if (lane != 0) return;
    // the kMergeLanes states of this column group, in lane order
    float M = -INFINITY;
#pragma unroll
    for (int y = 0; y < kMergeLanes; ++y) M = fmaxf(M, ml_sh[y][0]);
    float L = 0.f;
    f32x4 out_acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int y = 0; y < kMergeLanes; ++y) {
        const float w = ml_sh[y][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml_sh[y][0] - M);
        L += w * ml_sh[y][1];
        out_acc += w * acc_sh[y][d4];
    }
    // M is -inf only for a row that no key reaches: all weights 0, O = 0, LSE = -inf
    const float inv = M == -INFINITY ? 0.f : 1.0f / L;
    vec4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = (T)(out_acc[e] * inv);
    *(vec4 *)(o + (size_t)r * D + d4 * 4) = out;
    if (lse != nullptr && d4 == 0)
        lse[r] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * 0.69314718055994530942f : -INFINITY;
#endif
}

}  // namespace tsdpa
