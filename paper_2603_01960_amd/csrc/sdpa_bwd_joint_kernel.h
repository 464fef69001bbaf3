// Backward pass with dQ and dK + dV in one grid, after a launch for the statistics of the query rows.
//
// As launches of their own (sdpa_bwd_kernel.h) the two passes run one after the other, and where neither fills the card, or
// fills it with an uneven last round, the CUs wait: two launches of one round each, both as long as their longest chain of
// tiles.  In one grid they share the card.  Then the dQ pass cannot leave the statistics for the other any more; a launch
// before them computes them (3 us on small problems; on large ones the time to read O and dO, which is why most of those keep the
// passes apart: pick_bwd_joint in sdpa_bwd_pick.h).
// BF16, us per call, passes apart -> one grid: one head S = 1159 D = 64 20.9 -> 14.1, D = 128 34.4 -> 21.4, D = 160 52.7 -> 22.3;
// two entries of 16 heads over 2, S = 57, D = 128 20.4 -> 17.7; 8 heads over 2, S = 1346, D = 128 78 -> 60; 65 heads of S = 679, G = 4,
// D = 64 71.5 -> 58; 30 heads over 2, S = 2969, D = 128 277 -> 238.
#pragma once
#include "sdpa_bwd_kernel.h"
#include "sdpa_bwd_pair_kernel.h"

namespace tsdpa {

// Statistics of all query rows, -Delta and LSE in log2 units, into `stats`.  Four lanes per row, 64 rows per workgroup, from
// workgroup `short_heads` on; the workgroups before it take Delta of the rows that see at most kBwdShortRow keys from its
// definition, one per query head: wavefront 2 * b + j pairs the queries 32b ... with the keys 32j ... .
// TILED (for sdpa_bwd_chain_kernel.h): `pitch` rows per head, of which those past S get weights of 0; and `nclear` words at `clear` are cleared.
template <typename T, int D, bool TILED>
__global__ void __launch_bounds__(256)
sdpa_bwd_stats_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                      const T *__restrict__ o, const float *__restrict__ lse, float *__restrict__ stats, int rows, int S,
                      Divisor by_S, int group, float c, uint32_t rsign, int causal, unsigned stat_bytes, int short_heads,
                      unsigned *__restrict__ clear, int nclear, int pitch)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    constexpr int KK = D / 16, CPL = D / 32;      // k-steps; 16-byte chunks per lane of a quarter row
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float *lse2 = (float *)((char *)stats + stat_bytes);
    if constexpr (TILED) {
        for (int i = (int)blockIdx.x * 256 + tid; i < nclear; i += (int)gridDim.x * 256) clear[i] = 0;
        for (int h = (int)blockIdx.x; h < rows / S; h += (int)gridDim.x)
            if (tid < pitch - S) {
                stats[(size_t)h * pitch + S + tid] = 0.f;
                lse2[(size_t)h * pitch + S + tid] = __builtin_inff();
            }
    } else {
        pitch = S;
    }
    if ((int)blockIdx.x < short_heads) {
        __shared__ float part[4][32];
        const int head = blockIdx.x, g = lane >> 5, l32 = lane & 31, qb = wave >> 1, kb = wave & 1;
        const int row = qb * 32 + l32, row_c = row < S ? row : S - 1, key_c = kb * 32 + l32 < S ? kb * 32 + l32 : S - 1;
        const size_t qoff = ((size_t)head * S + row_c) * D + g * 8, koff = ((size_t)(head / group) * S + key_c) * D + g * 8;
        float sum = 0.f;
        const float l2 = lse[(size_t)head * S + row_c] * 1.44269504088896340736f;
        if (qb * 32 < S && kb * 32 < S && !(causal && kb > qb)) {
            u32x4 qr[KK], kr[KK], dr[KK], vr[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                qr[kk] = *(const u32x4 *)(q + qoff + kk * 16);
                kr[kk] = *(const u32x4 *)(k + koff + kk * 16);
                dr[kk] = *(const u32x4 *)(dout + qoff + kk * 16);
                vr[kk] = *(const u32x4 *)(v + koff + kk * 16);
            }
            f32x16 sacc, dpacc;
#pragma unroll
            for (int i = 0; i < 16; ++i) sacc[i] = dpacc[i] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                sacc = E::mfma(__builtin_bit_cast(vec8, kr[kk]), __builtin_bit_cast(vec8, qr[kk] ^ rsign), sacc);
                dpacc = E::mfma(__builtin_bit_cast(vec8, vr[kk]), __builtin_bit_cast(vec8, dr[kk]), dpacc);
            }
            const int last = causal ? row_c : S - 1;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int key = kb * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                if (key <= last) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -l2)) * dpacc[i];
            }
            sum = pair_sum(sum);
        }
        if (g == 0) part[wave][l32] = sum;
        __syncthreads();
        if (kb == 0 && g == 0 && row < S) {
            stats[(size_t)head * pitch + row] = -(sum + part[wave + 1][l32]);
            lse2[(size_t)head * pitch + row] = l2;
        }
        return;
    }
    const int row = ((int)blockIdx.x - short_heads) * 64 + (tid >> 2), part = tid & 3;
    if (row >= rows) return;
    const T *orow = o + (size_t)row * D + part * 8, *drow = dout + (size_t)row * D + part * 8;
    vec8 x[CPL], y[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        x[i] = *(const vec8 *)(orow + i * 32);
        y[i] = *(const vec8 *)(drow + i * 32);
    }
    const float l2 = lse[row] * 1.44269504088896340736f;
    float delta = 0.f;
#pragma unroll
    for (int i = 0; i < CPL; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) delta += (float)x[i][e] * (float)y[i][e];
    delta += __shfl_xor(delta, 1);
    delta += __shfl_xor(delta, 2);
    if (part == 0 && !(short_heads > 0 && row - divide(row, by_S) * S < kBwdShortRow)) {
        const size_t at = TILED ? (size_t)row + (size_t)divide(row, by_S) * (pitch - S) : row;
        stats[at] = -delta;
        lse2[at] = l2;
    }
#endif
}

// Both passes in one grid: a workgroup finds its pass and its number within it.  Where both have the same number of workgroups
// eight numbers of one pass (one per XCD) are followed by the same eight of the other; otherwise the keys-resident pass, whose
// chains are the longer ones, comes first.  NWQ, NSQ: wavefronts along the rows and streams of the dQ pass; NWK, NSK:
// those of the keys-resident one (D = 160: pairs and streams), with the same number of threads.
template <int D, int NSQ> constexpr int bwd_joint_tq() { return NSQ == 1 && (D == 64 || D == 128) ? 64 : 32; }
template <int D, int NSK> constexpr int bwd_joint_tk() { return NSK == 1 && D == 64 ? 64 : 32; }
template <typename T, int D, int NWQ, int NSQ, int NWK, int NSK, bool GRP>
__global__ void __launch_bounds__(NWQ * NSQ * 64, 2)
sdpa_bwd_joint_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                      float *__restrict__ stats, T *__restrict__ dq, T *__restrict__ dk, T *__restrict__ dv, int S, int nRq, int nRk,
                      int Nq, int Nk, float c, float scale, uint32_t rsign, int causal, unsigned stat_bytes, int group,
                      TileOrder order_q, TileOrder order_k)
{
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(NWQ * NSQ == NWK * NSK * (D == 160 ? 2 : 1), "one size of workgroup");
    int id = blockIdx.x;
    bool keys;
    if (Nq == Nk) {
        const int whole = Nq & ~7;
        if (id < 2 * whole) {
            keys = (id & 8) == 0;
            id = (id >> 4 << 3) + (id & 7);
        } else {
            id -= whole;                          // whole ... whole + 2 * rem - 1
            keys = id < Nk;
            if (!keys) id -= Nq - whole;
        }
    } else {
        keys = id < Nk;
        if (!keys) id -= Nk;
    }
    if (!keys)
        bwd_pass<T, D, NWQ, NSQ, bwd_joint_tq<D, NSQ>(), BWD_DQ, GRP, D == 160, true>(q, k, v, dout, nullptr, nullptr, stats, dq, nullptr,
                                                                                     S, nRq, Nq, c, scale, rsign, causal, stat_bytes, group, order_q, id);
    else if constexpr (D == 160)
        bwd_pair_pass<T, D, NWK, NSK, GRP>(q, k, v, dout, stats, dk, dv, S, nRk, Nk, c, scale, rsign, causal, stat_bytes, group, order_k, id);
    else
        bwd_pass<T, D, NWK, NSK, bwd_joint_tk<D, NSK>(), BWD_DKV, GRP, D == 128, true>(q, k, v, dout, nullptr, nullptr, stats, dk, dv,
                                                                                      S, nRk, Nk, c, scale, rsign, causal, stat_bytes, group, order_k, id);
#endif
}

template <int D, int NWQ, int NSQ, int NWK, int NSK> constexpr int bwd_joint_lds()
{
    const int a = bwd_lds_bytes<D, NWQ, NSQ, bwd_joint_tq<D, NSQ>(), BWD_DQ, D == 160>();
    int b = 0;
    if constexpr (D == 160) b = BwdPairGeom<D, NWK, NSK>::LDS_BYTES;
    else b = bwd_lds_bytes<D, NWK, NSK, bwd_joint_tk<D, NSK>(), BWD_DKV, D == 128>();
    return a > b ? a : b;
}

template <typename T, int D, int NWQ, int NSQ, int NWK, int NSK, bool GRP> int launch_bwd_joint_nw(const BwdLaunchArgs &a)
{
    auto kern = sdpa_bwd_joint_kernel<T, D, NWQ, NSQ, NWK, NSK, GRP>;
    constexpr int lds_bytes = bwd_joint_lds<D, NWQ, NSQ, NWK, NSK>();
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    const int kv = a.BH / a.group, nRq = (a.S + NWQ * 32 - 1) / (NWQ * 32), nRk = (a.S + NWK * 32 - 1) / (NWK * 32);
    const int Nq = a.BH * nRq, Nk = kv * nRk;
    const TileOrder oq = tile_order(a.BH, nRq, a.causal != 0, (long long)a.S * D * 2 * (long long)sizeof(T));
    const TileOrder ok = tile_order(kv, nRk, a.causal != 0, (long long)a.group * a.S * D * 2 * (long long)sizeof(T));
    hipLaunchKernelGGL(kern, dim3(Nq + Nk), dim3(NWQ * NSQ * 64), lds_bytes, a.stream, (const T *)a.q, (const T *)a.k,
                       (const T *)a.v, (const T *)a.dout, a.stats, (T *)a.dq, (T *)a.dk, (T *)a.dv, a.S, nRq, nRk, Nq, Nk, a.c, a.scale,
                       a.rsign, a.causal, a.stat_bytes, a.group, oq, ok);
    return (int)hipGetLastError();
}

template <typename T, int D, bool TILED = false> int launch_bwd_stats(const BwdLaunchArgs &a, unsigned *clear = nullptr, int nclear = 0, int pitch = 0)
{
    const int rows = a.BH * a.S;
    const int short_heads = a.causal || a.S <= kBwdShortRow ? a.BH : 0;
    const int rest = a.S <= kBwdShortRow ? 0 : (rows + 63) / 64;
    hipLaunchKernelGGL((sdpa_bwd_stats_kernel<T, D, TILED>), dim3(short_heads + rest), dim3(256), 0, a.stream, (const T *)a.q,
                       (const T *)a.k, (const T *)a.v, (const T *)a.dout, (const T *)a.o, a.lse, a.stats, rows, a.S,
                       divisor((uint32_t)a.S), a.group, a.c, a.rsign, a.causal, a.stat_bytes, short_heads, clear, nclear, pitch);
    return (int)hipGetLastError();
}

}  // namespace tsdpa
