// Instantiates the forward kernel for one (element type, head dim) over the tile grid
// T_M in {64,128} x T_N in {32,64,128} (the paper's Table 1 knobs) and the 256 x 64 tile of this library's own,
// plus the general Sq x Skv / split-KV variant over T_M in {64,128} x T_N in {32,64} (and 256 x 64 on a dense cache),
// and provides its launcher.
// The kernel table is fixed at build time: there is no JIT step to cache (Section 4.2.2).
#pragma once
#include <mutex>

#include "sdpa_fwd_kernel.h"
#include "sdpa_fwd_launch.h"

namespace tsdpa {

constexpr int kLdsPerCU = 160 * 1024;

// Register budget of an instantiation, in wavefronts per SIMD (512 registers per lane divided among
// them).  Three for 32-row K/V tiles up to D = 128: the main loop then fits 168 registers without
// spilling and the third wavefront fills more of the phases in which the other two leave the matrix
// pipe idle (+4-6 % on the long workloads).  Two otherwise, also where the LDS admits only one: a
// budget of one wavefront per SIMD makes the compiler split accumulators between the VGPR and AGPR
// halves and move them back and forth (or to scratch) inside the loop.
template <int D, int NW, int TN> constexpr int waves_per_simd() { return (TN == 32 && D <= 128) ? 3 : 2; }

template <typename T, int D, int NW, int TN, int KV = 0, int NS = 1>     // KV: 0 square, 1 dense cache, 2 paged cache, 3 and 4 these with halved weights; NS streams
int launch_one(const LaunchArgs &a)
{
    constexpr int WPS = NS > 1 ? 2 : waves_per_simd<D, NW, TN>();
    auto kern = sdpa_fwd_kernel<T, D, NW, stream_tile(TN, NS), WPS, KV>;
    // K/V tile slots during the loop; then the states of all streams but the first, and one 32 x D block per wavefront for the
    // output transpose
    constexpr int stage_bytes = NW * 32 * TileGeom<D, TN>::OROW, state_bytes = (NS - 1) * NW * (32 * D * 4 + 512);
    constexpr int after_bytes = stage_bytes > state_bytes ? stage_bytes : state_bytes;
    constexpr int lds_bytes = NS * TileGeom<D, TN>::LDS_BYTES > after_bytes ? NS * TileGeom<D, TN>::LDS_BYTES : after_bytes;
    static_assert(lds_bytes <= kLdsPerCU, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    constexpr int TM = NW * 32;
    const int nQ = (a.S + TM - 1) / TM;
    const int heads = a.BH * (KV ? a.splits : 1);
    const int N = heads * nQ;
    // (entries of different lengths: eight heads per XCD and chunk whatever they stream, for the balance between them)
    // Square problem, plain form, up to three workgroups per CU (768), up to three tiles per head or D = 64: sixteen heads per XCD
    // and chunk instead of eight (us, plain order / eight / sixteen: 231 heads of S = 384 D = 64 14.7 / 15.4 / 13.6, D = 96 18.6 /
    // 19.1 / 17.7; 224 of S = 364 D = 160 29.5 / 28.7 / 26.2; with more tiles eight are ahead: 130 of S = 640 D = 128 29.2 / 25.9 /
    // 27.4; so they are with up to four tiles and little over two workgroups per CU: 190 of S = 384 D = 64 13.7 / 12.0 / 12.9).
    // (against a cache the tiles of a head are uneven by the queries' share of the keys only; below a twelfth of the capacity
    // the plain order: 32 entries of 286 queries, 8192 ... 16384 keys, D = 64 587 -> 550 us, 300 queries of 16384 keys D = 96 575 ->
    // 562, where 1024 queries of 2048 keys go 47.6 -> 44.2 with the causal order, 2048 of 8192 222.6 -> 215.6)
    const bool uneven = a.causal != 0 && (!KV || (long long)a.rows_per_head * 12 >= a.Skv);
    TileOrder order = tile_order(heads, nQ, uneven, a.kv_lens ? 0 : (long long)(KV ? a.Skv : a.S) * D * 2 * (long long)sizeof(T),
                                 !KV && NS == 1 && (nQ <= 4 ? N > (D <= 96 ? 576 : 520) && (nQ <= 3 || D == 64) : D == 64));
    // Two tiles of about the same work (33 ... 64 rows in the second: two wavefronts of six steps against four of four) in up to
    // two rounds: there is no long one to start first, and the plain order keeps a head's tiles together (576 heads of S = 171,
    // D = 64 14.7 -> 14.4, D = 96 19.0 -> 17.6, D = 160 30.9 -> 30.5; 700 of S = 185 2 % at D = 96; beyond two rounds 1-8 % behind)
    if (!KV && NS == 1 && NW == 4 && N <= 1536 && a.S > 160 && a.S <= 192) order.heads = 0;
    hipLaunchKernelGGL(kern, dim3(N), dim3(NW * NS * 64), lds_bytes, a.stream,
                       (const T *)a.q, (const T *)a.k, (const T *)a.v, (T *)a.o, a.lse,
                       a.S, nQ, N, a.c, a.tau, a.qsign, a.linear_grid, a.causal, order,
                       a.Skv, a.splits, a.ws, a.rows_per_head, a.kv_lens, a.heads_per_batch,
                       a.block_table, a.max_blocks, a.block_shift, a.tile_rot, a.batches, divisor((uint32_t)(KV ? a.batches : 1)));
    return (int)hipGetLastError();
}

// The 64-row K/V tile instantiations live in translation units of their own (sdpa_fwd_*_tn64.hip): the
// build compiles those with another machine scheduler, which gains 3-5 % there and loses badly on the
// 32-row tile kernels, and a scheduler is chosen per compiler invocation.
template <typename T, int D>
int launch_dispatch_tn64(int tile_m, const LaunchArgs &a)
{
    if (tile_m != 64 && tile_m != 128 && tile_m != 256) return (int)hipErrorInvalidValue;
    // 256 query rows per workgroup (eight wavefronts, one workgroup per CU): the square problem and the dense cache
    if (tile_m == 256) {
        if (a.kv && a.block_table != nullptr) return (int)hipErrorInvalidValue;
        return a.kv ? launch_one<T, D, 8, 64, 1>(a) : launch_one<T, D, 8, 64>(a);
    }
    if (a.kv && a.block_table != nullptr)
        return tile_m == 64 ? launch_one<T, D, 2, 64, 2>(a) : launch_one<T, D, 4, 64, 2>(a);
    if (a.kv)
        return tile_m == 64 ? launch_one<T, D, 2, 64, 1>(a) : launch_one<T, D, 4, 64, 1>(a);
    return tile_m == 64 ? launch_one<T, D, 2, 64>(a) : launch_one<T, D, 4, 64>(a);
}

// Streams (a.streams > 1): tile_m / 32 wavefronts each, 32-row K/V tiles; the forms that pick_streams and
// pick_streams_kv (tiled_sdpa.hip) choose from.
template <typename T, int D, int KV>
int launch_streams(int tile_m, const LaunchArgs &a)
{
    switch (tile_m * 10 + a.streams) {
        case 324:
            if constexpr (KV != 0 && D < 160)
                if (a.halves) return launch_one<T, D, 1, 32, KV + 2, 4>(a);
            return launch_one<T, D, 1, 32, KV, 4>(a);
        case 642: return launch_one<T, D, 2, 32, KV, 2>(a);
        case 1282:
            if constexpr (KV == 0) return launch_one<T, D, 4, 32, KV, 2>(a);
            break;
        case 643:
            if constexpr (D == 160) return launch_one<T, D, 2, 32, KV, 3>(a);
            break;
        case 644:
            if constexpr (D < 160) return launch_one<T, D, 2, 32, KV, 4>(a);
            break;
        case 328:
            if constexpr (D == 64 && KV == 0) return launch_one<T, D, 1, 32, KV, 8>(a);
            break;
    }
    return (int)hipErrorInvalidValue;
}

using LaunchTn64 = int (*)(int tile_m, const LaunchArgs &a);

template <typename T, int D>
int launch_dispatch(int tile_m, int tile_n, const LaunchArgs &a, LaunchTn64 tn64)
{
    if (tile_n == 64) return tn64(tile_m, a);
    const int key = tile_m * 1000 + tile_n;
    if (a.streams > 1) {
        if (!a.kv) return launch_streams<T, D, 0>(tile_m, a);
        return a.block_table ? launch_streams<T, D, 2>(tile_m, a) : launch_streams<T, D, 1>(tile_m, a);
    }
    if (a.kv && a.block_table != nullptr) {
        switch (key) {
            case 64032: return launch_one<T, D, 2, 32, 2>(a);
            case 128032: return launch_one<T, D, 4, 32, 2>(a);
            default: return (int)hipErrorInvalidValue;
        }
    }
    if (a.kv) {
        switch (key) {
            case 64032: return launch_one<T, D, 2, 32, 1>(a);
            case 128032: return launch_one<T, D, 4, 32, 1>(a);
            default: return (int)hipErrorInvalidValue;
        }
    }
    switch (key) {
        case 64032: return launch_one<T, D, 2, 32>(a);
        case 64128:
            if constexpr (D <= 128) return launch_one<T, D, 2, 128>(a);
            else return (int)hipErrorInvalidValue;   // four 128-row slots of 320-byte rows are all of a CU's LDS
        case 128032: return launch_one<T, D, 4, 32>(a);
        case 128128:
            if constexpr (D <= 128) return launch_one<T, D, 4, 128>(a);
            else return (int)hipErrorInvalidValue;
        default: return (int)hipErrorInvalidValue;
    }
}

}  // namespace tsdpa
