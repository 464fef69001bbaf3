// Instantiates the backward kernels for one (element type, head dim) and provides their launcher.
#pragma once
#include <mutex>

#include "sdpa_bwd_kernel.h"
#include "sdpa_fwd_launch.h"

namespace tsdpa {

// Tile shapes: 32*NW resident rows per workgroup, TS streamed rows per tile for the dQ / dK / dV / fused pass, the
// wavefronts per SIMD its register budget is sized for, and whether its second resident operand stays in the LDS.
// The passes are held by the clock on large problems, so that the choices are within a few per cent of each other
// there: D = 128, dQ on 64-row tiles 1 % ahead of 32-row ones on large problems, 4 % at S = 1024 of nine heads; D = 96,
// dQ on 32-row tiles at three wavefronts per SIMD 1-2 % ahead of 64-row ones at two; D = 64, the fused pass on 32-row
// tiles 1-6 % behind.  D = 160 needs the resident operand in the LDS for two wavefronts per SIMD.
template <int D> struct BwdShape;
template <> struct BwdShape<64>  { static constexpr int NW = 4, WPS[4] = {2, 2, 2, 2}, TS[4] = {64, 64, 64, 64}; static constexpr bool R2[4] = {0, 0, 0, 0}, FUSED_DKV = true; };
template <> struct BwdShape<96>  { static constexpr int NW = 4, WPS[4] = {3, 2, 2, 2}, TS[4] = {32, 32, 64, 32}; static constexpr bool R2[4] = {0, 0, 0, 0}, FUSED_DKV = true; };
template <> struct BwdShape<128> { static constexpr int NW = 4, WPS[4] = {2, 2, 2, 2}, TS[4] = {64, 32, 64, 32}; static constexpr bool R2[4] = {0, 0, 0, 1}, FUSED_DKV = true; };
template <> struct BwdShape<160> { static constexpr int NW = 4, WPS[4] = {2, 2, 2, 1}, TS[4] = {32, 32, 32, 32}; static constexpr bool R2[4] = {1, 1, 0, 0}, FUSED_DKV = false; };

template <typename T, int D, int MODE, bool GRP, int NW>
int launch_bwd_pass_nw(const BwdLaunchArgs &a)
{
    using Sh = BwdShape<D>;
    constexpr int TS = Sh::TS[MODE], WPS = Sh::WPS[MODE];
    constexpr bool R2 = Sh::R2[MODE];
    auto kern = sdpa_bwd_kernel<T, D, NW, TS, WPS, MODE, GRP, R2>;
    constexpr int lds_bytes = bwd_lds_bytes<D, NW, TS, MODE, R2>();
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    const int nR = (a.S + NW * 32 - 1) / (NW * 32);
    // one workgroup per (head of the resident side, tile of its rows): query heads in the dQ pass, key/value heads otherwise
    const int heads = MODE == BWD_DQ ? a.BH : a.BH / a.group;
    const int N = heads * nR;
    const CausalChunks chunks = causal_chunks(heads, nR, (long long)(MODE == BWD_DQ ? 1 : a.group) * a.S * D * 2 * (long long)sizeof(T));
    void *out = MODE == BWD_DQ ? a.dq : (MODE == BWD_DV ? a.dv : a.dk);
    hipLaunchKernelGGL(kern, dim3(N), dim3(NW * 64), lds_bytes, a.stream,
                       (const T *)a.q, (const T *)a.k, (const T *)a.v, (const T *)a.dout, (const T *)a.o, a.lse, a.stats,
                       (T *)out, (T *)(MODE == BWD_DKV ? a.dv : nullptr), a.S, nR, N, a.c, a.scale, a.rsign, a.causal, a.stat_bytes, a.group,
                       chunks.first, chunks.heads);
    return (int)hipGetLastError();
}

// Eight wavefronts per workgroup (256 resident rows, one workgroup per CU) at D = 128 without the causal mask, once
// that gives every CU a workgroup: each streamed tile is then loaded once for twice the rows, half the load
// instructions per wavefront (3-4 % on the whole call from S = 2048 to 16384; with the mask the coarser tiles lose 3-12 %,
// at D = 96 and 64 the gain is 0.5-2 %, and the D = 160 passes have no registers for it).
template <typename T, int D, int MODE, bool GRP>
int launch_bwd_pass(const BwdLaunchArgs &a)
{
    if constexpr (D == 128) {
        const long long heads = MODE == BWD_DQ ? a.BH : a.BH / a.group;
        if (!a.causal && heads * ((a.S + 255) / 256) >= 256) return launch_bwd_pass_nw<T, D, MODE, GRP, 8>(a);
    }
    return launch_bwd_pass_nw<T, D, MODE, GRP, BwdShape<D>::NW>(a);
}

template <typename T, int D, bool GRP>
int launch_bwd_passes(const BwdLaunchArgs &a)
{
    // the dQ pass leaves the statistics of the query rows for the others
    int err = launch_bwd_pass<T, D, BWD_DQ, GRP>(a);
    if (err != 0) return err;
    if constexpr (BwdShape<D>::FUSED_DKV) {
        return launch_bwd_pass<T, D, BWD_DKV, GRP>(a);
    } else {
        err = launch_bwd_pass<T, D, BWD_DV, GRP>(a);
        if (err != 0) return err;
        return launch_bwd_pass<T, D, BWD_DK, GRP>(a);
    }
}

template <typename T, int D>
int launch_bwd(const BwdLaunchArgs &a)
{
    // one query head per key/value head keeps the kernels without the loop over a group
    return a.group == 1 ? launch_bwd_passes<T, D, false>(a) : launch_bwd_passes<T, D, true>(a);
}

}  // namespace tsdpa
