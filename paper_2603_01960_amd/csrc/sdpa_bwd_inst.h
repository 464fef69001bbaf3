// Instantiates the backward kernels for one (element type, head dim) and provides their launcher.
#pragma once
#include <mutex>

#include "sdpa_bwd_kernel.h"
#include "sdpa_bwd_joint_kernel.h"
#include "sdpa_bwd_pick.h"
#include "sdpa_bwd_short_kernel.h"
#include "sdpa_fwd_launch.h"

namespace tsdpa {

// Tile shapes: 32*NW resident rows per workgroup, TS streamed rows per tile for the dQ and the dK + dV pass, the
// wavefronts per SIMD its register budget is sized for, and whether its second resident operand stays in the LDS.
// The passes are held by the clock on large problems, so that the choices are within a few per cent of each other
// there: D = 128, dQ on 64-row tiles 1 % ahead of 32-row ones on large problems, 4 % at S = 1024 of nine heads; D = 96,
// dQ on 32-row tiles at three wavefronts per SIMD 1-2 % ahead of 64-row ones at two; D = 64, dK + dV on 32-row
// tiles 1-6 % behind.  D = 160 needs the resident operand in the LDS for two wavefronts per SIMD.
template <int D> struct BwdShape;
template <> struct BwdShape<64>  { static constexpr int NW = 4, WPS[2] = {2, 2}, TS[2] = {64, 64}; static constexpr bool R2[2] = {0, 0}; };
template <> struct BwdShape<96>  { static constexpr int NW = 4, WPS[2] = {3, 2}, TS[2] = {32, 32}; static constexpr bool R2[2] = {0, 0}; };
template <> struct BwdShape<128> { static constexpr int NW = 4, WPS[2] = {2, 2}, TS[2] = {64, 32}; static constexpr bool R2[2] = {0, 1}; };
template <> struct BwdShape<160> { static constexpr int NW = 4, WPS[2] = {2, 2}, TS[2] = {32, 32}; static constexpr bool R2[2] = {1, 0}; };

template <typename T, int D, int MODE, bool GRP, int NW, int NS, int TS, int WPS>
int launch_bwd_pass_nw(const BwdLaunchArgs &a)
{
    using Sh = BwdShape<D>;
    constexpr bool R2 = Sh::R2[MODE];
    auto kern = sdpa_bwd_kernel<T, D, NW, NS, TS, WPS, MODE, GRP, R2>;
    constexpr int lds_bytes = bwd_lds_bytes<D, NW, NS, TS, MODE, R2>();
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
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
    const TileOrder order = tile_order(heads, nR, a.causal != 0, (long long)(MODE == BWD_DQ ? 1 : a.group) * a.S * D * 2 * (long long)sizeof(T));
    void *out = MODE == BWD_DQ ? a.dq : a.dk;
    hipLaunchKernelGGL(kern, dim3(N), dim3(NW * NS * 64), lds_bytes, a.stream,
                       (const T *)a.q, (const T *)a.k, (const T *)a.v, (const T *)a.dout, (const T *)a.o, a.lse, a.stats,
                       (T *)out, (T *)(MODE == BWD_DKV ? a.dv : nullptr), a.S, nR, N, a.c, a.scale, a.rsign, a.causal, a.stat_bytes, a.group,
                       order);
    return (int)hipGetLastError();
}

template <typename T, int D, int MODE, bool GRP>
int launch_bwd_pass(const BwdLaunchArgs &a)
{
    using Sh = BwdShape<D>;
    const long long heads = MODE == BWD_DQ ? a.BH : a.BH / a.group;
    if constexpr (D == 96 || D == 128) {
        const BwdForm f = pick_bwd_form(D, a.causal != 0, MODE != BWD_DQ, heads * ((a.S + 127) / 128),
                                        (long long)(MODE == BWD_DQ ? 1 : a.group) * ((a.S + 31) / 32));
        // (the forms with streams have the loop over a group compiled in: one instantiation for both)
        if (f.ns > 1) {
            if (f.nw == 4) return launch_bwd_pass_nw<T, D, MODE, true, 4, 2, 32, 2>(a);
            if (f.nw == 1) return launch_bwd_pass_nw<T, D, MODE, true, 1, 4, 32, 2>(a);
            return f.ns == 2 ? launch_bwd_pass_nw<T, D, MODE, true, 2, 2, 32, 2>(a) : launch_bwd_pass_nw<T, D, MODE, true, 2, 4, 32, 2>(a);
        }
    }
    if constexpr (D == 128) {
        if (!a.causal && bwd_wide_rows(heads, a.S)) return launch_bwd_pass_nw<T, D, MODE, GRP, 8, 1, Sh::TS[MODE], Sh::WPS[MODE]>(a);
    }
    return launch_bwd_pass_nw<T, D, MODE, GRP, Sh::NW, 1, Sh::TS[MODE], Sh::WPS[MODE]>(a);
}

template <typename T, int D, bool GRP>
int launch_bwd_pairs(const BwdLaunchArgs &a)
{
    switch (pick_bwd_pairs(a.causal != 0, a.BH, a.group, a.S)) {
        case 22: return launch_bwd_pair<T, D, 2, 2, true>(a);
        case 41: return launch_bwd_pair<T, D, 4, 1, GRP>(a);
        default: return launch_bwd_pair<T, D, 2, 1, GRP>(a);
    }
}

template <typename T, int D, bool GRP>
int launch_bwd_passes(const BwdLaunchArgs &a)
{
    // the dQ pass leaves the statistics of the query rows for the other
    const int err = launch_bwd_pass<T, D, BWD_DQ, GRP>(a);
    if (err != 0) return err;
    if constexpr (D == 160) return launch_bwd_pairs<T, D, GRP>(a);
    else return launch_bwd_pass<T, D, BWD_DKV, GRP>(a);
}

template <typename T, int D, int NWQ, int NSQ, int NWK, int NSK>
int launch_bwd_joint_form(const BwdLaunchArgs &a)
{
    // (forms with streams of keys have the loop over a group compiled in)
    if constexpr (NSK == 1)
        if (a.group == 1) return launch_bwd_joint_nw<T, D, NWQ, NSQ, NWK, NSK, false>(a);
    return launch_bwd_joint_nw<T, D, NWQ, NSQ, NWK, NSK, true>(a);
}

template <typename T, int D>
int launch_bwd_joint(const BwdLaunchArgs &a, int form)
{
    const int err = launch_bwd_stats<T, D>(a);
    if (err != 0) return err;
    if constexpr (D == 160) {
        if (form == 4121) return launch_bwd_joint_form<T, D, 4, 1, 2, 1>(a);
        return form == 4222 ? launch_bwd_joint_form<T, D, 4, 2, 2, 2>(a) : launch_bwd_joint_form<T, D, 2, 2, 1, 2>(a);
    } else {
        if constexpr (D == 64) {
            if (form == 2241) return launch_bwd_joint_form<T, D, 2, 2, 4, 1>(a);
        } else {                                  // (never picked for grouped heads there)
            if (form == 2241 && a.group == 1) return launch_bwd_joint_nw<T, D, 2, 2, 4, 1, false>(a);
        }
        if (form == 4122) return launch_bwd_joint_form<T, D, 4, 1, 2, 2>(a);
        if constexpr (D <= 96)
            if (form == 2222) return launch_bwd_joint_form<T, D, 2, 2, 2, 2>(a);
        if constexpr (D >= 96)
            if (form == 4224) return launch_bwd_joint_form<T, D, 4, 2, 2, 4>(a);
        if constexpr (D == 64) {
            if (form == 2418) return launch_bwd_joint_form<T, D, 2, 4, 1, 8>(a);
            if (form == 4114) return launch_bwd_joint_form<T, D, 4, 1, 1, 4>(a);
            if (form == 1414) return launch_bwd_joint_form<T, D, 1, 4, 1, 4>(a);
        } else if constexpr (D == 96) {
            if (form == 2424) return launch_bwd_joint_form<T, D, 2, 4, 2, 4>(a);
        } else {
            if (form == 4141) return launch_bwd_joint_form<T, D, 4, 1, 4, 1>(a);
        }
        return launch_bwd_joint_form<T, D, 2, 2, 1, 4>(a);
    }
}

template <typename T, int D>
int launch_bwd(const BwdLaunchArgs &a)
{
    if constexpr (D <= 96) {
        if (a.group == 1 && a.S <= 256 && bwd_in_one_launch(D, a.BH, a.S)) {
            // A workgroup that takes several heads hides one's loads behind another's work.  Up to 256 heads there is nothing to hide and its
            // prologue costs more (us, a workgroup per head -> that: 256 heads of 197 rows 17.6 -> 18.3, 200 of 256 20.1 -> 20.2), from 257 on
            // it gains (257 of 256 34.8 -> 34.7, 300 of 129 23.5 -> 23.2, more above 512: see there).  At up to 128 rows several workgroups
            // share a CU and do the same for each other.
            if constexpr (D == 64)
                if (a.S > 128 && a.BH > 256) return launch_bwd_heads<T>(a);
            return a.S <= 64 ? launch_bwd_short_nw<T, D, 2>(a) : a.S <= 128 ? launch_bwd_short_nw<T, D, 4>(a) : launch_bwd_short_nw<T, D, 8>(a);
        }
    }
    if (const int form = pick_bwd_joint(D, a.causal != 0, a.BH, a.group, a.S)) return launch_bwd_joint<T, D>(a, form);
    // one query head per key/value head keeps the kernels without the loop over a group
    return a.group == 1 ? launch_bwd_passes<T, D, false>(a) : launch_bwd_passes<T, D, true>(a);
}

}  // namespace tsdpa
