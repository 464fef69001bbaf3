// Instantiates the backward kernels for one (element type, head dim) and provides their launcher.
#pragma once
#include <mutex>

#include "sdpa_bwd_kernel.h"
#include "sdpa_bwd_pair_kernel.h"
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

// Wavefronts along the resident rows and streams of a pass whose plain form (128 resident rows, one stream) has `n`
// workgroups, each with a chain of `chain` 32-row steps (over all query heads of its group).  Up to one such workgroup per CU
// a SIMD has one wavefront or none and waits through every chain alone; streams shorten the chain, fewer resident rows make
// more workgroups of it.  The lines between the cases are those of timings of every form on 560 shapes (16 ... 400 workgroups,
// chains of 4 ... 256), where this choice is within 0.7 % of the best one on average:
//   * up to 64 workgroups: one wavefront of 32 rows and its private tiles per stream, as many streams as the LDS holds
//     (BF16, us per call with the one pass changed: 8 query heads per key/value head, S = 512, D = 64 104 -> 33, D = 128
//     150 -> 66; S = 2048 of one head 75.9 -> 45.0);
//   * up to 128: 64 rows, four streams on long chains (D = 128, S = 2048: 121 -> 97 us in the dQ pass), two on short ones;
//     under the causal mask the 32-row form, whose uneven workgroups pack better, where its LDS lets two share a CU (D = 64)
//     or the chain is long;
//   * up to 256: under the mask 64 rows and two ... four streams (D = 160, four query heads per key/value head, S = 2048:
//     540 -> 379 us), without it, where nothing is uneven, 128 rows and two streams on long chains (3-12 %);
//   * up to 400, under the mask, long chains: 5-15 %.  Beyond, and on short chains, the plain form.
struct BwdForm { int nw, ns; };
inline BwdForm pick_bwd_form(int D, bool causal, bool keys_resident, long long n, long long chain)
{
    const BwdForm plain{4, 1};
    if (chain <= 2) return plain;
    if (n <= 64) {
        if (D == 160) return BwdForm{1, 3};
        if (!keys_resident && chain <= 8) return BwdForm{2, 2};
        return BwdForm{1, D == 64 && chain >= 64 ? 8 : 4};
    }
    if (n <= 128) {
        if (causal && chain >= (D == 64 ? 16 : D == 160 ? 64 : 128)) return BwdForm{1, D == 160 ? 3 : 4};
        if (D == 160) return BwdForm{2, chain >= 64 ? 3 : 2};
        return BwdForm{2, chain >= 32 ? 4 : 2};
    }
    if (n <= 256) {
        if (!causal) return chain >= (keys_resident ? 16 : 32) ? BwdForm{4, 2} : plain;
        if (chain >= 64) return D == 64 ? BwdForm{1, 4} : BwdForm{2, D == 160 ? 3 : 4};
        return chain >= (D == 160 ? 32 : 16) ? BwdForm{2, 2} : plain;
    }
    if (n <= 400 && causal && chain >= 64) return D == 160 || (D == 128 && keys_resident) ? BwdForm{4, 2} : BwdForm{2, 2};
    return plain;
}

// Eight wavefronts per workgroup (256 resident rows, one workgroup per CU) at D = 128 without the causal mask: each
// streamed tile is then loaded once for twice the rows, half the load instructions per wavefront, 2.5 % per full round of
// 256 such workgroups against 512 of 128 rows (us per call, 256 rows / 128: 32 heads S = 2048 212 / 218, 64 of 4096 1596 /
// 1616, 16 of 8192 1551 / 1585, 50 of 2048 379 / 395).  A last round that leaves the CUs one workgroup of 128 rows or
// none takes 0.6 of a full one, which 256 rows cannot use (100 heads S = 2048 786 / 716, 20 of 4096 688 / 607, 64 of 1536
// 295 / 265), and below S = 1024 the rows missing in a tile and the prologue cost more than the loads (512 of 300 202 /
// 158, 768 of 128 88 / 68).  With the mask the coarser tiles lose 3-12 %, at D = 96 and 64 the gain is 0.5-2 %, and the
// D = 160 passes have no registers for it.
inline bool bwd_wide_rows(long long heads, int S)
{
    const long long narrow = heads * ((S + 127) / 128), wide = heads * ((S + 255) / 256);
    const long long rest = narrow % 512;
    const long long t_narrow = 200 * (narrow / 512) + (rest == 0 ? 0 : rest <= 256 ? 120 : 200);
    return S >= 1024 && wide >= 256 && 195 * ((wide + 255) / 256) <= t_narrow;
}

template <typename T, int D, int MODE, bool GRP>
int launch_bwd_pass(const BwdLaunchArgs &a)
{
    using Sh = BwdShape<D>;
    const long long heads = MODE == BWD_DQ ? a.BH : a.BH / a.group;
    const BwdForm f = pick_bwd_form(D, a.causal != 0, MODE != BWD_DQ, heads * ((a.S + 127) / 128),
                                    (long long)(MODE == BWD_DQ ? 1 : a.group) * ((a.S + 31) / 32));
    // (the forms with streams have the loop over a group compiled in: one instantiation for both)
    if (f.ns > 1) {
        if (f.nw == 4) return launch_bwd_pass_nw<T, D, MODE, true, 4, 2, 32, 2>(a);
        if (f.nw == 2 && f.ns == 2) return launch_bwd_pass_nw<T, D, MODE, true, 2, 2, 32, 2>(a);
        if constexpr (D == 160) {
            if (f.nw == 2) return launch_bwd_pass_nw<T, D, MODE, true, 2, 3, 32, 2>(a);
            return launch_bwd_pass_nw<T, D, MODE, true, 1, 3, 32, 2>(a);
        } else {
            if (f.nw == 2) return launch_bwd_pass_nw<T, D, MODE, true, 2, 4, 32, 2>(a);
            if constexpr (D == 64)
                if (f.ns == 8) return launch_bwd_pass_nw<T, D, MODE, true, 1, 8, 32, 2>(a);
            return launch_bwd_pass_nw<T, D, MODE, true, 1, 4, 32, 2>(a);
        }
    }
    if constexpr (D == 128) {
        if (!a.causal && bwd_wide_rows(heads, a.S)) return launch_bwd_pass_nw<T, D, MODE, GRP, 8, 1, Sh::TS[MODE], Sh::WPS[MODE]>(a);
    }
    return launch_bwd_pass_nw<T, D, MODE, GRP, Sh::NW, 1, Sh::TS[MODE], Sh::WPS[MODE]>(a);
}

// Short sequences of one query head per key/value head in one launch (sdpa_bwd_short_kernel.h), D = 64 and 96 (two accumulators
// beside both resident operands do not fit above).  us per call, passes -> one launch: D = 64, S = 32 10.7 -> 6.5 (60 heads),
// 19.4 -> 9.5 (768); S = 64 21.2 -> 14.9 (768); S = 128 11.3 -> 9.5 (60), 32.3 -> 25.2 (768); S = 197 25.5 -> 18.7 (200),
// 67.6 -> 56.6 (768) but 14.8 -> 16.7 (60), where the passes spread a head over more CUs; D = 96, S = 64 12.3 -> 10.1 (60), 27.1 ->
// 19.6 (768); S = 128 43.8 -> 34.9 (768); S = 256 31.4 -> 28.2 (200), 115 -> 101 (768) but 46.7 -> 52.1 (300): a second
// round of one workgroup per CU that is mostly empty.
inline bool bwd_in_one_launch(int D, int heads, int S)
{
    if (S <= (D == 64 ? 128 : 64)) return true;
    if (heads < 110) return false;
    if (D == 64 || S <= 128) return true;
    return heads * 10 >= (heads + 255) / 256 * 256 * 7;
}

// Pairs and streams of the dK + dV pass at D = 160, by the workgroups of 128 keys and the 32-row steps of their chains; from
// timings of four forms on 200 shapes (BF16, us).  Few workgroups: one pair and two streams (S = 2187 of one head 99.5 with
// four pairs, 62.2), as many as fit; up to 150, and to 400 whose chains run over a group's heads: two of both (two
// entries of 16 heads over 4, S = 4096: 10-15 %).  Else two pairs, two workgroups per CU, 2-10 % ahead of four on causal
// and short problems; four pairs, which read a tile once for 128 keys, 3-4 % ahead on long ones without the mask (32 heads,
// S = 8192: 2084 / 2002).
template <typename T, int D, bool GRP>
int launch_bwd_pairs(const BwdLaunchArgs &a)
{
    const long long nk = (long long)(a.BH / a.group) * ((a.S + 127) / 128), chain = (long long)a.group * ((a.S + 31) / 32);
    if (chain > 3 && nk <= 75) return launch_bwd_pair<T, D, 1, 2, true>(a);
    if (chain > 3 && (nk <= 153 || (nk <= 400 && chain > 140))) return launch_bwd_pair<T, D, 2, 2, true>(a);
    if (!a.causal && a.S >= 600 && nk >= 430) return launch_bwd_pair<T, D, 4, 1, GRP>(a);
    return launch_bwd_pair<T, D, 2, 1, GRP>(a);
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

template <typename T, int D>
int launch_bwd(const BwdLaunchArgs &a)
{
    if constexpr (D <= 96) {
        if (a.group == 1 && a.S <= 256 && bwd_in_one_launch(D, a.BH, a.S))
            return a.S <= 64 ? launch_bwd_short_nw<T, D, 2>(a) : a.S <= 128 ? launch_bwd_short_nw<T, D, 4>(a) : launch_bwd_short_nw<T, D, 8>(a);
    }
    // one query head per key/value head keeps the kernels without the loop over a group
    return a.group == 1 ? launch_bwd_passes<T, D, false>(a) : launch_bwd_passes<T, D, true>(a);
}

}  // namespace tsdpa
