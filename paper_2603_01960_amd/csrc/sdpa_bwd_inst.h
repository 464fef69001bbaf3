// Instantiates the backward kernels for one (element type, head dim) and provides their launcher.
#pragma once
#include <mutex>

#include "sdpa_bwd_kernel.h"
#include "sdpa_bwd_joint_kernel.h"
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

// Wavefronts along the resident rows and streams of a pass launched by itself at D = 96 and 128 whose plain form (128 resident
// rows, one stream) has `n` workgroups, each with a chain of `chain` 32-row steps (over all query heads of its group).  (At D = 64 and
// 160 only large problems launch the passes by themselves: pick_bwd_joint.)  Up to one such workgroup per CU
// a SIMD has one wavefront or none and waits through every chain alone; streams shorten the chain, fewer resident rows make
// more workgroups of it.  The lines between the cases are those of timings of every form on 560 shapes (16 ... 400 workgroups,
// chains of 4 ... 256), where this choice is within 0.7 % of the best one on average:
//   * up to 64 workgroups: one wavefront of 32 rows and its private tiles per stream, as many streams as the LDS holds
//     (BF16, us per call with the one pass changed, D = 128: 8 query heads per key/value head, S = 512, 150 -> 66);
//   * up to 128: 64 rows, four streams on long chains (D = 128, S = 2048: 121 -> 97 us in the dQ pass), two on short ones;
//     under the causal mask the 32-row form, whose uneven workgroups pack better, where the chain is long;
//   * up to 256: under the mask 64 rows and two ... four streams, without it, where nothing is uneven, 128 rows and two streams on
//     long chains (3-12 %);
//   * up to 400, under the mask, long chains: 5-15 %.  Beyond, and on short chains, the plain form.
struct BwdForm { int nw, ns; };
inline BwdForm pick_bwd_form(int D, bool causal, bool keys_resident, long long n, long long chain)
{
    const BwdForm plain{4, 1};
    if (chain <= 2) return plain;
    if (n <= 64) return !keys_resident && chain <= 8 ? BwdForm{2, 2} : BwdForm{1, 4};
    if (n <= 128) return causal && chain >= 128 ? BwdForm{1, 4} : BwdForm{2, chain >= 32 ? 4 : 2};
    if (n <= 256) {
        if (!causal) return chain >= (keys_resident ? 16 : 32) ? BwdForm{4, 2} : plain;
        return chain >= 64 ? BwdForm{2, 4} : chain >= 16 ? BwdForm{2, 2} : plain;
    }
    if (n <= 400 && causal && chain >= 64) return D == 128 && keys_resident ? BwdForm{4, 2} : BwdForm{2, 2};
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

// The dK + dV pass at D = 160 as a launch of its own (large problems: pick_bwd_joint).  Two pairs, two workgroups per CU, 2-10 %
// ahead of four on causal and short problems; four pairs, which read a tile once for 128 keys, 3-4 % ahead on long ones without the
// mask (32 heads of S = 8192, us: 2084 / 2002); two pairs and two streams where up to 400 tiles of 128 keys have chains that run
// over a group's heads (four entries of 16 heads over 4, S = 2048, causal: 374 / 305).
template <typename T, int D, bool GRP>
int launch_bwd_pairs(const BwdLaunchArgs &a)
{
    const long long nk = (long long)(a.BH / a.group) * ((a.S + 127) / 128), chain = (long long)a.group * ((a.S + 31) / 32);
    if (nk <= 400 && chain > 140) return launch_bwd_pair<T, D, 2, 2, true>(a);
    if (!a.causal && a.S >= 600) return launch_bwd_pair<T, D, 4, 1, GRP>(a);
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

// The form of the joint grid: wavefronts along the rows and streams of the dQ pass, then of the dK + dV pass (D = 160: pairs and
// streams), as four digits; 0: the passes as launches of their own.  `nk`: workgroups of 128 keys; n: those and the ones of 128
// queries; `chain`: the 32-row steps of a workgroup of keys, over the query heads of its group; work: their product.  The lines are
// those of timings of a dozen forms on 1100 shapes (BF16; drawn over the whole range, and the neighbourhood of the lines), where
// this choice is 1.9, 1.7, 2.8 and 1.8 % from the best of all forms on average at D = 64, 96, 128 and 160, and 1.12, 1.11,
// 1.12 and 1.15 (there against pairs in a launch of their own) times as fast as the passes apart.  What decides:
//   * few workgroups: a wavefront per 32 keys with tiles of its own (..14; D = 160 ..12), whose chains are the shortest; where a group's heads
//     make them long, eight streams at D = 64 (2418);
//   * more of them: workgroups that share tiles, 64 keys in two or four streams (4122, 2222, 2424, 4224) or 128 (2241, 4141, 4120);
//   * many workgroups of ungrouped heads: the passes apart, which are level there and save reading O and dO once more.  Grouped
//     heads keep the joint grid longer: their few long chains of keys drain beside the many short ones of the queries.
// Us, passes apart / here: D = 64, 260 tiles of 128 (S = 1236, causal) 50.6 / 34.3; D = 96, one head S = 1159 25.9 / 17.2; D = 128, six
// heads over 2 of S = 1024, causal 66.9 / 50.6; D = 160, 8 heads over 2 of S = 1346 139 / 86.
inline int pick_bwd_joint(int D, bool causal, int heads, int group, int S)
{
    const long long tiles = (S + 127) / 128, nk = heads / group * tiles, n = nk + heads * tiles;
    const long long chain = (long long)group * ((S + 31) / 32), work = nk * chain;
    if (D == 64 && group == 1) {
        if (S <= 256) return n <= 330 || (n <= 440 && S <= 190) ? 4122 : causal ? 2241 : 0;
        if (causal) {
            if (n <= 220 && chain >= 30) return 1414;
            return n <= 150 ? 2214 : n <= 514 ? 2222 : n <= 1850 ? 2241 : 0;
        }
        if (n <= 240) return n <= 170 ? 2214 : 4122;
        if (n <= 950) return S <= 600 ? 4122 : 2241;
        return S >= 1600 && n <= 1850 ? 2241 : 0;
    }
    if (D == 64) {
        if (!causal) return nk > 100 ? 4122 : nk <= 32 && chain > 80 ? 2418 : 2214;
        if (nk <= 48) return chain <= 36 || S <= 256 ? 2214 : 2418;
        if (S <= 850) return nk <= 170 && n <= 1540 ? 4114 : 4122;
        return nk <= 68 && n <= 1540 ? 2418 : n <= 1540 && chain <= 290 ? 2214 : nk <= 180 ? 4114 : 4122;
    }
    if (D == 96 && group == 1) {
        if (n <= (causal ? 70 : 90)) return 2214;
        if (causal) {
            if (n <= 216 && chain >= 30) return 2424;
            return n <= 514 || (n <= 960 && chain > 64) ? 2222 : n <= 960 ? 2241 : 0;
        }
        if (work <= 2800) return 4122;
        if (n <= 120) return 2424;
        if (n <= 300) return n <= 170 && chain >= 100 ? 4224 : 0;
        if (n <= 340) return 4122;
        return n <= 860 || (S >= 3000 && n <= 2700) ? 2241 : 0;
    }
    if (D == 96) {
        if (nk > 740) return 0;
        if (!causal) return nk <= 48 ? 2214 : nk <= 86 ? 4224 : 4122;
        if (n <= 365) return 2214;
        if (nk <= 200) return S <= 550 ? 0 : 4224;
        return chain <= 440 ? 4122 : 4224;
    }
    if (D == 128 && group == 1) {
        if (causal) {
            if (work <= 240) return 4141;
            if (n <= 200) return n <= 80 ? 2214 : 4224;
            return n > 514 && n <= 994 ? 2241 : 0;
        }
        if (n <= 168) return S <= 90 ? 4141 : S <= 160 ? 4122 : S <= 480 || n <= 92 ? 2214 : 4224;
        if (work <= 3000) return 4141;
        return work > 6150 && (n <= 900 || (n <= 2000 && S >= 1500)) ? 2241 : 0;
    }
    if (D == 128) {
        if (nk <= (causal ? 54 : 42)) return 2214;
        if (!causal) return work <= 2290 ? 4122 : nk <= 73 ? 4224 : nk <= 230 ? 0 : 4141;
        return chain <= 175 || (nk <= 384 && n > 1300) ? 0 : nk <= 384 ? 4224 : 4141;
    }
    if (group == 1) return n <= 90 ? (S <= 64 ? 4120 : 2212) : n <= (causal ? 800 : 2000) ? 4120 : 0;
    if (nk <= (S <= 64 ? 60 : 51)) return 2212;
    if (nk <= 75 && S > 64) return 4223;
    if (causal && nk >= 240) return 0;
    if (chain > 80 && nk < (causal ? 240 : chain > 400 ? 130 : 100)) return 4223;
    return nk <= 500 ? 4120 : 0;
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
        if (form == 4120) return launch_bwd_joint_form<T, D, 4, 1, 2, 1>(a);
        return form == 4223 ? launch_bwd_joint_form<T, D, 4, 2, 2, 2>(a) : launch_bwd_joint_form<T, D, 2, 2, 1, 2>(a);
    } else {
        if (form == 2241) return launch_bwd_joint_form<T, D, 2, 2, 4, 1>(a);
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
        if (a.group == 1 && a.S <= 256 && bwd_in_one_launch(D, a.BH, a.S))
            return a.S <= 64 ? launch_bwd_short_nw<T, D, 2>(a) : a.S <= 128 ? launch_bwd_short_nw<T, D, 4>(a) : launch_bwd_short_nw<T, D, 8>(a);
    }
    if (const int form = pick_bwd_joint(D, a.causal != 0, a.BH, a.group, a.S)) return launch_bwd_joint<T, D>(a, form);
    // one query head per key/value head keeps the kernels without the loop over a group
    return a.group == 1 ? launch_bwd_passes<T, D, false>(a) : launch_bwd_passes<T, D, true>(a);
}

}  // namespace tsdpa
