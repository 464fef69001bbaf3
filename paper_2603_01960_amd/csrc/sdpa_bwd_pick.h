// Which kernels a backward call takes, by its sizes: host rules without device code, so that a host program can evaluate them too.
#pragma once
#include <stddef.h>

namespace tsdpa {

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
    if (n <= 64) return BwdForm{1, 4};
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

// The dK + dV pass at D = 160 as a launch of its own (large problems: pick_bwd_joint), pairs and streams as two digits.  Two pairs,
// two workgroups per CU, 2-10 % ahead of four on causal and short problems; four pairs, which read a tile once for 128 keys, 3-4 %
// ahead on long ones without the mask (32 heads of S = 8192, us: 2084 / 2002); two pairs and two streams where up to 400 tiles
// of 128 keys have chains that run over a group's heads (four entries of 16 heads over 4, S = 2048, causal: 374 / 305).
inline int pick_bwd_pairs(bool causal, int heads, int group, int S)
{
    const long long nk = (long long)(heads / group) * ((S + 127) / 128), chain = (long long)group * ((S + 31) / 32);
    if (nk <= 400 && chain > 140) return 22;
    return !causal && S >= 600 ? 41 : 21;
}

// The form of the joint grid: wavefronts along the rows and streams of the dQ pass, then of the dK + dV pass (D = 160: pairs and
// streams), as four digits; 0: the passes as launches of their own.  `nk`: workgroups of 128 keys; n: those and the ones of 128
// queries; `chain`: the 32-row steps of a workgroup of keys, over the query heads of its group; work: their product.  The lines are
// those of timings of every form on 6100 shapes (BF16; one to sixteen query heads per key/value head, S = 16 ... 16384).  What decides:
//   * few workgroups: a wavefront per 32 keys with tiles of its own (..14; D = 160 ..12), whose chains are the shortest, while the CUs
//     hold all of its workgroups; where a group's heads make the chains long, eight streams at D = 64 (2418);
//   * more of them: workgroups that share tiles, 64 keys in two or four streams (4122, 2222, 2424, 4224) or 128 (2241, 4141, 4121),
//     the form that comes out just below a whole number of workgroups per CU;
//   * many workgroups: the passes apart, which are level there or ahead and save reading O and dO once more (us, joint / apart: D = 64, 64
//     heads over 32 of S = 8192 9073 / 8654, 88 over 44 of S = 2048 364 / 333; D = 96, 60 over 30 of S = 2048 350 / 306).  But D = 128
//     with grouped heads, where 4141 is ahead at any size (80 heads over 20 of S = 4096 2005 / 2206, 48 over 12 of S = 8192 4731 / 4825,
//     64 over 16 of S = 8192, causal, 3287 / 3383) unless the passes' workgroups of keys come in whole rounds without the mask (64 over
//     16 of S = 8192 6285 / 6239, of S = 4096 1602 / 1589; level at S = 2048, 433 / 440 at S = 1024), and D = 64 and 96 without the mask on long
//     chains up to the lines below (12 to 20 % just past whole rounds of the passes' workgroups).
// On 1473 other shapes (profiles/sdpa_bwd_joint_forms.csv) this choice is 1.9 % from the best of all forms on average, and 0.89, 0.88,
// 0.87 and 0.64 of the time of the two passes with streams in each (D = 160: three passes) that went before; more than 10 % behind
// those on 7, more than 3 % on 36.  On 589 of 64 to 1024 full key tiles, powers of two, D = 64 to 128: 0.97 of that time, more than
// 10 % behind on 2, 3 % on 33.
inline int pick_bwd_joint(int D, bool causal, int heads, int group, int S)
{
    const long long tiles = (S + 127) / 128, nk = heads / group * tiles, n = nk + heads * tiles;
    const long long chain = (long long)group * ((S + 31) / 32), work = nk * chain;
    // 2214 with its workgroups of 32 keys and of 64 queries on a CU each
    const bool spread = heads / group * (long long)((S + 31) / 32) + heads * (long long)((S + 63) / 64) <= 256;
    // the passes in forms of their own (pick_bwd_form) are whole rounds: long chains then gain nothing from one grid (us, joint / apart:
    // four heads over 2 of S = 8192, causal, D = 96 281 / 213, D = 128 358 / 286; 32 heads of S = 2048, D = 128 225 / 213)
    const bool even = chain > 24 && (nk == 128 || nk == 256 || nk % 512 == 0);
    if (D == 64 && !causal && even && nk >= 512) return 0;
    if (D == 96 && even && (group == 1 || !causal || nk <= 256)) return 0;
    if (D == 128 && even && (group == 1 || nk == (causal ? 256 : 128) || (causal && group == 2 && nk == 128))) return 0;
    if (D == 64 && group == 1) {
        if (S <= 256) return n <= 330 || (n <= 440 && S <= 190) ? 4122 : causal ? 2241 : 0;
        if (causal) {
            if (n <= 256 && chain >= 30) return 1414;
            return n <= 150 ? 2214 : n <= 514 ? 2222 : n <= 1850 ? 2241 : 0;
        }
        if (n <= 256) return n <= 130 ? 1414 : n <= 170 ? 2214 : 2222;
        if (n <= 950) return S <= 600 || n <= 340 ? 4122 : 2241;
        return S >= 1600 && n <= 1850 ? 2241 : 0;
    }
    if (D == 64) {
        if (nk <= 34) return chain <= 35 ? 4114 : 2418;
        if (causal) {
            if (nk <= 130) return S <= 270 ? (group <= 3 ? 4122 : 4114) : chain <= 260 || nk > 64 ? 2214 : 2418;
            return nk > 580 ? 0 : group == 2 && S > 900 ? 2222 : chain <= 600 ? 4122 : 4114;
        }
        if (nk <= 110) return chain > 350 || (S > 620 && group > 2) ? 2214 : S > 620 ? 1414 : nk <= 80 ? 4114 : 4122;
        if (nk <= 310) return nk == 256 ? 2241 : n <= 870 && S > 270 ? 2222 : 4122;
        return S > 2300 && nk <= 1200 ? 2241 : 0;
    }
    if (D == 96 && group == 1) {
        if (causal ? n <= 70 : spread) return 2214;
        if (causal) {
            if (n <= 232 && chain >= 30) return n <= 128 ? 2424 : 0;
            return n <= 514 || (n <= 960 && chain > 64) ? 2222 : n <= 960 ? 2241 : 0;
        }
        if (work <= 2800) return 4122;
        if (n <= 120) return 2424;
        if (n <= 300) return n <= 170 && chain >= 100 ? 4224 : 0;
        if (n <= 340) return 4122;
        return n <= 860 || (S >= 3000 && n <= 2700) ? 2241 : 0;
    }
    if (D == 96 && causal) {
        if (group == 2 ? nk <= 32 : nk <= 51 || (nk <= 72 && chain > 100)) return 2214;
        if (S <= 63) return 4122;
        if (nk <= 185 && S > 550) return 4224;
        return group >= 3 && nk > 256 && nk <= 750 ? 4122 : 0;
    }
    if (D == 96) {
        if (nk <= 34) return 2214;
        if (chain <= 15) return 4122;
        if (chain > 520) return nk <= 740 ? 4224 : 0;
        return n <= 260 ? 2424 : nk > 78 && n <= 600 ? 2222 : 0;
    }
    if (D == 128 && group == 1) {
        if (causal) {
            if (n <= 98) return chain <= 3 ? 2241 : chain <= 6 ? 4122 : 2214;
            if (S <= 370) return n <= 170 ? 4122 : n <= 350 ? 4141 : 0;
            return n <= 170 ? 4224 : 0;
        }
        if (n <= 168) return S <= 90 ? 4141 : S > 160 && spread ? 2214 : S <= 480 ? 4122 : 4224;
        if (chain == 2 && nk > 128) return 0;
        if (work <= 3000) return 4141;
        if (n <= 290) return n <= 256 ? 0 : 4224;
        return work > 6150 && (n <= 900 || (n <= 2000 && S >= 1500)) ? 2241 : 0;
    }
    if (D == 128) {
        if (nk <= (group == 2 ? 32 : 40)) return chain <= 6 ? 4122 : 2214;
        if (nk > (causal ? 290 : 150)) return !causal && nk % 512 == 0 && S > 1920 ? 0 : 4141;
        if (chain <= 6) return 4141;
        if (causal) return chain > 260 || (group >= 3 && S > 650) ? 4224 : 0;
        return chain > 150 || n <= 260 ? 4224 : 0;
    }
    if (group == 1) return n <= 90 ? (S <= 64 ? 4121 : 2212) : n <= (causal ? 800 : 2000) ? 4121 : 0;
    if (nk <= (S <= 64 ? 60 : 51)) return 2212;
    if (nk <= 75 && S > 64) return 4222;
    if (causal && nk >= 240) return 0;
    if (chain > 80 && nk < (causal ? 240 : chain > 400 ? 130 : 100)) return 4222;
    return nk <= 500 ? 4121 : 0;
}

// ---- five products, dQ summed from block to block (sdpa_bwd_chain_kernel.h)
constexpr int kChainWaves = 4, kChainKeys = 64 * kChainWaves;       // wavefronts and keys of a workgroup
constexpr int kChainGroups = 256, kChainXcds = 16;                  // workgroups: one per CU; XCDs that a hardware id can name
constexpr int kChainFlag = 32;                                      // words from one progress counter to the next: a cache line each
constexpr int kChainQueueBytes = 128 * (1 + kChainXcds);

// Where its workspace holds what: the queue and the claims of every XCD and the progress counters (zero at the start), the row statistics,
// 32 rows per tile, and the sums.  An XCD's workgroups look at the places of all its claims and of one past the end each at most.
struct ChainLayout {
    int nT, nB, nclaims, max_slots;
    unsigned stat_bytes;
    size_t zero_bytes, stats_at, part_at, bytes;
};
inline ChainLayout chain_layout(int heads, int group, int S, int D, int per_claim)
{
    ChainLayout l{};
    const int HK = heads / group;
    l.nT = (S + 31) / 32;
    l.nB = (S + kChainKeys - 1) / kChainKeys;
    l.nclaims = (HK + per_claim - 1) / per_claim;
    l.max_slots = l.nclaims + kChainGroups + 1;
    l.zero_bytes = kChainQueueBytes + (size_t)kChainXcds * l.max_slots * 4 + (size_t)HK * l.nB * kChainWaves * kChainFlag * 4;
    l.stats_at = (l.zero_bytes + 255) & ~(size_t)255;
    l.stat_bytes = (unsigned)((size_t)heads * l.nT * 32 * 4);
    l.part_at = (l.stats_at + 2 * (size_t)l.stat_bytes + 255) & ~(size_t)255;
    l.bytes = l.part_at + (size_t)heads * l.nT * 32 * D * 4;
    return l;
}

// Key/value heads that an XCD claims at a time if a call takes the five products, else 0.  In steps of 256 keys by 32 queries, one per workgroup:
// `ideal` is the call's work dealt over 256 CUs (causal: half the plane), `cost` what its workgroups take, who get blocks of 256 keys
// by whole heads per XCD:
//   * rounds of 32 blocks; causal, where the blocks of a head get shorter, all blocks of the XCD dealt over its 32 CUs, but no less than the
//     longest block of the last claim, which starts when the claims before it are through;
//   * four steps of prologue and epilogue per round, and a step per block that follows another of its head at the same time: the fewer
//     heads in a claim, the more;
//   * 2.2 % for every doubling of the claim's blocks beyond two per CU, of which the L2 holds less.
// (us, claims of 1, 2, 4, 8 heads, D = 128 causal: 64 heads S = 8192 2908, 2800, 2868, 2925; S = 2048 277, 268, 238, 240.)
// The step itself is 0.75 ... 0.9 of the two passes' time for the same work, which leaves the first of the lines below (us, passes / five
// products, mean of both types and of several runs; ideal / cost):
//   D = 128  64 heads S = 1024 117 / 114 (0.80), 32 heads S = 2048 213 / 201 (0.84), 16 heads S = 3777 383 / 346 (0.80); causal 230 heads S = 2048
//            892 / 898 (0.77), 64 heads S = 2048 249 / 232 (0.80); grouped, causal 192 over 64 heads S = 2304 888 / 888 (0.86);
//   D = 96   32 heads S = 2048 174 / 170 (0.84), 128 heads S = 1024 178 / 171 (0.87); causal 64 heads S = 2779 327 / 334 (0.83), 128 heads S = 3456
//            968 / 935 (0.87);
//   D = 64   (what a wavefront issues beside the products weighs twice as much) 8 heads S = 8192 460 / 464 (0.88), 128 heads S = 2048 462 / 439
//            (0.93), 64 heads S = 8192 3476 / 3279 (0.98); causal 32 heads S = 8192 896 / 847 (0.93); grouped, causal not at all (64 over 16
//            heads S = 8192 1798 / 1901, 0.96).
// Where the step is short, at D = 64, and causal at D = 96, a call has to reach a second line as well, with eight or four more steps of
// prologue and epilogue per round and a quarter of the steps of a claim's start for every claim that follows another: D = 64, 384 over 128
// heads S = 512 101 / 105, 1648 over 206 heads S = 1408 2818 / 3004, causal 128 heads S = 4096 962 / 987; D = 96, causal, 64 heads S = 2432 260 / 269,
// 222 heads S = 2048 666 / 687.
// Timed on 1943 shapes above the first lines, most within a tenth: 34 of them are below the second ones (mean of five products / passes 1.01);
// the others are at 0.915 on average, 18 of them above 1.02 (the worst 92 over 23 heads S = 4992, causal, D = 128, 1.08).  One card and
// the next differ by 3 % in that quotient.
// D = 160 has no registers for 64 keys per wavefront (320 accumulators); with 32 it would, which is not built.  At most 2 GiB of sums, and 1 GiB per group of heads (the range of their descriptor).
constexpr size_t kChainMostBytes = (size_t)2 << 30;
inline int pick_bwd_chain(int D, bool causal, int heads, int group, int S)
{
    const long long HK = heads / group, nT = ((long long)S + 31) / 32, nB = ((long long)S + kChainKeys - 1) / kChainKeys;
    if (D == 160 || (D == 64 && causal && group > 1) || HK * nB < 128) return 0;
    if (heads * nT * 32 * D * 4 > (long long)kChainMostBytes || group * nT * 32 * D * 4 >= 1ll << 30) return 0;
    const long long per_head = group * (causal ? nB * nT - 4 * nB * (nB - 1) : nB * nT);     // steps (causal: blocks of nT, nT - 8, ... tiles)
    long long pick = 0, least = 0, more = 0;      // costs times 1000
    for (long long m = 1; m <= (HK + 7) / 8 && m <= 32; ++m) {
        const long long most = ((HK + m - 1) / m + 7) / 8 * m, rounds = (most * nB + 31) / 32;      // heads of the XCD that gets the most
        const long long links = nB < (32 + m - 1) / m ? nB : (32 + m - 1) / m;
        long long cost = rounds * group * nT + links;
        if (causal) {
            const long long share = (most * per_head + 31) / 32, last = (most - m) * per_head / 32 + group * nT + links;
            cost = share > last ? share : last;
        }
        cost = (cost + 4 * rounds) * 1000;
        for (long long b = m * nB; b >= 128; b /= 2) cost += cost / 45;
        if (pick == 0 || cost < least) {
            pick = m;
            least = cost;
            more = (D == 64 ? 8000 : 4000) * rounds + 250 * links * (most / m - 1);
        }
    }
    const long long ideal = HK * S * group * nT / (causal ? 2 : 1);      // times 256 * 256
    auto reaches = [&](long long cost, int line) { return ideal * 15625 >= cost * 1024 * line; };        // line per mille, both sides over 64
    if (!reaches(least, D == 64 ? (!causal && group >= 4 ? 875 : 870) : causal && group > 1 ? 850 : D == 96 ? (causal ? 790 : 830) : causal ? 760 : 780)) return 0;
    if (D == 64 && !reaches(least + more, causal ? 800 : group > 1 ? 805 : 750)) return 0;
    if (D == 96 && causal && group == 1 && !reaches(least + more, 728)) return 0;
    return (int)pick;
}

}  // namespace tsdpa
