// C-ABI of the tiled SDPA library: argument validation, tile and split heuristics, dispatch.
// See include/tiled_sdpa.h for the contract of every entry point.
#include "tiled_sdpa.h"

#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdint>
#include <limits>
#include <mutex>
#include <random>

#include "sdpa_bwd_pick.h"
#include "sdpa_fwd_launch.h"
#include "sdpa_merge_kernel.h"

// Split states of tiled_sdpa_fwd_kvcache_static: device memory that belongs to the library, one copy per
// GPU the code object is loaded on.  In host code this name is only a handle for hipGetSymbolAddress;
// the address kernels and copies use is the one that call returns (static_scratch_ptr below).
static __device__ __align__(256) unsigned char scratch[TSDPA_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kVersion = 300;  // 0.3.0

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];      // per device: address of that device's copy of `scratch`, once looked up
std::mutex g_scratch_mutex;

// Device address of the current device's copy of `scratch` (looked up once per device, with that device
// current); nullptr if the runtime cannot name it.  Allocates nothing.
void *static_scratch_ptr()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

bool valid_tile(int tm, int tn, int D)
{
    // 256 query rows per workgroup: an addition to the paper's Table 1 grid, built for 64-row K/V tiles only
    if (tm == 256) return tn == 64;
    if (!(tm == 64 || tm == 128) || !(tn == 32 || tn == 64 || tn == 128)) return false;
    // 128-row K/V tiles up to D = 128 (above D = 64 the kernel works through such a tile in two halves, its
    // score accumulators for 128 rows not fitting the registers beside the output accumulator); at D = 160
    // the four tile slots would take 256 KiB of LDS
    return tn != 128 || D <= 128;
}

// Shape heuristic (the static counterpart of the paper's shape-aware schedule policy, Section 5.6).
void pick_tile(int BH, int S, int D, bool causal, int *tm, int *tn)
{
    // From the tile sweeps on MI355X (every tile of a shape timed in turn, the order reversing from round to
    // round): among the paper's query tiles, 128 rows per workgroup (four wavefronts) win wherever a sequence is
    // longer than two such tiles.  Up to D = 128 the two K/V tile heights are within 2 % of each other on
    // long sequences: 32 rows fit three wavefronts per SIMD, 64 rows halve the barriers and are built
    // with the scheduler that suits them.  The 64-row tile is ahead by 4-14 % on mid-length sequences
    // (512-2048) and under the causal mask, where the finer diagonal of the 32-row tile does not pay
    // for its barriers; at D = 128 its masked step also spills, so every S above one tile takes 64
    // rows there.  Short sequences (S = 197, 333) are level or better on 32 rows at D = 64, 96 and 160.
    // At D = 160 the 64-row tile, whose four slots of unpadded rows are 80 KiB and leave room for two workgroups
    // per CU, is 3-5 % ahead under the mask and 5-20 % ahead without it from S = 512 up to where the 256-row
    // tile below takes over.
    *tm = S <= 64 ? 64 : 128;
    *tn = 32;
    if (D == 128 && S > 64) *tn = 64;
    if (D != 128 && S >= 512) *tn = 64;
    // up to two 128-row tiles per head and fewer of them than CUs: 64 query rows per workgroup start twice as
    // many (1-4 % at D = 128, 2-12 % at D = 160; level at D = 64 and 96)
    if (D >= 128 && S <= 256 && (long long)BH * ((S + 127) / 128) < 256) *tm = 64;
    // many short heads under the mask at D = 96 and 160 (S = 512, 1024; four 128-row workgroups per CU and more):
    // the 64 x 32 tile, which cuts the diagonal finest, is 4-7 % ahead
    if (causal && (D == 96 || D == 160) && S >= 512 && S <= 1024 && (long long)BH * ((S + 127) / 128) >= 1024) {
        *tm = 64;
        *tn = 32;
    }
    // 256 query rows per workgroup (eight wavefronts share every K/V tile: half the tile loads per MFMA; one
    // workgroup per CU) win from D = 96 upward once they give every CU a workgroup and the sequence is long
    // enough: 2-3 % at D = 96 from S = 4096 (level at 2048, 6 % behind there with 256 heads), 3 % at D = 128
    // from S = 2048, 1-2.5 % over 128 x 64 at D = 160 from S = 1024.
    // Not under the causal mask (a workgroup's diagonal band is four masked tiles instead of two and the query
    // tiles of a head balance worse: within 2 % either way at S = 8192 and 16384, 5-25 % slower at S = 2048),
    // not at D = 64 (3-14 % slower).
    const long long wg256 = (long long)BH * ((S + 255) / 256);
    bool wide = !causal && D >= 96 && wg256 >= 256 && S >= (D == 160 ? 1024 : D == 96 ? 4096 : 2048);
    // (D = 160 below S = 4096: ahead while a CU gets up to three such workgroups, 3-4 % behind 128 x 64 with more)
    if (D == 160 && S < 4096 && wg256 >= 1024) wide = false;
    if (wide) {
        *tm = 256;
        *tn = 64;
    }
}

// Streams of K/V tiles per workgroup of the square problem, and the query rows that go with them (1: the plain form on
// pick_tile's tile).  Up to one workgroup of 128 rows per CU a SIMD has one wavefront or none, which waits through the
// whole chain of tiles alone; streams cut the chain, fewer rows make more workgroups.  From timings of every form on 680
// shapes (4 ... 512 such workgroups, S = 64 ... 8192, BF16; mean gain of this choice over them 16-38 % by head dim and
// mask, within 0.2-2 % of the best form; us, plain -> chosen): 32 workgroups, S = 512 8.1 -> 5.8 (D = 64), 10.1 -> 7.2 (D = 96
// causal); 64 workgroups, S = 1024 12.8 -> 7.5, S = 8192 78.7 -> 26.7 (D = 64), 94.4 -> 36.2 (D = 96 causal); 128
// workgroups, S = 4096 41.5 -> 24.5 (D = 64), 59.6 -> 35.0 (D = 128 causal); 160 workgroups, S = 4096 causal 41.8 -> 23.3
// (D = 64); 256 workgroups, S = 2048 causal 28.2 -> 21.4 (D = 96); without the mask, where nothing is uneven, 3-8 % there.
int pick_streams(long long BH, int S, int D, bool causal, int *tm)
{
    const long long n = BH * ((S + 127) / 128);      // workgroups of the plain form
    const int chain = (S + 31) / 32;
    auto form = [&](int rows, int streams) { *tm = rows; return streams; };
    // (the plain 64 x 32 tile spills in its masked step at D = 128: one key tile per stream, 12.2 -> 8.5 with 512 heads)
    if (chain == 2 && causal && D == 128 && n <= 512) return form(64, 2);
    if (chain <= 2 || n > 400) return 1;
    if (n <= 64) {
        if (!causal && chain <= 4) return 1;
        return D == 64 && chain >= 64 ? form(32, 8) : form(32, 4);
    }
    if (n <= 128) {
        if (causal && D == 64 && chain >= 16) return form(32, 4);
        if (causal && D == 160 && chain >= 64) return form(32, 4);
        if (chain <= 4) return causal && D != 128 ? form(64, 2) : 1;
        return chain >= 32 ? form(64, D == 160 ? 3 : 4) : form(64, 2);
    }
    if (n <= 256) {
        if (!causal) return chain < 32 ? 1 : D == 64 ? form(64, 2) : form(128, 2);
        if (chain >= 64 && n <= 192) return D == 64 ? form(32, 4) : form(64, D == 160 ? 3 : 4);
        if (chain >= 64 && D == 64) return form(64, 4);
        return chain >= 8 ? form(64, 2) : 1;
    }
    if (!causal || chain < (n <= 320 ? 32 : 64)) return 1;
    return D == 64 && chain >= 128 ? form(64, 4) : form(64, 2);
}

int validate_shape(int B, int H, int S, int D, int dtype)
{
    if (dtype != TSDPA_F16 && dtype != TSDPA_BF16) return TSDPA_ERR_BAD_DTYPE;
    if (D != 64 && D != 96 && D != 128 && D != 160) return TSDPA_ERR_UNSUPPORTED_D;
    if (B < 0 || H < 0 || S < 0) return TSDPA_ERR_BAD_SHAPE;
    const int64_t bh = (int64_t)B * (int64_t)H;
    // the grid is B*H*ceil(S/tile_m) <= B*H*ceil(S/64) workgroups and must fit an int
    if (bh > 0 && S > 0 && bh * (((int64_t)S + 63) / 64) > (int64_t)std::numeric_limits<int>::max())
        return TSDPA_ERR_BAD_SHAPE;
    // one head's K (or V) is addressed through a 32-bit byte range with room for a "fetch nothing"
    // offset above it: keep it, prefetch distance included, below 2^30 bytes
    if (((int64_t)S + 1024) * D * 2 >= ((int64_t)1 << 30)) return TSDPA_ERR_BAD_SHAPE;
    return TSDPA_OK;
}

// Splits along the key axis (from timings on MI355X).  None when the query tiles alone give every CU
// two workgroups.  64- and 256-row query tiles (and the fewest splits that the library settles for): two workgroups per CU if
// every split then still streams 16 tiles or more (long caches: more loads in flight pay), else one per CU, never cutting runs
// shorter than 4 tiles for up to 64 query rows or 16 tiles beyond (each split of a query tile writes and the
// merge re-reads T_M x D floats, which a short run does not amortise).
int round_splits(int64_t base, int64_t tiles, int Sq)
{
    int64_t want = (512 + base - 1) / base;
    if (tiles / want < 16) {
        want = (256 + base - 1) / base;
        const int64_t shortest = Sq <= 64 ? 4 : 16;
        const int64_t most = tiles / shortest > 1 ? tiles / shortest : 1;
        if (want > most) want = most;
    }
    return (int)(want > TSDPA_MAX_SPLITS ? TSDPA_MAX_SPLITS : want);
}

// 128-row query tiles: the count of the least cost, in steps of 64 keys.  A CU holds two workgroups and no more, so the grid runs
// in rounds of 512, each as long as a run; a last round (or the only one) that gives a CU one workgroup at most takes
// 0.72 of that, at D = 160 0.9 (two splits against one: 204 tiles of 3776 keys there 0.76 of the time, 252 of 3648 keys at D = 64
// 0.98).  Then a run's prologue (0.7), the merge kernel (2.3), the states that it reads (6.7 for every 512 tiles) and its walk over
// the splits (0.19 each).  The constants are a fit to 700 calls, each timed at every split count (BF16; 8 to 511 tiles, 1500 to 40000
// keys, lengths from all, half and a tenth of the capacity on): on average 1.3 % behind the best count, where 512 / tiles rounded
// up was 15.6 % and rounded down 5.3 % (us, up / down / this: 16 tiles of 11000 keys 27.5 / 27.5 / 22.9, 144 of 16384, lengths from a
// tenth, 78 / 93 / 84, 156 of 4520 97 / 78 / 78).  Behind the former by more than 10 %: 6 of the 700, most of them with lengths from a
// tenth of the capacity.  Up to four rounds (eight would be 0.1 % ahead at twice the workspace) of runs of 512 keys or more.
// A longer cache never gets fewer splits, so that a workspace sized for the capacity serves every length on the way there: the
// cost is keys * a(n) + b(n) with b growing in n, and the counts that 512 keys per run leave out are the largest.  (With runs
// rounded up to whole tiles, which gained nothing on the 700 calls, 24 tiles had 21 splits at 15872 keys and 20 at 16384.)
int pick_splits(int BH, int Sq, int Skv, int D, int tm, int tn, bool fewest = false)
{
    const int64_t base = (int64_t)BH * ((Sq + tm - 1) / tm);
    const int tiles = (int)(((int64_t)Skv + tn - 1) / tn);
    if (base <= 0 || base >= 512) return 1;
    if (tm != 128 || fewest) return round_splits(base, tiles, Sq);
    const double alone = D == 160 ? 0.9 : 0.72;
    int best = 1;
    double least = 0;
    for (int n = 1; n <= TSDPA_MAX_SPLITS && (n == 1 || (n * (int)base <= 2048 && Skv / n >= 512)); ++n) {
        const int grid = n * (int)base, last = grid % 512;
        const double rounds = grid / 512 + (last > 256 ? 1.0 : last > 0 ? alone : 0.0);
        const double run = Skv / (64.0 * n);
        const double cost = rounds * (run + 0.7) + (n == 1 ? 0.0 : 2.3 + 6.7 * grid / 512 + 0.19 * n);
        if (n == 1 || cost < least) {
            best = n;
            least = cost;
        }
    }
    return best;
}

// A 64-bit number that no other call of any process has had, as far as chance goes: a counter from a random start,
// scrambled (the splitmix64 finaliser, a bijection) so that it looks like no data anybody would store.
unsigned long long call_ticket()
{
    static std::atomic<unsigned long long> counter{[]() noexcept {
        try {
            std::random_device rd;
            return ((unsigned long long)rd() << 32) ^ rd();
        } catch (...) {          // no random source: the time in nanoseconds, and where the loader put this library
            return (unsigned long long)std::chrono::system_clock::now().time_since_epoch().count() ^ ((unsigned long long)(uintptr_t)&kVersion << 24);
        }
    }()};
    unsigned long long x = counter.fetch_add(0x9E3779B97F4A7C15ull, std::memory_order_relaxed);
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x != 0 ? x : 1;
}

// Most query rows per key/value head that the decoding kernel takes (its tile is not the caller's to choose); above 16
// rows pick_streams_kv may send a call elsewhere.
constexpr int kDecodeRows = 32;

// Splits of a decoding step (BF16, cold cache, us; s = splits): one workgroup per CU in all, of runs of at least 128 keys.
// None where a workgroup is through a head's K about as soon as it could be through the second look at the states: 105000
// elements, or 200000 with more than 64 heads, where the CUs are nearly full without (one split / the best of more: 12 heads
// of 1608 keys D = 64 6.9 / 7.8; 15 of 627 D = 128 7.4 / 7.9; 64 of 746 D = 128 9.5 / 10.6; 70 of 2048 D = 96 12.8 / 14.3; 24
// heads of 772 D = 160, past the line, 10.4 / 9.3; with more than 16 rows several runs are ahead: 10 heads of 20 rows, 621 keys
// D = 160 13.9 / 10.8).  Nor from half as many key/value heads as CUs on: a pass is then as fast
// (256 heads of 8192 keys: s1 177, s2 181, s4 185; lengths from a quarter of that: 127, 131-133, 130-132; 160 heads of 1024:
// 18.0 / 22.5 / 23.5; 96 heads of 3000: 28.1 / 24.2 / 25.9; 32 heads of 8192: s4 30.9, s8 27.4, s16 28.5; 84 heads of 4096,
// all full: s2 29.4, s3 30.4, and with lengths from a tenth of that s2 47.2, s3 38.1 for 66 of 8127).
int pick_splits_decode(int BH, int rows, int Skv, int D)
{
    if (rows <= 16 && (int64_t)Skv * D <= (BH > 64 ? 200000 : 105000)) return 1;
    const int most = Skv > 256 ? (Skv + 127) / 128 : 1;
    int want = BH >= 128 ? 1 : BH > 64 ? 2 : 256 / BH;
    if (want > most) want = most;
    if (want > TSDPA_MAX_SPLITS) want = TSDPA_MAX_SPLITS;
    return want;
}

void pick_tile_kv(long long heads, int Sq, int Skv, int D, int *tm, int *tn);

// The same for a block of queries against a cache (rows = query rows per key/value head, grouped heads folded; Skv the
// capacity).  Such a call used to be split over the key range only, with a whole state of rows x D floats per split through
// memory and at least sixteen 64-row tiles per split: 24 to 64 workgroups that each waited through their tiles alone.  BF16,
// us, splits alone -> streams (with the splits of default_splits): 8 workgroups of 128 rows, 512 keys 8.7 -> 5.9 (D = 64), 12.1 ->
// 8.5 (128), 15.4 -> 10.3 (160); 4096 keys 19.3 -> 10.0, 25.8 -> 14.0, 30.8 -> 18.6; 32 of them, 2048 keys 20.1 -> 13.2, 27.3 ->
// 18.2, 37.0 -> 22.0; 64, 2048 keys 21.8 -> 13.1, 30.4 -> 18.8, 40.8 -> 24.1; 128, 2048 keys 25.6 -> 16.9, 35.0 -> 26.5, 46.6
// -> 36.9; 160, 2048 keys 30.8 -> 25.2, 40.2 -> 36.9, 51.4 -> 45.6.  With many keys per workgroup (16384 from 16 workgroups on,
// 8192 from 32) the plain form's 128 rows per tile load win back what the shorter chain gains.
int pick_streams_kv(long long heads, int rows, int Skv, int D, int *tm)
{
    if (rows <= 16) return 1;
    const long long n = heads * (((long long)rows + 127) / 128), n32 = heads * (((long long)rows + 31) / 32);
    auto form = [&](int r, int streams) { *tm = r; return streams; };
    // 17 to 32 rows, where the decoding kernel is the other choice (us, decoding kernel -> here, weights in halves): 69
    // heads of 607 keys D = 96 17.7 -> 10.3, 92 of 1450 21.5 -> 17.9; 157 of 292 keys D = 128 13.2 -> 10.3; 147 of 309 keys D = 64
    // 8.4 -> 7.0; 112 heads of 256 keys D = 160 13.6 -> 9.2, 48 of 64 keys 8.2 -> 7.5.  Past 256 workgroups only
    // D = 64 has two on a CU (320 heads of 512 keys 11.7 -> 9.9, D = 128 21.4 -> 22.6), and there long caches of many heads are
    // the decoding kernel's (160 heads of 4096 keys 32.8 / 36.1).  D = 160 past 256 keys: the same kernel has no registers for
    // two halves of each weight (21 to 48 spilled, 8.9 -> 11.8), and whole ones leave a larger error than the decoding kernel's
    // runs (16 heads of 23 rows, 807 keys, FP16 2.86e-4 / 2.53e-4).
    if (rows <= kDecodeRows && D == 160 && Skv > 256 && (n > 64 || (n <= 16 && Skv < 2048))) return 1;
    if (rows <= kDecodeRows && (n > 64 || Skv <= 64)) {
        const bool pays = Skv <= 4096 && (n <= 128 || (Skv <= 2048 && D == 64 && n <= 512) || (D > 64 && n <= 256));
        return pays ? form(32, 4) : 1;
    }
    if (n <= 64) {
        const bool pays = Skv <= 4096 ? Skv > 64 : n32 <= 32 || (Skv <= 8192 && (D == 64 || (D <= 128 && n32 <= 128)));
        return pays ? form(32, 4) : 1;
    }
    if (Skv > 4096 || Skv <= 256) return 1;
    if (n <= 128) return Skv < 1024 ? form(64, 2) : form(64, D == 160 ? 3 : 4);
    return n <= (Skv < 1024 ? 160 : 192) ? form(64, 2) : 1;
}

// Whether a call of up to 32 rows multiplies each weight as two 16-bit halves, half of it rounded and what that leaves, so that the
// rounding is half as coarse.  (Halves rather than the rounded weight and its remainder: both are positive, so that an infinite
// value stays one.)  The weights of a run are rounded against the greatest score of its first tile, which itself is exact; a
// wavefront that takes its keys in several runs thus rounds less than one that takes them all.  So where one run, or streams, took
// the place of the decoding kernel's runs of a tile or two per wavefront, the error was 5 to 18 % larger, and is smaller this way
// (BF16, 16 heads, 2 rows, 744 keys, D = 96 in six runs 1.96e-3, in one 2.32e-3, this way 1.81e-3).  The calls take 0 to
// 4 % longer for it (us: 7 heads, 2 rows, 365 keys D = 64 in several runs 6.7, in one 4.6, this way 4.7; 68 heads, 26 rows, 1607 keys
// in the decoding kernel 16.3, in streams 14.7, this way 15.5).
bool pick_halves(int BH, int rows, int Skv, int D, int splits, int streams)
{
    if (Skv <= 256) return false;                 // (one run of a tile or two at all times)
    return streams > 1 ? rows <= kDecodeRows && BH > 64 && D < 160 : rows <= 16 && splits == 1 && BH < 128;
}

// Splits of a cache call whose tile is left to the library too.
int default_splits(int BH, int rows, int Skv, int D, bool fewest = false)
{
    int tile_m;
    const bool streams = pick_streams_kv(BH, rows, Skv, D, &tile_m) > 1;
    if (rows <= kDecodeRows && !streams) return pick_splits_decode(BH, rows, Skv, D);
    if (streams) {
        // one workgroup per CU in all, once a stream has sixteen tiles to share (the states of a split cost a second kernel).  Up to
        // 32 rows: with more than 64 heads what the decoding kernel has, which takes over as the cache grows (112 heads of 2048 keys D =
        // 64 s1 13.1, s2 14.9), but four from 1024 keys on at D = 160 (8 heads s1 12.8, s4 10.8; 27 heads 15.6 / 13.8; at D = 128
        // 9.4 / 9.8)
        const long long wg = (long long)BH * ((rows + tile_m - 1) / tile_m);
        if (rows <= kDecodeRows && BH > 64) return Skv < 2048 ? 1 : pick_splits_decode(BH, rows, Skv, D);
        if (tile_m > 32) return 1;
        const bool short_wide = !fewest && D == 160 && rows <= kDecodeRows && BH <= 64 && Skv >= 1024 && Skv < 2048;
        if (Skv < 2048 && !short_wide) return 1;
        const long long most = short_wide ? 4 : 16, want = 256 / wg;
        return want < 1 ? 1 : want > most ? (int)most : (int)want;
    }
    int tm, tn;
    pick_tile_kv(BH, rows, Skv, D, &tm, &tn);
    return pick_splits(BH, rows, Skv, D, tm, tn, fewest);
}

int validate_shape_kv(int B, int H, int Sq, int Skv, int D, int dtype, unsigned flags)
{
    if (dtype != TSDPA_F16 && dtype != TSDPA_BF16) return TSDPA_ERR_BAD_DTYPE;
    if (D != 64 && D != 96 && D != 128 && D != 160) return TSDPA_ERR_UNSUPPORTED_D;
    if (B < 0 || H < 0 || Sq < 0 || Skv < 0) return TSDPA_ERR_BAD_SHAPE;
    const int64_t bh = (int64_t)B * (int64_t)H;
    // B*H*ceil(Sq/64)*splits workgroups must fit an int
    if (bh > 0 && Sq > 0 &&
        bh * (((int64_t)Sq + 63) / 64) * TSDPA_MAX_SPLITS > (int64_t)std::numeric_limits<int>::max())
        return TSDPA_ERR_BAD_SHAPE;
    if (((int64_t)Skv + 1024) * D * 2 >= ((int64_t)1 << 30)) return TSDPA_ERR_BAD_SHAPE;
    if (bh > 0 && Sq > 0 && Skv == 0) return TSDPA_ERR_BAD_SHAPE;
    if ((flags & TSDPA_FLAG_CAUSAL) && Skv < Sq) return TSDPA_ERR_BAD_SHAPE;
    return TSDPA_OK;
}

// tiles of the Sq x Skv entry points: T_M in {64,128} x T_N in {32,64}, and 256 x 64 on a dense cache
bool valid_tile_kv(int tm, int tn, bool paged)
{
    if (tm == 256) return tn == 64 && !paged;
    return (tm == 64 || tm == 128) && (tn == 32 || tn == 64);
}

void pick_tile_kv(long long heads, int Sq, int Skv, int D, int *tm, int *tn)
{
    // (up to 32 rows the decoding kernel takes over, whose tile is its own)
    *tm = Sq <= 64 ? 64 : 128;
    // (D = 128: 64-row tiles on short caches too, 1.3 to 1.5 times as fast: 42 heads of 512 rows, 128
    // keys 11.7 -> 7.8 us, 210 of 920 rows, 230 keys 68.3 -> 48.0)
    *tn = Skv >= 512 || D == 128 ? 64 : 32;
    // D = 160: 32-row tiles are level or ahead (3-10 %) until the query block is long (2048 rows: 64-row tiles
    // 2-5 % ahead) or its 128-row tiles are fewer than the CUs (15 % ahead at one head's 512 or 1024 rows)
    if (D == 160) *tn = (Sq >= 2048 || (Sq >= 128 && Skv >= 512 && heads * ((Sq + 127) / 128) < 256)) ? 64 : 32;
}

}  // namespace

static int fwd_kv_impl(const void *q, const void *k, const void *v, void *o, float *lse, const int *kv_lens,
                       const int *block_table, int max_blocks, int block_shift,
                       int B, int H, int Hkv, int Sq, int Skv, int D, float scale, int dtype, void *stream,
                       int tile_m, int tile_n, unsigned flags,
                       int splits, void *workspace, unsigned long long workspace_bytes);

// Combines the states of a call's splits (a.BH heads of a.S rows).  Each kernel in the form that loads no more than the splits
// need: see its header.
template <typename T> static void launch_merge(const tsdpa::LaunchArgs &a, void *o, bool wide, int D)
{
    using namespace tsdpa;
    if (wide) {
        static_assert(kMergeLanes * kMergePerLane >= TSDPA_MAX_SPLITS, "every split needs a thread");
        const auto kernel = a.splits <= 4 * kMergeLanes ? sdpa_merge_wide_kernel<T, 4>
                          : a.splits <= 8 * kMergeLanes ? sdpa_merge_wide_kernel<T, 8> : sdpa_merge_wide_kernel<T, kMergePerLane>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)a.S, (unsigned)a.BH), dim3(D / 4, kMergeLanes), 0, a.stream,
                           (const float *)a.ws, (T *)o, a.lse, D, a.splits);
        return;
    }
    const unsigned rows = (unsigned)((int64_t)a.BH * a.S);     // below 2^30: see validate_shape_kv
    const dim3 block(D / 4, 256 / (D / 4));
    const auto kernel = a.splits <= 4 ? sdpa_merge_kernel<T, 4> : a.splits <= 8 ? sdpa_merge_kernel<T, 8> : sdpa_merge_kernel<T, 0>;
    hipLaunchKernelGGL(kernel, dim3((rows + block.y - 1) / block.y), block, 0, a.stream,
                       (const float *)a.ws, (T *)o, a.lse, rows, (unsigned)a.S, D, a.splits);
}

extern "C" {

int tiled_sdpa_version(void) { return kVersion; }

const char *tiled_sdpa_status_string(int status)
{
    switch (status) {
        case TSDPA_OK: return "ok";
        case TSDPA_ERR_NULL_PTR: return "null pointer for q, k, v or o";
        case TSDPA_ERR_BAD_SHAPE: return "bad shape: B, H, S must be >= 0 and the grid must fit an int";
        case TSDPA_ERR_BAD_DTYPE: return "bad dtype: expected TSDPA_F16 or TSDPA_BF16";
        case TSDPA_ERR_UNSUPPORTED_D: return "unsupported head dimension: D must be 64, 96, 128 or 160";
        case TSDPA_ERR_MISALIGNED: return "misaligned pointer: q, k, v, o need 16-byte, lse 4-byte alignment";
        case TSDPA_ERR_BAD_TILE: return "bad tile: tile_m in {64,128}, tile_n in {32,64,128} (128 not at D = 160), or (256,64), or both 0";
        case TSDPA_ERR_BAD_SCALE: return "bad scale: must be finite (NaN selects 1/sqrt(D))";
        case TSDPA_ERR_LAUNCH: return "kernel launch failed";
        case TSDPA_ERR_WORKSPACE: return "split workspace is null, misaligned or too small";
        case TSDPA_ERR_BAD_SPLITS: return "bad splits: must be 0 (heuristic) or 1..128";
        case TSDPA_ERR_STATIC_SCRATCH:
            return "split states exceed the library's static scratch buffer (or its address is unavailable): "
                   "use tiled_sdpa_fwd_kvcache with a workspace of the caller's, or fewer splits";
        default: return "unknown status";
    }
}

int tiled_sdpa_default_tile(int B, int H, int S, int D, int dtype, unsigned flags, int *tile_m, int *tile_n)
{
    if (!tile_m || !tile_n) return TSDPA_ERR_NULL_PTR;
    const int st = validate_shape(B, H, S, D, dtype);
    if (st != TSDPA_OK) return st;
    pick_tile(B * H, S, D, (flags & TSDPA_FLAG_CAUSAL) != 0, tile_m, tile_n);
    return TSDPA_OK;
}

int tiled_sdpa_tune_tile(const void *q, const void *k, const void *v, void *o,
                         int B, int H, int S, int D, float scale, int dtype, void *stream, unsigned flags,
                         int launches, int *tile_m, int *tile_n, float *ms_per_launch)
{
    if (!tile_m || !tile_n) return TSDPA_ERR_NULL_PTR;
    if (launches < 1 || launches > 1000) return TSDPA_ERR_BAD_SHAPE;
    int st = validate_shape(B, H, S, D, dtype);
    if (st != TSDPA_OK) return st;
    pick_tile(B * H, S, D, (flags & TSDPA_FLAG_CAUSAL) != 0, tile_m, tile_n);
    if (ms_per_launch)
        for (int i = 0; i < TSDPA_TUNE_TILES; ++i) ms_per_launch[i] = -1.0f;
    if ((int64_t)B * H * S == 0) return TSDPA_OK;
    if (!q || !k || !v || !o) return TSDPA_ERR_NULL_PTR;
    if ((((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15u) != 0) return TSDPA_ERR_MISALIGNED;
    if (std::isinf(scale)) return TSDPA_ERR_BAD_SCALE;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return TSDPA_ERR_LAUNCH;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return TSDPA_ERR_LAUNCH; }
    static const int tms[TSDPA_TUNE_TILES] = {64, 64, 64, 128, 128, 128, 256};
    static const int tns[TSDPA_TUNE_TILES] = {32, 64, 128, 32, 64, 128, 64};
    float best = -1.0f;
    st = TSDPA_OK;
    for (int i = 0; i < TSDPA_TUNE_TILES && st == TSDPA_OK; ++i) {
        const int tm = tms[i], tn = tns[i];
        if (!valid_tile(tm, tn, D)) continue;
        // one untimed launch (first use of an instantiation sets its attributes), then the timed run
        st = tiled_sdpa_fwd_ex(q, k, v, o, nullptr, B, H, S, D, scale, dtype, stream, tm, tn, flags);
        if (st != TSDPA_OK) break;
        if (hipEventRecord(e0, (hipStream_t)stream) != hipSuccess) { st = TSDPA_ERR_LAUNCH; break; }
        for (int r = 0; r < launches && st == TSDPA_OK; ++r)
            st = tiled_sdpa_fwd_ex(q, k, v, o, nullptr, B, H, S, D, scale, dtype, stream, tm, tn, flags);
        if (st != TSDPA_OK) break;
        float ms = 0.0f;
        if (hipEventRecord(e1, (hipStream_t)stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = TSDPA_ERR_LAUNCH; break; }
        ms /= (float)launches;
        if (ms_per_launch) ms_per_launch[i] = ms;
        if (best < 0.0f || ms < best) { best = ms; *tile_m = tm; *tile_n = tn; }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return st;
}

int tiled_sdpa_fwd_ex(const void *q, const void *k, const void *v, void *o, float *lse,
                      int B, int H, int S, int D, float scale, int dtype, void *stream,
                      int tile_m, int tile_n, unsigned flags)
{
    int st = validate_shape(B, H, S, D, dtype);
    if (st != TSDPA_OK) return st;
    if ((int64_t)B * H * S == 0) return TSDPA_OK;
    if (!q || !k || !v || !o) return TSDPA_ERR_NULL_PTR;
    const uintptr_t bits = (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o;
    if ((bits & 15u) != 0 || ((uintptr_t)lse & 3u) != 0) return TSDPA_ERR_MISALIGNED;
    int streams = 1;
    if (tile_m == 0 && tile_n == 0) {
        streams = pick_streams((long long)B * H, S, D, (flags & TSDPA_FLAG_CAUSAL) != 0, &tile_m);
        if (streams > 1) tile_n = 32;
        else pick_tile(B * H, S, D, (flags & TSDPA_FLAG_CAUSAL) != 0, &tile_m, &tile_n);
    } else if (!valid_tile(tile_m, tile_n, D))
        return TSDPA_ERR_BAD_TILE;
    if (std::isnan(scale)) scale = 1.0f / std::sqrt((float)D);
    if (std::isinf(scale)) return TSDPA_ERR_BAD_SCALE;

    tsdpa::LaunchArgs a{};
    a.streams = streams;
    a.q = q;
    a.k = k;
    a.v = v;
    a.o = o;
    a.lse = lse;
    a.BH = B * H;
    a.S = S;
    a.rows_per_head = S;
    a.c = std::fabs(scale) * 1.44269504088896340736f;
    a.tau = (flags & TSDPA_FLAG_EXACT_MAX) ? 0.0f : 8.0f;
    a.qsign = std::signbit(scale) && scale != 0.0f ? 0x80008000u : 0u;
    a.linear_grid = (flags & TSDPA_FLAG_LINEAR_GRID) ? 1 : 0;
    a.causal = (flags & TSDPA_FLAG_CAUSAL) ? 1 : 0;
    a.stream = (hipStream_t)stream;

    int err;
    if (dtype == TSDPA_F16) {
        switch (D) {
            case 64: err = tsdpa::launch_f16_d64(tile_m, tile_n, a); break;
            case 96: err = tsdpa::launch_f16_d96(tile_m, tile_n, a); break;
            case 128: err = tsdpa::launch_f16_d128(tile_m, tile_n, a); break;
            default: err = tsdpa::launch_f16_d160(tile_m, tile_n, a); break;
        }
    } else {
        switch (D) {
            case 64: err = tsdpa::launch_bf16_d64(tile_m, tile_n, a); break;
            case 96: err = tsdpa::launch_bf16_d96(tile_m, tile_n, a); break;
            case 128: err = tsdpa::launch_bf16_d128(tile_m, tile_n, a); break;
            default: err = tsdpa::launch_bf16_d160(tile_m, tile_n, a); break;
        }
    }
    return err == 0 ? TSDPA_OK : TSDPA_ERR_LAUNCH;
}

unsigned long long tiled_sdpa_kv_workspace_bytes(int B, int H, int Sq, int D, int splits)
{
    if (B < 0 || H < 0 || Sq < 0 || D < 0 || splits <= 1) return 0;
    return (unsigned long long)B * H * splits * Sq * (D + 2) * sizeof(float);
}

int tiled_sdpa_kv_default_splits(int B, int H, int Sq, int Skv, int D, int dtype, unsigned flags, int *splits)
{
    if (!splits) return TSDPA_ERR_NULL_PTR;
    const int st = validate_shape_kv(B, H, Sq, Skv, D, dtype, flags);
    if (st != TSDPA_OK) return st;
    if ((int64_t)B * H * Sq == 0) {
        *splits = 1;
        return TSDPA_OK;
    }
    *splits = default_splits(B * H, Sq, Skv, D);
    return TSDPA_OK;
}

int tiled_sdpa_kv_tile_splits(int B, int H, int Sq, int Skv, int D, int dtype, unsigned flags, int tile_m, int tile_n, int *splits)
{
    const int st = tiled_sdpa_kv_default_splits(B, H, Sq, Skv, D, dtype, flags, splits);
    if (st != TSDPA_OK || (int64_t)B * H * Sq == 0 || (tile_m == 0 && tile_n == 0)) return st;
    if (!valid_tile_kv(tile_m, tile_n, false)) return TSDPA_ERR_BAD_TILE;
    *splits = pick_splits(B * H, Sq, Skv, D, tile_m, tile_n);
    return TSDPA_OK;
}

int tiled_sdpa_fwd_kv(const void *q, const void *k, const void *v, void *o, float *lse,
                      int B, int H, int Sq, int Skv, int D, float scale, int dtype, void *stream,
                      int tile_m, int tile_n, unsigned flags,
                      int splits, void *workspace, unsigned long long workspace_bytes)
{
    return tiled_sdpa_fwd_gqa(q, k, v, o, lse, B, H, H, Sq, Skv, D, scale, dtype, stream, tile_m, tile_n, flags,
                              splits, workspace, workspace_bytes);
}

int tiled_sdpa_fwd_gqa(const void *q, const void *k, const void *v, void *o, float *lse,
                       int B, int H, int Hkv, int Sq, int Skv, int D, float scale, int dtype, void *stream,
                       int tile_m, int tile_n, unsigned flags,
                       int splits, void *workspace, unsigned long long workspace_bytes)
{
    return tiled_sdpa_fwd_kvcache(q, k, v, o, lse, nullptr, B, H, Hkv, Sq, Skv, D, scale, dtype, stream, tile_m,
                                  tile_n, flags, splits, workspace, workspace_bytes);
}

int tiled_sdpa_fwd_kvcache(const void *q, const void *k, const void *v, void *o, float *lse, const int *kv_lens,
                           int B, int H, int Hkv, int Sq, int Skv, int D, float scale, int dtype, void *stream,
                           int tile_m, int tile_n, unsigned flags,
                           int splits, void *workspace, unsigned long long workspace_bytes)
{
    return fwd_kv_impl(q, k, v, o, lse, kv_lens, nullptr, 0, 0, B, H, Hkv, Sq, Skv, D, scale, dtype, stream, tile_m,
                       tile_n, flags, splits, workspace, workspace_bytes);
}

int tiled_sdpa_fwd_kvcache_static(const void *q, const void *k, const void *v, void *o, float *lse,
                                  const int *kv_lens, int B, int H, int Hkv, int Sq, int Skv, int D, float scale,
                                  int dtype, void *stream, int tile_m, int tile_n, unsigned flags, int splits)
{
    // the checks that decide the split count, in the order of tiled_sdpa_fwd_kvcache, so that the size
    // of the split states is known before anything is enqueued
    int st = validate_shape_kv(B, H, Sq, Skv, D, dtype, flags);
    if (st != TSDPA_OK) return st;
    if (Hkv < 0 || (H > 0 && (Hkv == 0 || H % Hkv != 0))) return TSDPA_ERR_BAD_SHAPE;
    if ((int64_t)B * H * Sq == 0) return TSDPA_OK;
    if (splits < 0 || splits > TSDPA_MAX_SPLITS) return TSDPA_ERR_BAD_SPLITS;
    if ((int64_t)(H / Hkv) * Sq > (int64_t)std::numeric_limits<int>::max()) return TSDPA_ERR_BAD_SHAPE;
    if (splits == 0) {
        if (!(tile_m == 0 && tile_n == 0) && !valid_tile_kv(tile_m, tile_n, false)) return TSDPA_ERR_BAD_TILE;
        // (the count that runs best, or the smaller one if only that fits the buffer)
        for (const bool fewest : {false, true}) {
            splits = tile_m == 0 ? default_splits(B * Hkv, (H / Hkv) * Sq, Skv, D, fewest)
                                 : pick_splits(B * Hkv, (H / Hkv) * Sq, Skv, D, tile_m, tile_n, fewest);
            if (tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits) <= (unsigned long long)TSDPA_STATIC_SCRATCH_BYTES) break;
        }
    }
    const unsigned long long need = tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits);
    if (need > (unsigned long long)TSDPA_STATIC_SCRATCH_BYTES) return TSDPA_ERR_STATIC_SCRATCH;
    void *ws = nullptr;
    if (need > 0) {
        ws = static_scratch_ptr();
        if (ws == nullptr) return TSDPA_ERR_STATIC_SCRATCH;
    }
    // every word of the split states that the combination uses is written by the attention kernel of the same call ((m, l) of
    // every split; o of those with l != 0), so nothing has to be cleared
    return fwd_kv_impl(q, k, v, o, lse, kv_lens, nullptr, 0, 0, B, H, Hkv, Sq, Skv, D, scale, dtype, stream, tile_m,
                       tile_n, flags, splits, ws, need);
}

int tiled_sdpa_fwd_paged(const void *q, const void *k_pages, const void *v_pages, void *o, float *lse,
                         const int *kv_lens, const int *block_table,
                         int B, int H, int Hkv, int Sq, int max_blocks, int block_rows, int D,
                         float scale, int dtype, void *stream, int tile_m, int tile_n, unsigned flags,
                         int splits, void *workspace, unsigned long long workspace_bytes)
{
    // pages of 64 << n rows, so that a K/V tile of 32 or 64 rows never straddles two pages
    int shift = 6;
    while (shift < 20 && (1 << shift) != block_rows) ++shift;
    if (max_blocks < 0 || (1 << shift) != block_rows) return TSDPA_ERR_BAD_SHAPE;
    if ((int64_t)max_blocks * block_rows > (int64_t)std::numeric_limits<int>::max()) return TSDPA_ERR_BAD_SHAPE;
    const int cap = max_blocks * block_rows;
    const int st = validate_shape_kv(B, H, Sq, cap, D, dtype, flags);
    if (st != TSDPA_OK) return st;
    if ((int64_t)B * H * Sq != 0 && (!kv_lens || !block_table)) return TSDPA_ERR_NULL_PTR;
    if (((uintptr_t)block_table & 3u) != 0) return TSDPA_ERR_MISALIGNED;
    return fwd_kv_impl(q, k_pages, v_pages, o, lse, kv_lens, block_table, max_blocks, shift, B, H, Hkv, Sq, cap, D,
                       scale, dtype, stream, tile_m, tile_n, flags, splits, workspace, workspace_bytes);
}

}  // extern "C"

// Everything behind tiled_sdpa_fwd_kv / _gqa / _kvcache / _paged: one query block per query head against a
// cache of Skv rows per key/value head, dense (block_table NULL) or paged.
static int fwd_kv_impl(const void *q, const void *k, const void *v, void *o, float *lse, const int *kv_lens,
                       const int *block_table, int max_blocks, int block_shift,
                       int B, int H, int Hkv, int Sq, int Skv, int D, float scale, int dtype, void *stream,
                       int tile_m, int tile_n, unsigned flags,
                       int splits, void *workspace, unsigned long long workspace_bytes)
{
    int st = validate_shape_kv(B, H, Sq, Skv, D, dtype, flags);
    if (st != TSDPA_OK) return st;
    if (Hkv < 0 || (H > 0 && (Hkv == 0 || H % Hkv != 0))) return TSDPA_ERR_BAD_SHAPE;
    if ((int64_t)B * H * Sq == 0) return TSDPA_OK;
    // the G query heads of a group are adjacent, so q, o and lse are also [B, Hkv, G*Sq, ...]: the
    // kernel runs one "head" per key/value head over the G*Sq rows that read it
    const int G = H / Hkv;
    if ((int64_t)G * Sq > (int64_t)std::numeric_limits<int>::max()) return TSDPA_ERR_BAD_SHAPE;
    const int rows = G * Sq;
    if (!q || !k || !v || !o) return TSDPA_ERR_NULL_PTR;
    const uintptr_t bits = (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o;
    if ((bits & 15u) != 0 || (((uintptr_t)lse | (uintptr_t)kv_lens) & 3u) != 0) return TSDPA_ERR_MISALIGNED;
    const bool heuristic_tile = tile_m == 0 && tile_n == 0;
    if (heuristic_tile)
        pick_tile_kv((long long)B * Hkv, rows, Skv, D, &tile_m, &tile_n);
    else if (!valid_tile_kv(tile_m, tile_n, block_table != nullptr))
        return TSDPA_ERR_BAD_TILE;
    if (std::isnan(scale)) scale = 1.0f / std::sqrt((float)D);
    if (std::isinf(scale)) return TSDPA_ERR_BAD_SCALE;
    if (splits < 0 || splits > TSDPA_MAX_SPLITS) return TSDPA_ERR_BAD_SPLITS;
    if (splits == 0) {
        splits = default_splits(B * Hkv, rows, Skv, D);
        if (!heuristic_tile) {
            // the tile's own count, unless the workspace holds the states of the default count only (a caller may have sized it by
            // tiled_sdpa_kv_default_splits, which speaks of forms that an explicit tile never takes)
            const int own = pick_splits(B * Hkv, rows, Skv, D, tile_m, tile_n);
            if (own <= splits || (workspace && workspace_bytes >= tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, own))) splits = own;
        }
        // (the count that runs best, or the smaller one if only that fits what the caller gave, be it nothing)
        const unsigned long long given = workspace ? workspace_bytes : 0;
        if (tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits) > given) {
            const int few = heuristic_tile ? default_splits(B * Hkv, rows, Skv, D, true) : pick_splits(B * Hkv, rows, Skv, D, tile_m, tile_n, true);
            if (tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, few) <= given) splits = few;
        }
    }
    // Long query blocks against a dense cache of one length, no mask, no split: the 256-row query tile of the
    // square problem, under the same conditions.  Not where its workgroups begin a second round that 128-row ones, two per CU,
    // do without, the last 256 rows of the heads being half empty (us, 256 rows / 128: 29 heads of 2100 rows, D = 128, 1024 keys
    // 54.9 / 33.3, 4096 keys 188 / 113; 13 of 4900, D = 96, 4096 keys 159 / 93; 52 of 1100, D = 160, 4096 keys 253 / 154; one
    // round of either, 16 of 3900, D = 128, 4096 keys 111.9 / 113.1).
    const int64_t wide = (int64_t)B * Hkv * ((rows + 255) / 256);
    if (heuristic_tile && splits == 1 && block_table == nullptr && kv_lens == nullptr &&
        !(flags & TSDPA_FLAG_CAUSAL) && D >= 96 && rows >= (D == 160 ? 1024 : D == 96 ? 4096 : 2048) &&
        (wide == 256 || (wide > 256 && (int64_t)B * Hkv * ((rows + 127) / 128) >= 512))) {
        tile_m = 256;
        tile_n = 64;
    }
    if (splits > 1) {
        if (!workspace || ((uintptr_t)workspace & 15u) != 0 ||
            workspace_bytes < tiled_sdpa_kv_workspace_bytes(B, H, Sq, D, splits))
            return TSDPA_ERR_WORKSPACE;
    }

    tsdpa::LaunchArgs a{};
    a.q = q;
    a.k = k;
    a.v = v;
    a.o = o;
    a.lse = lse;
    a.BH = B * Hkv;
    a.S = rows;
    a.rows_per_head = Sq;
    a.kv_lens = kv_lens;
    a.heads_per_batch = Hkv;
    a.batches = B;
    a.block_table = block_table;
    a.max_blocks = max_blocks;
    a.block_shift = block_shift;
    a.tile_rot = (block_table == nullptr && rows <= tile_m) ? 1 : 0;    // one query tile per head: see the kernel
    a.c = std::fabs(scale) * 1.44269504088896340736f;
    a.tau = (flags & TSDPA_FLAG_EXACT_MAX) ? 0.0f : 8.0f;
    a.qsign = std::signbit(scale) && scale != 0.0f ? 0x80008000u : 0u;
    a.linear_grid = (flags & TSDPA_FLAG_LINEAR_GRID) ? 1 : 0;
    a.causal = (flags & TSDPA_FLAG_CAUSAL) ? 1 : 0;
    a.kv = 1;
    a.Skv = Skv;
    a.splits = splits;
    a.ws = (float *)workspace;
    a.stream = (hipStream_t)stream;

    int err;
    if (heuristic_tile) {
        int rows_per_wg;
        a.streams = pick_streams_kv((long long)B * Hkv, rows, Skv, D, &rows_per_wg);
        if (a.streams > 1) {
            tile_m = rows_per_wg;
            tile_n = 32;
        }
    }
    const bool decode = heuristic_tile && rows <= kDecodeRows && a.streams <= 1;
    a.halves = (decode || a.streams > 1) && pick_halves(a.BH, rows, Skv, D, splits, a.streams) ? 1 : 0;
    // The decoding kernel combines the runs itself while they are few: a mark (8 bytes) per run must fit a head's part of o,
    // and past 32 states per head, eight rows, or four columns for each thread, the one workgroup that does it is slower than the
    // merge kernel's many (time with the marks / with two kernels, over 300 shapes: one row 0.95 at 2 runs, 0.97 at 8, 1.04 at 20;
    // up to four rows 0.95, 0.99, 1.07; up to eight 0.99 at 2, 1.05 at 8; 9 to 16 rows 1.20 at 2; 24 heads, 8 rows of D = 160, 8
    // runs of 97 keys 11.0 us against 9.3)
    if (decode && splits > 1 && rows <= 8 && splits * rows <= 32 && splits <= rows * D / 4 &&
        rows * D <= 256 * tsdpa::decode_waves(a.BH, splits, Skv))
        a.ticket = call_ticket();
    if (decode) {
        err = dtype == TSDPA_F16 ? tsdpa::launch_decode_f16(D, a) : tsdpa::launch_decode_bf16(D, a);
    } else if (dtype == TSDPA_F16) {
        switch (D) {
            case 64: err = tsdpa::launch_f16_d64(tile_m, tile_n, a); break;
            case 96: err = tsdpa::launch_f16_d96(tile_m, tile_n, a); break;
            case 128: err = tsdpa::launch_f16_d128(tile_m, tile_n, a); break;
            default: err = tsdpa::launch_f16_d160(tile_m, tile_n, a); break;
        }
    } else {
        switch (D) {
            case 64: err = tsdpa::launch_bf16_d64(tile_m, tile_n, a); break;
            case 96: err = tsdpa::launch_bf16_d96(tile_m, tile_n, a); break;
            case 128: err = tsdpa::launch_bf16_d128(tile_m, tile_n, a); break;
            default: err = tsdpa::launch_bf16_d160(tile_m, tile_n, a); break;
        }
    }
    if (err != 0) return TSDPA_ERR_LAUNCH;
    if (a.ticket != 0) return TSDPA_OK;
    const size_t out_rows = (size_t)B * H * Sq;
    // Which merge: with more than eight splits (or after the decoding kernel, whose rows are few) a thread that walks them waits for its loads in several
    // batches, and when the rows are few (decoding) nothing else hides that: one workgroup per row, the
    // splits shared among eight threads (32 splits of 32 rows: 3.5 us against 12.5 us; 8 splits of 1024 rows at D = 64 and
    // 128 2-3 us less for the call, level at D = 160).  With thousands of
    // rows the walking threads are many enough to hide it themselves and launch an eighth of the threads
    // (8 splits of 8192 rows: 47 us per call against 55 us).
    if (splits > 1) {
        const bool wide = (splits > 8 || decode || (splits >= 4 && out_rows * D <= 131072)) && out_rows <= 2048;
        if (dtype == TSDPA_F16) launch_merge<_Float16>(a, o, wide, D);
        else launch_merge<__bf16>(a, o, wide, D);
        if (hipGetLastError() != hipSuccess) return TSDPA_ERR_LAUNCH;
    }
    return TSDPA_OK;
}

// Where the workspace of the five products begins within the caller's (behind the statistics that every other form keeps), and the
// bytes of both wherever the caller's begins.  At an address that 256 divides: a cache line of two tiles' sums, read for the first of
// them, would still be in the CU's cache, with what the second one's place held then, when that one's turn comes.
static uintptr_t chain_at(uintptr_t workspace, int BH, int S)
{
    return (workspace + 2 * ((size_t)BH * S + tsdpa::kBwdStatPad) * sizeof(float) + 255) & ~(uintptr_t)255;
}
static unsigned long long chain_workspace(int BH, int group, int S, int D, int per_claim)
{
    return chain_at(256 - 16, BH, S) + tsdpa::chain_layout(BH, group, S, D, per_claim).bytes;
}

extern "C" {

unsigned long long tiled_sdpa_bwd_workspace_bytes(int B, int H, int S)
{
    if (B < 0 || H < 0 || S < 0) return 0;
    return 2ull * ((unsigned long long)B * H * S + tsdpa::kBwdStatPad) * sizeof(float);
}

unsigned long long tiled_sdpa_bwd_full_workspace_bytes(int B, int H, int Hkv, int S, int D, unsigned flags)
{
    if (B < 0 || H < 0 || S < 0) return 0;
    const unsigned long long least = tiled_sdpa_bwd_workspace_bytes(B, H, S);
    if (validate_shape(B, H, S, D, TSDPA_F16) != TSDPA_OK || Hkv <= 0 || H % Hkv != 0 || (int64_t)B * H * S == 0 ||
        (int64_t)B * H * S >= ((int64_t)1 << 29))
        return least;
    const int per_claim = tsdpa::pick_bwd_chain(D, (flags & TSDPA_FLAG_CAUSAL) != 0, B * H, H / Hkv, S);
    return per_claim > 0 ? chain_workspace(B * H, H / Hkv, S, D, per_claim) : least;
}

int tiled_sdpa_bwd(const void *q, const void *k, const void *v, const void *o, const void *dout,
                   const float *lse, void *dq, void *dk, void *dv,
                   int B, int H, int S, int D, float scale, int dtype, unsigned flags,
                   void *workspace, unsigned long long workspace_bytes, void *stream)
{
    return tiled_sdpa_bwd_gqa(q, k, v, o, dout, lse, dq, dk, dv, B, H, H, S, D, scale, dtype, flags, workspace,
                              workspace_bytes, stream);
}

int tiled_sdpa_bwd_gqa(const void *q, const void *k, const void *v, const void *o, const void *dout,
                       const float *lse, void *dq, void *dk, void *dv,
                       int B, int H, int Hkv, int S, int D, float scale, int dtype, unsigned flags,
                       void *workspace, unsigned long long workspace_bytes, void *stream)
{
    if (dtype != TSDPA_F16 && dtype != TSDPA_BF16) return TSDPA_ERR_BAD_DTYPE;
    int st = validate_shape(B, H, S, D, dtype);
    if (st != TSDPA_OK) return st;
    if (Hkv < 0 || (H > 0 && (Hkv == 0 || H % Hkv != 0))) return TSDPA_ERR_BAD_SHAPE;
    // the statistics arrays are addressed through a 32-bit byte range
    if ((int64_t)B * H * S >= ((int64_t)1 << 29)) return TSDPA_ERR_BAD_SHAPE;
    if ((int64_t)B * H * S == 0) return TSDPA_OK;
    if (!q || !k || !v || !o || !dout || !lse || !dq || !dk || !dv) return TSDPA_ERR_NULL_PTR;
    const uintptr_t bits = (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)dout |
                           (uintptr_t)dq | (uintptr_t)dk | (uintptr_t)dv;
    if ((bits & 15u) != 0 || ((uintptr_t)lse & 3u) != 0) return TSDPA_ERR_MISALIGNED;
    if (std::isnan(scale)) scale = 1.0f / std::sqrt((float)D);
    if (std::isinf(scale)) return TSDPA_ERR_BAD_SCALE;
    if (!workspace || ((uintptr_t)workspace & 15u) != 0 ||
        workspace_bytes < tiled_sdpa_bwd_workspace_bytes(B, H, S))
        return TSDPA_ERR_WORKSPACE;

    tsdpa::BwdLaunchArgs a{};
    a.q = q; a.k = k; a.v = v; a.o = o; a.dout = dout; a.lse = lse;
    a.dq = dq; a.dk = dk; a.dv = dv;
    const size_t half = (size_t)B * H * S + tsdpa::kBwdStatPad;
    a.stats = (float *)workspace;
    a.stat_bytes = (unsigned)(half * sizeof(float));
    a.BH = B * H;
    a.S = S;
    a.group = H / Hkv;
    a.c = std::fabs(scale) * 1.44269504088896340736f;
    a.scale = scale;
    a.rsign = std::signbit(scale) && scale != 0.0f ? 0x80008000u : 0u;
    a.causal = (flags & TSDPA_FLAG_CAUSAL) ? 1 : 0;
    a.stream = (hipStream_t)stream;
    int err;
    const int per_claim = tsdpa::pick_bwd_chain(D, a.causal != 0, a.BH, a.group, S);
    if (per_claim > 0 && workspace_bytes >= chain_workspace(a.BH, a.group, S, D, per_claim)) {
        a.chain = (void *)chain_at((uintptr_t)workspace, a.BH, S);
        if (dtype == TSDPA_F16) {
            switch (D) {
                case 64: err = tsdpa::launch_bwd_chain_f16_d64(a, per_claim); break;
                case 96: err = tsdpa::launch_bwd_chain_f16_d96(a, per_claim); break;
                default: err = tsdpa::launch_bwd_chain_f16_d128(a, per_claim); break;
            }
        } else {
            switch (D) {
                case 64: err = tsdpa::launch_bwd_chain_bf16_d64(a, per_claim); break;
                case 96: err = tsdpa::launch_bwd_chain_bf16_d96(a, per_claim); break;
                default: err = tsdpa::launch_bwd_chain_bf16_d128(a, per_claim); break;
            }
        }
    } else if (dtype == TSDPA_F16) {
        switch (D) {
            case 64: err = tsdpa::launch_bwd_f16_d64(a); break;
            case 96: err = tsdpa::launch_bwd_f16_d96(a); break;
            case 128: err = tsdpa::launch_bwd_f16_d128(a); break;
            default: err = tsdpa::launch_bwd_f16_d160(a); break;
        }
    } else {
        switch (D) {
            case 64: err = tsdpa::launch_bwd_bf16_d64(a); break;
            case 96: err = tsdpa::launch_bwd_bf16_d96(a); break;
            case 128: err = tsdpa::launch_bwd_bf16_d128(a); break;
            default: err = tsdpa::launch_bwd_bf16_d160(a); break;
        }
    }
    return err == 0 ? TSDPA_OK : TSDPA_ERR_LAUNCH;
}

int tiled_sdpa_fwd(const void *q, const void *k, const void *v, void *o, float *lse,
                   int B, int H, int S, int D, float scale, int dtype, void *stream)
{
    return tiled_sdpa_fwd_ex(q, k, v, o, lse, B, H, S, D, scale, dtype, stream, 0, 0, 0u);
}

}  // extern "C"
