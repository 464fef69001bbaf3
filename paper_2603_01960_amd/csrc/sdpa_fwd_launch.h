// Host-side launch plumbing shared by the per-(dtype, D) instantiation files and the C-ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsdpa {

struct LaunchArgs {
    const void *q, *k, *v;
    void *o;
    float *lse;
    int BH, S;
    float c;          // |scale| * log2(e)
    float tau;        // lazy-rescale threshold in log2 units (0 = raise the reference on every new maximum)
    uint32_t qsign;   // 0x80008000 when scale < 0 (sign folded into Q), else 0
    int linear_grid;
    int causal;       // causal mask (Section 4.1.3): key j contributes to query i only if j <= i + Skv - S
    int kv;           // 0: S queries against the same S keys.  1: the general kernel (Skv keys, split key range)
    int Skv;          // key/value rows per head (kv = 1)
    int splits;       // workgroups per (head, query tile) along the key axis (kv = 1); > 1 writes partials to ws
    float *ws;        // split workspace: float [BH][splits][S][D] then [BH][splits][S][2]
    const int *kv_lens;   // kv = 1: NULL, or valid key rows per batch entry (device, int32 [B]); Skv is then the capacity
    int heads_per_batch;  // kv = 1: key/value heads per batch entry (head / heads_per_batch indexes kv_lens)
    const int *block_table; // kv = 1: NULL, or pages of a paged cache (device, int32 [B][max_blocks]); k, v are then [pages][heads_per_batch][1 << block_shift][D]
    int max_blocks, block_shift;
    int tile_rot;      // kv = 1, dense cache: 1 = every workgroup starts its sweep over the unmasked tiles at a tile of its own
    int batches;       // kv = 1: batch entries (BH / heads_per_batch)
    int halves;        // kv = 1, at most 32 rows: 1 = each weight goes into the output product as two 16-bit halves (pick_halves)
    unsigned long long ticket; // decoding kernel, splits > 1: a number of this call alone (never 0) if it combines the runs itself, else 0
    int streams;       // kv = 0: streams of K/V tiles per workgroup (0 or 1: the plain form)
    int rows_per_head; // kv = 1: query positions per query head; S / rows_per_head query heads are folded into the S rows
    hipStream_t stream;
};

// Wavefronts per workgroup of the decoding kernel.  Up to one workgroup per CU eight (two workgroups of four per CU hold as
// many beyond that): level on large caches, 256 heads of 2048 keys 52.5 -> 48.4 us.  With less than a tile of 32 keys per
// wavefront to do, four.
inline int decode_waves(int heads, int splits, int Skv)
{
    return (long long)heads * splits <= 256 && Skv / splits >= 256 ? 8 : 4;
}

// Chunks in which causal_tile (sdpa_fwd_kernel.h) takes the heads: heads per XCD and chunk (0: the plain order, head
// after head), and heads of the first chunk.  `tiles` workgroups per head, `stream_bytes` of streamed operands per head.
// From timings of every chunk size on 24 shapes (us, plain order -> this rule):
//   * up to one workgroup per CU all of them start at once and the order is moot: the plain one, whose index arithmetic
//     is shorter (0.3-0.5 us of 13-19 at nine heads of S = 1024);
//   * up to two per CU: all heads in one chunk, so that a CU holds a long tile and a short one (BF16, 64 heads of
//     S = 1024 at D = 128: 29.8 -> 27.4; nine heads of S = 4096: 78.3 -> 64.2);
//   * beyond, eight heads per XCD, as long as the chunk streams at most 8 MiB per XCD, twice its L2 (64 heads of
//     S = 2048, D = 96: 71.5 -> 60, D = 128: 89 -> 72; S = 4096, D = 128: 274 -> 248 with four heads; S = 8192: 962 ->
//     930 with two and 982 with eight).  Up to three per CU sixteen heads where the caller found it so (`wide`).
struct CausalChunks { int first, heads; };
inline CausalChunks causal_chunks(int heads, int tiles, long long stream_bytes, bool wide)
{
    const long long n = (long long)heads * tiles;
    int hg = (heads + 7) / 8;
    if (n <= 256 || tiles == 1) return CausalChunks{heads, 0};
    if (n > 512) {
        const long long fit = stream_bytes > 0 ? (8ll << 20) / stream_bytes : 8;
        const int most = wide && n <= 768 ? 16 : fit > 8 ? 8 : fit < 1 ? 1 : (int)fit;
        if (hg > most) hg = most;
    }
    return CausalChunks{heads - (heads - 1) / (8 * hg) * (8 * hg), hg};
}

// Division by a number known at launch, for n < 2^31: n * mul >> (31 + shift) with mul = ceil(2^(31 + shift) / d) and shift =
// ceil(log2 d).  (mul * d exceeds 2^(31 + shift) by less than d <= 2^shift, so the quotient is n / d plus less than 2^-shift <=
// 1 / d.)  In the kernels' prologues: a division by a variable is a serial chain of some thirty instructions.  With these
// divisions and the arguments read at once the plain forward forms are back at what they took before the causal order came (us,
// before it / with variable divisions / now, no mask: 200 heads of S = 768 D = 128 73.2 / 74.1 / 72.9, 1586 of S = 131 D = 160
// 72.4 / 73.6 / 72.2, 937 of S = 178 D = 96 28.9 / 29.4 / 28.8; the backward passes of 8 heads of S = 1024 gain 0.5-1 us).
struct Divisor { uint32_t mul, shift; };
inline Divisor divisor(uint32_t d)
{
    const uint32_t shift = d <= 1 ? 0 : 32 - __builtin_clz(d - 1);
    return Divisor{(uint32_t)(((1ull << (31 + shift)) + d - 1) / d), shift};
}

// What a kernel needs to find its workgroup's head and tile: `tiles` per head, and the chunks of the causal order (heads = 0
// where it is not taken; the divisors after it are then not looked at).
struct TileOrder {
    Divisor by_tiles;
    int first, heads;          // CausalChunks
    Divisor by_chunk, by_first, by_full;    // heads * tiles, first, 8 * heads
};
inline TileOrder tile_order(int heads, int tiles, bool causal, long long stream_bytes, bool wide = false)
{
    TileOrder order{divisor((uint32_t)tiles), heads, 0, {}, {}, {}};
    if (!causal) return order;
    const CausalChunks c = causal_chunks(heads, tiles, stream_bytes, wide);
    if (c.heads == 0) return order;
    order.first = c.first;
    order.heads = c.heads;
    order.by_chunk = divisor((uint32_t)(c.heads * tiles));
    order.by_first = divisor((uint32_t)c.first);
    order.by_full = divisor((uint32_t)(8 * c.heads));
    return order;
}

// Rows of slack after the B*H*S entries of each backward statistics array: the keys-resident pass
// reads them 4 rows at a time up to a tile past the last row of the last head.
constexpr int kBwdStatPad = 128;

struct BwdLaunchArgs {
    const void *q, *k, *v, *o, *dout;
    const float *lse;        // natural-log LSE of the forward pass, [BH, S]
    void *dq, *dk, *dv;
    float *stats;            // workspace, two halves of [BH*S + slack]: Delta, then LSE in log2 units
    unsigned stat_bytes;     // bytes of one half
    void *chain;             // workspace of the five products (chain_layout in sdpa_bwd_pick.h)
    int BH, S;               // query heads (B * H) and rows per head
    int group;               // query heads per key/value head (1: k, v, dk, dv have BH heads too; else BH / group)
    float c;                 // |scale| * log2(e)
    float scale;             // signed scale: factor of dQ and dK
    uint32_t rsign;          // 0x80008000 when scale < 0 (sign folded into the resident Q or K), else 0
    int causal;
    hipStream_t stream;
};

// Each returns a hipError_t cast to int (0 = success); tile_m in {64,128}, tile_n in {32,64,128}
// (tile_n in {32,64} when a.kv is set).
int launch_f16_d64(int tile_m, int tile_n, const LaunchArgs &a);
int launch_f16_d96(int tile_m, int tile_n, const LaunchArgs &a);
int launch_f16_d128(int tile_m, int tile_n, const LaunchArgs &a);
int launch_f16_d160(int tile_m, int tile_n, const LaunchArgs &a);
int launch_bf16_d64(int tile_m, int tile_n, const LaunchArgs &a);
int launch_bf16_d96(int tile_m, int tile_n, const LaunchArgs &a);
int launch_bf16_d128(int tile_m, int tile_n, const LaunchArgs &a);
int launch_bf16_d160(int tile_m, int tile_n, const LaunchArgs &a);

// Decoding steps (a.S <= 32 query rows per key/value head; sdpa_decode_kernel.h).
int launch_decode_f16(int D, const LaunchArgs &a);
int launch_decode_bf16(int D, const LaunchArgs &a);

// Backward pass: dQ (queries resident) and dK + dV (keys resident) in one grid after the row statistics, or one after the other with
// the statistics on the way, or whole heads in one launch (sdpa_bwd_pick.h).
int launch_bwd_f16_d64(const BwdLaunchArgs &a);
int launch_bwd_f16_d96(const BwdLaunchArgs &a);
int launch_bwd_f16_d128(const BwdLaunchArgs &a);
int launch_bwd_f16_d160(const BwdLaunchArgs &a);
int launch_bwd_bf16_d64(const BwdLaunchArgs &a);
int launch_bwd_bf16_d96(const BwdLaunchArgs &a);
int launch_bwd_bf16_d128(const BwdLaunchArgs &a);
int launch_bwd_bf16_d160(const BwdLaunchArgs &a);

// ... in five products (per_claim: key/value heads that an XCD takes at a time)
int launch_bwd_chain_f16_d64(const BwdLaunchArgs &a, int per_claim);
int launch_bwd_chain_f16_d96(const BwdLaunchArgs &a, int per_claim);
int launch_bwd_chain_f16_d128(const BwdLaunchArgs &a, int per_claim);
int launch_bwd_chain_bf16_d64(const BwdLaunchArgs &a, int per_claim);
int launch_bwd_chain_bf16_d96(const BwdLaunchArgs &a, int per_claim);
int launch_bwd_chain_bf16_d128(const BwdLaunchArgs &a, int per_claim);

}  // namespace tsdpa
