// Backward pass of tiled SDPA for gfx950 (MI355X).  The paper leaves it as future work (Section 7);
// what is computed is the derivative of its Eq. 1 (Section 3.1), with P recomputed tile by tile from
// the forward pass's log-sum-exp instead of being stored, in the spirit of Section 4.1.2:
//
//     P_ij  = exp(scale * <q_i, k_j> - LSE_i)          (0 for masked keys)
//     dV_j  = sum_i P_ij dO_i
//     dP_ij = <dO_i, v_j>
//     dS_ij = P_ij (dP_ij - Delta_i),   Delta_i = <dO_i, O_i>   (= sum_j P_ij dP_ij)
//     dQ_i  = scale * sum_j dS_ij k_j,  dK_j = scale * sum_i dS_ij q_i
//
// Two passes over the S x S score plane, instances of ONE template, so that no sum crosses workgroups (no atomics,
// deterministic results):
//   * BWD_DQ: a workgroup owns 32*NW query rows (Q and dO rows resident), streams K and V tiles; it also computes the
//     statistics of its rows (-Delta, LSE in log2 units) for the passes after it;
//   * BWD_DKV: a workgroup owns 32*NW key rows (K and V rows resident), streams Q and dO tiles; two accumulators (D = 160,
//     where they do not fit one wavefront: sdpa_bwd_pair_kernel.h).
// With R the resident and T the streamed rows, a pass computes, per streamed tile,
//     acc[t][r]  = <T1_t, R1_r>  (scores)        acc2[t][r] = <T2_t, R2_r>  (dP)
//     out^T[d][r] += sum_t T1[t][d] dS[t][r]     (dQ^T or dK^T)
//     out^T[d][r] += sum_t T2[t][d] P[t][r]      (dV^T)
// (T1, T2, R1, R2) = (K, V, Q, dO) or (Q, dO, K, V).  The scores and dP are thus computed twice (7 S x S x D products
// against the 5 of the formulas): the price of summing nothing across workgroups.
// What bounds it: the matrix pipe and the clock under its power limit; what decides is that every pass fits 256
// registers per lane (two wavefronts per SIMD, of which one does matrix work while the other is in its exponentials).
// That took three things: the step exists ONCE in the loop (with copies of it for the two LDS slots and for masked
// tiles, the accumulators of every copy met at joins, and the fused pass at D = 128 spilled 279 registers instead of
// none); V stays in the LDS at D = 128; and an LDS layout that needs few pointers (BwdGeom).  Before, D = 96 and 128 ran
// dK and dV as two passes (8 products), D = 160 ran one wavefront per SIMD, and the statistics had kernels of their own.
// BF16, 64 heads, S = 8192, ms per call before / now: D = 64 3.73 / 3.63, D = 96 6.27 / 5.08, D = 128 7.88 / 6.38,
// D = 160 12.9 / 10.7; S = 2048 causal, us: D = 64 205 / 145, D = 96 335 / 198, D = 128 428 / 253, D = 160 644 / 425.
// Since then the dP accumulators start from -Delta and the operand kept in the LDS lies in operand order: 64 heads, S =
// 4096, us, D = 64 931 / 907, D = 128 1628 / 1612.
// The MFMA formulation is the forward kernel's:
// transposed accumulators (a lane owns one resident row), P and dS handed to the second product
// straight from the accumulator registers as B-operands, the streamed tile read row-wise for the
// first product and through the transposing LDS read for the second.
#pragma once
#include "sdpa_fwd_kernel.h"
#include "sdpa_fwd_launch.h"

namespace tsdpa {

// LDS geometry of a block of rows of D 16-bit values, filled by direct-to-LDS loads of 1 KiB ("units": 64 lanes x 16 B)
// and read both row-wise (16 lanes fetch one chunk index of 16 consecutive rows) and through the transposing read (32
// lanes fetch one 64-byte block, 4 chunks, of 4 consecutive rows); neither has bank conflicts (64 banks: 256 bytes).
// Where the layout allows it the swizzle touches few bits of the chunk index, so that few per-lane pointers are needed
// and the rest of an address is an immediate: registers are what bounds the passes above D = 64.
//   D = 64:  rows of 128 bytes; chunk c of row r at c ^ (bit 1 of r in bit 2, bits 3:2 of r in bits 1:0).
//   D = 128: rows of 256 bytes, four to a unit, units 16 bytes further apart than they are long.  c ^ ((r & 3) << 2)
//            puts the four rows of a unit on different 64-byte blocks (the transposing read), the 16 bytes move the next
//            unit one 16-byte slot on (16 consecutive rows: 16 slots).  Four row pointers and four transposing ones
//            instead of 8 + 8.
//   D = 96, 160: rows of 192 or 320 bytes start 3 or 5 quarters of the banks after one another, so that four rows put
//            the same block on different quarters by themselves; c ^ (bits 3:2 of r).  Two row pointers, two
//            transposing ones.  A tile is as long as in memory (padded to 256 or 512 bytes per row, D = 160 had one
//            workgroup per CU and 37.5 % of its load lanes fetched nothing).
template <int D> struct BwdGeom {
    static_assert(D == 64 || D == 96 || D == 128 || D == 160, "head dims of the paper's grid");
    static constexpr int GROW = D * 2;              // bytes per row in global memory, and per row in the LDS
    static constexpr int CPR = D / 8;               // 16-byte chunks per row
    static constexpr int UNIT = D == 128 ? 1040 : 1024;     // distance between units in the LDS
    static constexpr int DG = D <= 64 ? 64 : (D <= 128 ? 128 : 256);
    static constexpr int OROW = DG * 2;             // bytes per row of the output transpose after the loop
    static constexpr int bytes(int rows) { return rows * CPR / 64 * UNIT; }         // a block of rows (a multiple of 16)
    static __host__ __device__ constexpr int swz(int r) {
        return D == 64 ? ((((r >> 1) & 1) << 2) | ((r >> 2) & 3)) : D == 128 ? (r & 3) << 2 : (r >> 2) & 3;
    }
    // byte offset of chunk c of row r
    static __host__ __device__ constexpr int at(int r, int c) {
        return D == 128 ? (r >> 2) * UNIT + (r & 3) * GROW + ((c ^ swz(r)) << 4) : r * GROW + ((c ^ swz(r)) << 4);
    }
    // per-lane pointers: row-wise ones serve chunk groups kk with the same key, transposing ones blocks db likewise
    static constexpr int NRP = D == 64 || D == 128 ? 4 : 2, NTP = D == 64 ? 2 : D == 128 ? 4 : 1;
    static constexpr int rp(int kk) { return D == 64 ? kk : D == 128 ? kk >> 1 : kk & 1; }
    static constexpr int rp_kk(int i) { return D == 128 ? 2 * i : i; }              // the kk that pointer i is computed for
    static constexpr int rp_imm(int kk) { return D == 64 ? 0 : D == 128 ? (kk & 1) * 32 : (kk >> 1) * 64; }
    static constexpr int tp(int db) { return D == 64 || D == 128 ? db : 0; }
    static constexpr int tp_imm(int db) { return D == 64 || D == 128 ? 0 : db * 64; }
    // load instructions: the swizzle repeats every LCP units, the lane's offset with it
    static constexpr int LCP = D == 64 ? 2 : D == 128 ? 1 : CPR / 4;
};

// BWD_DKV: scores and P computed once for dK and dV; two output accumulators, which fit 256 registers per lane (two
// wavefronts per SIMD) up to D = 128.
enum { BWD_DQ = 0, BWD_DKV = 1 };

// Delta_i of query rows that see at most this many keys (the first rows under the causal mask; every row of a sequence
// of up to so many) is taken from its definition  Delta_i = sum_j P_ij dP_ij  in FP32.  <dO_i, O_i> equals it only in
// exact arithmetic: O arrives rounded to 16 bits, and the rounding error of the D-term sum goes into dS_ij = P_ij (dP_ij
// - Delta_i) scaled by P_ij, which is of order 1 exactly on such rows (on a row of n comparable keys it is of order 1/n).
constexpr int kBwdShortRow = 64;

// HBM -> LDS loads in assembly, 16 or 4 bytes per lane, for kernels that count their loads themselves: left to the compiler, the first
// transposing read waits for all of them.
//   * That m0 is written has to be said: the compiler keeps the m0 of its own loads to the LDS from one to the next.  (Its warning that m0
//     is reserved is about registers that it would restore, which nothing here relies on.)
//   * A memory instruction must not follow a vector instruction that writes one of its scalar registers by less than five wait states, and
//     the compiler, which reads spilled ones back with v_readlane, does not look into assembly: the instructions before the load make five.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t dst, int voff, int soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" : : "s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "m0");
}
__device__ __forceinline__ void lds_load4(__amdgpu_buffer_rsrc_t rsrc, uint32_t dst, int voff, int soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, %3 offen lds" : : "s"(dst), "v"(voff), "s"(rsrc), "s"(soff) : "m0");
}
// ... past the L2
__device__ __forceinline__ void lds_load4_agent(__amdgpu_buffer_rsrc_t rsrc, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dword %1, %2, 0 offen sc1 lds" : : "s"(dst), "v"(0), "s"(rsrc) : "m0");
}
#pragma clang diagnostic pop

// LDS of one stream of tiles: two slots per tensor and, in the keys-resident passes, of the row statistics.
template <int D, int TS, int MODE> constexpr int bwd_stream_bytes() { return 4 * BwdGeom<D>::bytes(TS) + (MODE != BWD_DQ ? 2 * 2 * TS * 4 : 0); }

// GRP: grouped heads, G query heads reading one key/value head (query head h the head h / G).  The
// dQ pass then streams the K and V of its query head's group; the keys-resident passes run one
// workgroup per (key/value head, key tile) and stream the Q and dO tiles of the G query heads of the
// group one head after the other into the same accumulators, which is the sum over the group that dK
// and dV are.  GRP = false is G = 1 with that loop gone.
// R2LDS: the second resident operand (dO in the dQ pass, V otherwise) stays in the LDS instead of D/4 registers per
// lane; each of its MFMAs then reads two operands from there.
// NS: streams.  NS groups of NW wavefronts share the resident rows and take every NS-th tile of the chain each (over the
// heads of a group), in LDS slots of their own; at the end their sums are added in the order of the streams.  For passes
// of few workgroups, whose wavefronts would wait through the whole chain alone (the choice and its figures: pick_bwd_form).
// Launched by itself the dQ pass runs first: it has the query rows, so it computes their statistics (Delta_i, and LSE_i in log2
// units) in its prologue and leaves them in `stats` for the other.  HAVE_STATS: they are there already (sdpa_bwd_joint_kernel.h).
template <typename T, int D, int NW, int NS, int TS, int MODE, bool GRP, bool R2LDS, bool HAVE_STATS>
__device__ __forceinline__ void
bwd_pass(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
         const T *__restrict__ dout, const T *__restrict__ o, const float *__restrict__ lse,
         float *__restrict__ stats,   // -Delta [B*H*S + slack], then LSE in log2 units likewise
         T *__restrict__ out,   // dQ or dK
         T *__restrict__ out2,  // dV of the keys-resident pass, else unused
         int S, int nR, int N, float c, float scale, uint32_t rsign, int causal, unsigned stat_bytes,
         int group, const TileOrder &order, const int block)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    using vec4 = typename E::vec4;
    using G = BwdGeom<D>;
    constexpr bool KEYS_RES = MODE != BWD_DQ;
    constexpr bool FUSED = MODE == BWD_DKV;       // P kept next to dS, second accumulator for dV
    static_assert(!KEYS_RES || D != 160, "the keys-resident pass of D = 160 is sdpa_bwd_pair_kernel");
    constexpr int RM = NW * 32;                   // resident rows per workgroup
    constexpr int U = TS * G::CPR / 64;           // units per streamed tile of one tensor
    constexpr int L = 2 * U / NW;                 // load instructions per wavefront per tile pair (T1, T2)
    constexpr bool EVEN = U % NW == 0;            // a load is a T1 or a T2 load for all wavefronts alike
    constexpr int NLD = U / NW;                   // (then: loads per tensor)
    static_assert(TS * G::CPR % 64 == 0 && L >= 1 && (2 * U) % NW == 0, "tile pair does not divide over the workgroup");
    constexpr int NB = TS / 32, KK = D / 16, DB = D / 32;
    constexpr int TILE = G::bytes(TS), STATS = 2 * TS * 4;
    constexpr int STREAM = bwd_stream_bytes<D, TS, MODE>();       // LDS of one stream: two slots per tensor, and of the statistics
    constexpr int ROW16 = G::bytes(16);           // LDS distance of rows 16 apart (the swizzles repeat every 16 rows)

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int stream = NS > 1 ? wave_id / NW : 0, wave = NS > 1 ? wave_id % NW : wave_id;
    const lds_ptr slots = lds + stream * STREAM;
    const int g = lane >> 5, l32 = lane & 31;

    // (the arguments of the prologue all at once, as in the forward kernel)
    asm volatile("" : : "s"(q), "s"(k), "s"(v), "s"(dout), "s"(order.by_tiles.mul), "s"(order.by_tiles.shift), "s"(order.first),
                 "s"(order.heads), "s"(order.by_chunk.mul), "s"(order.by_chunk.shift), "s"(order.by_first.mul), "s"(order.by_first.shift),
                 "s"(order.by_full.mul), "s"(order.by_full.shift), "s"(S), "s"(causal));
    const int Gn = GRP ? group : 1;              // query heads per key/value head
    int head, rt;                                 // head of the resident side (a query head in the dQ pass, else a key/value head) and tile
    if (causal && order.heads > 0) {
        // query tiles get longer with their index, key tiles shorter: the long ones of all heads first (causal_tile)
        const CausalTile ct = causal_tile(block, nR, order, NS == 1 && D >= 128 && !HAVE_STATS ? N : 0);
        head = ct.head;
        rt = KEYS_RES ? ct.level : nR - 1 - ct.level;
    } else {
        const int wg = remap_workgroup(block, N, false);
        head = divide(wg, order.by_tiles);
        rt = (causal && !KEYS_RES) ? nR - 1 - (wg - head * nR) : wg - head * nR;
    }
    const size_t head_off = (size_t)head * (size_t)S * D;
    const T *r1 = (KEYS_RES ? k : q) + head_off;       // resident operands
    const T *r2 = (KEYS_RES ? v : dout) + head_off;
    // streamed operands: the key/value head of this query head, or the first query head of this key/value head
    const size_t shead0 = KEYS_RES ? (size_t)head * Gn : (size_t)(head / Gn);
    const T *t1 = (KEYS_RES ? q : k) + shead0 * (size_t)S * D;
    const T *t2 = (KEYS_RES ? dout : v) + shead0 * (size_t)S * D;

    constexpr int T2BASE = 2 * TILE;              // T1 slot s at s*TILE, T2 slot s at T2BASE + s*TILE
    constexpr int STBASE = 4 * TILE;              // statistics slot s at STBASE + s*STATS (keys-resident passes)
    constexpr int RBASE = NS * STREAM;            // second resident operand, 32 rows per wavefront of a stream

    // ---- resident rows as MFMA B-operands: lane holds R[row l32][kk*16 + g*8 .. +7]; the sign of a
    // negative scale is folded into R1 so that c = |scale| * log2(e) applies to the scores
    const int r0 = rt * RM;
    const int rrow = r0 + wave * 32 + l32;
    const int rrow_c = rrow < S ? rrow : S - 1;
    vec8 rf1[KK], rf2[R2LDS ? 1 : KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        u32x4 raw = *(const u32x4 *)(r1 + (size_t)rrow_c * D + kk * 16 + g * 8);
        raw ^= rsign;
        rf1[kk] = __builtin_bit_cast(vec8, raw);
        if constexpr (!R2LDS) rf2[kk] = *(const vec8 *)(r2 + (size_t)rrow_c * D + kk * 16 + g * 8);
    }
    if constexpr (R2LDS) {
        // this wavefront's 32 rows (rows >= S: zeros) in the order of the operand: k-step kk is one unit, lane after lane,
        // so that one pointer and immediates serve all reads.  Waited for with the first tile.
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)r2, (short)0, S * G::GROW, 0x00020000);
        const int row0 = (r0 + wave * 32) * G::GROW;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            if (NS == 1 || kk % NS == stream)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(lds + RBASE + (wave * KK + kk) * 1024), 16,
                                                         l32 * G::GROW + g * 16, row0 + kk * 32, 0, 0);
    }

    // ---- range of streamed tiles, and the streamed rows [tlo, thi] that pair with this lane's row
    const int nT = (S + TS - 1) / TS;
    const int last_row = (r0 + RM < S ? r0 + RM : S) - 1;
    int j0 = 0, j1 = nT;
    int tlo = 0, thi = S - 1;
    if (causal) {
        if (KEYS_RES) { j0 = r0 / TS; tlo = rrow; }                       // queries at or after the key
        else { j1 = last_row / TS + 1; thi = rrow < S ? rrow : S - 1; }   // keys up to the query
    }

    // Per-row statistics of the query side, LSE (log2 units) and Delta: scalars of this lane's row (dQ pass), or
    // streamed into the LDS with each tile.  The descriptor spans both arrays, slack included; rows >= S of a head pick
    // up the next head's values or whatever the slack holds, and are masked.
    float lse_r = 0.f, delta_r = 0.f;
    if constexpr (!KEYS_RES && HAVE_STATS) {
        delta_r = -stats[(size_t)head * S + rrow_c];
        lse_r = *(const float *)((const char *)stats + stat_bytes + ((size_t)head * S + rrow_c) * 4);
    } else if constexpr (!KEYS_RES) {
        lse_r = lse[(size_t)head * S + rrow_c] * 1.44269504088896340736f;
        // Delta = <dO, O>: the lane's half of the row, then the partner's (rows that see few keys: see below)
        const T *orow = o + head_off + (size_t)rrow_c * D + g * 8, *drow = r2 + (size_t)rrow_c * D + g * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const vec8 x = *(const vec8 *)(orow + kk * 16);
            const vec8 y = R2LDS ? *(const vec8 *)(drow + kk * 16) : rf2[R2LDS ? 0 : kk];
#pragma unroll
            for (int e = 0; e < 8; ++e) delta_r += (float)x[e] * (float)y[e];
        }
        delta_r = pair_sum(delta_r);
    }
    const auto stat_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)stats, (short)0, (int)(2 * stat_bytes), 0x00020000);
    constexpr int NST = 2 * TS / 64;              // 4-byte direct-to-LDS loads (wavefront 0) per tile: LSE rows, then Delta rows
    int stat_goff[NST];
#pragma unroll
    for (int it = 0; it < NST; ++it) {
        const int e = it * 64 + lane;             // element of the tile's statistics block
        stat_goff[it] = (e / TS == 0 ? (int)stat_bytes : 0) + ((int)shead0 * S + e % TS) * 4;
    }

    // ---- streamed tiles HBM -> LDS, as in the forward kernel: a descriptor per tensor covers this head's S rows (rows
    // >= S read as zeros); unit u of a tile fills LDS bytes u*UNIT ... with the global chunks the swizzle maps there.
    // The units of a tile pair, T1's then T2's, are dealt round-robin over the wavefronts; the lanes' offsets repeat
    // every LCP units, so EVEN needs one register per distinct offset; otherwise each load has its own.
    auto t1_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)t1, (short)0, S * G::GROW, 0x00020000);
    auto t2_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)t2, (short)0, S * G::GROW, 0x00020000);
    constexpr int NP = G::LCP % 2 == 0 ? (NW % 2 == 0 ? G::LCP / 2 : G::LCP) : G::LCP;     // (LCP is 1, 2, 3 or 5; NW 2, 4 or 8)
    constexpr int NCG = EVEN ? (NLD < NP ? NLD : NP) : L;
    int goff[NCG];
#pragma unroll
    for (int i = 0; i < NCG; ++i) {
        const int u = i * NW + wave;
        const int p = (EVEN || u < U ? u : u - U) * 64 + lane;
        const int r = p / G::CPR, cp = p % G::CPR;
        goff[i] = r * G::GROW + ((cp ^ G::swz(r)) << 4);
    }
    auto load_unit = [&](decltype(t1_rsrc) rsrc, lds_ptr dst, int unit, int voff, int soff) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(dst + unit * G::UNIT), 16, voff, soff, 0, 0);
    };
    // load instruction i (of L) of tile j (of the head the descriptors stand at) into slot `dst`
    auto load_part = [&](int j, bool valid, lds_ptr dst, int i) __attribute__((always_inline)) {
        const int soff = (valid ? j : nT) * TS * G::GROW;    // no such tile: outside the descriptor, zeros
        const int u = i * NW + wave;
        if constexpr (EVEN) {
            const int it = i % NLD;
            load_unit(i < NLD ? t1_rsrc : t2_rsrc, i < NLD ? dst : dst + T2BASE, it * NW + wave, goff[it % NCG],
                      soff + (it / NCG) * (NCG * NW * 1024));
        } else if ((i + 1) * NW <= U) {
            load_unit(t1_rsrc, dst, u, goff[i], soff);
        } else if (i * NW >= U) {
            load_unit(t2_rsrc, dst + T2BASE, u - U, goff[i], soff);
        } else {
            const bool first = u < U;             // T1 for some wavefronts, T2 for the others: scalar selects
            load_unit(first ? t1_rsrc : t2_rsrc, first ? dst : dst + T2BASE, first ? u : u - U, goff[i], soff);
        }
    };
    auto load_tile = [&](int j, bool valid, lds_ptr dst) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < L; ++i) load_part(j, valid, dst, i);
    };
    // statistics of the rows from row0 on, counted over the heads of the group
    auto load_stats = [&](int row0, int slot) __attribute__((always_inline)) {
        if constexpr (KEYS_RES) {
            if (wave == 0) {
#pragma unroll
                for (int it = 0; it < NST; ++it)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(stat_rsrc, (TSDPA_LDS void *)(slots + STBASE + slot * STATS + it * 256), 4,
                                                             stat_goff[it], row0 * 4, 0, 0);
            }
        }
    };

    f32x16 oacc[DB], oacc2[FUSED ? DB : 1];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            oacc[db][i] = 0.f;
            if constexpr (FUSED) oacc2[db][i] = 0.f;
        }

    // ---- per-lane LDS read pointers (tile slot, nb, ks enter as immediate offsets)
    // row-wise: row l32 (+32*nb), chunk 2*kk + g
    lds_ptr row_ptr[G::NRP];
#pragma unroll
    for (int i = 0; i < G::NRP; ++i) {
        row_ptr[i] = slots + G::at(l32, 2 * G::rp_kk(i) + g);
        TSDPA_OPAQUE(row_ptr[i]);
    }
    const lds_ptr res_ptr = lds + RBASE + wave * KK * 1024 + lane * 16;
    // transposing: row g*4 + (lane%16)/4 (+ multiples of 8), bytes db*64 + ((lane/16)%2)*32 + (lane%4)*8 of the row
    const int t_row = g * 4 + ((lane & 15) >> 2), t_chunk = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    lds_ptr tr_lo[G::NTP], tr_hi[D == 128 ? 1 : G::NTP];       // rows t_row (+16k) and t_row + 8 (+16k)
#pragma unroll
    for (int i = 0; i < G::NTP; ++i) {
        tr_lo[i] = slots + G::at(t_row, i * 4 + t_chunk) + (lane & 1) * 8;
        TSDPA_OPAQUE(tr_lo[i]);
        if constexpr (D != 128) {                 // (at D = 128 eight rows on is two units on, swizzled alike)
            tr_hi[i] = slots + G::at(t_row + 8, i * 4 + t_chunk) + (lane & 1) * 8;
            TSDPA_OPAQUE(tr_hi[i]);
        }
    }

    lds_ptr st_ptr = slots + STBASE + g * 16;       // statistics of rows g*4 ... g*4 + 3 (+8k) of the current tile

    // -Delta of the lane's row as an accumulator to start from (not at D = 96, whose dQ pass has no 16 registers left)
    constexpr bool DELTA16 = MODE == BWD_DQ && D != 96;
    f32x16 minus_delta;
    if constexpr (DELTA16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) minus_delta[i] = 0.f;
    }
    // acc[i] = <T_row, R_col>, row = nb*32 + (i/4)*8 + g*4 + i%4 of the tile, col = this lane's row.  The second product
    // starts from -Delta of the query row where that costs nothing: one vector instruction per element less in the weights.
    auto products = [&](int slot, int nb, bool second, f32x16 &acc, auto &&after_mfma) __attribute__((always_inline)) {
        if (second && KEYS_RES) {
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4 md = *(TSDPA_LDS f32x4 *)(st_ptr + (TS + nb * 32 + r4 * 8) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[r4 * 4 + e] = md[e];
            }
        } else if (second && DELTA16) {
            acc = minus_delta;
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = 0.f;
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const u32x4 raw = lds_read128(row_ptr[G::rp(kk)] + slot + nb * 2 * ROW16 + G::rp_imm(kk));
            vec8 b;
            if (!second) b = rf1[kk];
            else if (R2LDS) b = __builtin_bit_cast(vec8, lds_read128(res_ptr + kk * 1024));
            else b = rf2[R2LDS ? 0 : kk];
            acc = E::mfma(__builtin_bit_cast(vec8, raw), b, acc);
            after_mfma(kk);
        }
    };
    auto nothing = [](int) __attribute__((always_inline)) {};
    // out^T += T^T X, X taken from accumulator layout as B-operands (k-slots 0..3 / 4..7 of a lane <->
    // tile rows base+g*4+0..3 / base+8+g*4+0..3, mirrored on the A side by the two transposing reads)
    auto accumulate = [&](int slot, const vec8 (&xb)[NB][2], f32x16 (&acc)[DB]) __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const int off = slot + (nb * 2 + ks) * ROW16 + G::tp_imm(db);
                    const i16x4 lo = lds_read_tr16(tr_lo[G::tp(db)] + off);
                    const i16x4 hi = D == 128 ? lds_read_tr16(tr_lo[G::tp(db)] + off + 2 * G::UNIT)
                                              : lds_read_tr16(tr_hi[D == 128 ? 0 : G::tp(db)] + off);
                    const i16x8 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    acc[db] = E::mfma(__builtin_bit_cast(vec8, a), xb[nb][ks], acc[db]);
                }
    };

    // P (and dS) of one 32-row block, rounded to 16 bits as B-operands of the second products.  The 16 streamed rows this
    // lane meets in the block come in 4 runs of 4 consecutive rows; in the keys-resident passes their statistics are read
    // from the LDS run by run (scheduling barriers keep the compiler from fetching all of them ahead, 32 registers)
    vec8 xb[NB][2], pb[FUSED ? NB : 1][2];
    auto weights = [&](int nb, int trow0, const f32x16 &sacc, const f32x16 &dpacc, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            f32x4 st_lse;
            if constexpr (KEYS_RES) st_lse = *(TSDPA_LDS f32x4 *)(st_ptr + (nb * 32 + r4 * 8) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = r4 * 4 + e;
                const float l2 = KEYS_RES ? st_lse[e] : lse_r;
                const int trow = trow0 + nb * 32 + r4 * 8 + e;
                const bool masked = MASK && (trow < tlo || trow > thi);
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -l2));        // P
                if constexpr (FUSED) pb[nb][i >> 3][i & 7] = (T)(masked ? 0.f : p);
                float x = p;
                x *= KEYS_RES || DELTA16 ? dpacc[i] : dpacc[i] - delta_r;     // dS
                xb[nb][i >> 3][i & 7] = (T)(masked ? 0.f : x);
            }
            if constexpr (FUSED) __builtin_amdgcn_sched_barrier(0);
        }
    };
    // One streamed tile, its successor's loads issued early: they land while this one is computed.  One loop body serves
    // both slots (the pointers move by the slot distance and back) and both kinds of tile (only the weights branch), so
    // that the accumulators never meet at a join of two copies of the step.
    // (a raised priority during the MFMA chains, as in the forward kernel, gains 2-4 % at D = 160; at the other head dims
    // it gains 1-4 % on large problems and loses as much where a CU holds one workgroup)
    constexpr bool PRIO = D == 160;
    int shift = TILE;                             // from the current slot to the other
    auto other_slot = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < G::NRP; ++i) row_ptr[i] += shift;
#pragma unroll
        for (int i = 0; i < G::NTP; ++i) {
            tr_lo[i] += shift;
            if constexpr (D != 128) tr_hi[i] += shift;
        }
        if constexpr (KEYS_RES) st_ptr += shift > 0 ? STATS : -STATS;
        shift = -shift;
    };
    auto tile = [&](int j, bool mask, int next_j, int next_row, bool next_valid) __attribute__((always_inline)) {
        load_stats(next_row, shift > 0 ? 1 : 0);
        // The loads go out one at a time behind the MFMAs of the first products: back to back they hold the wavefront at
        // the issue stage while the CU's address unit works through them (S = 1024 of nine heads: 69 -> 65.5 us at D =
        // 128, 61 -> 55 at D = 96; 1-2 % where the CUs are full; level at D = 64)
        const lds_ptr nxt = slots + (shift > 0 ? TILE : 0);
        constexpr int HOOKS = NB * 2 * KK;
        auto spread = [&](int h) __attribute__((always_inline)) {
#pragma unroll
            for (int i = h * L / HOOKS; i < (h + 1) * L / HOOKS; ++i) load_part(next_j, next_valid, nxt, i);
            __builtin_amdgcn_sched_barrier(0x786);              // MFMAs and loads keep this order
        };
        const int trow0 = j * TS + g * 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {       // one 32-row block at a time: only its accumulators are live
            f32x16 sacc, dpacc;
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(1);
            products(0, nb, false, sacc, [&](int kk) __attribute__((always_inline)) { spread(nb * 2 * KK + kk); });
            products(T2BASE, nb, true, dpacc, [&](int kk) __attribute__((always_inline)) { spread((nb * 2 + 1) * KK + kk); });
            if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
            if (mask) weights(nb, trow0, sacc, dpacc, std::true_type{});
            else      weights(nb, trow0, sacc, dpacc, std::false_type{});
        }
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(2);
        accumulate(0, xb, oacc);
        if constexpr (FUSED) accumulate(T2BASE, pb, oacc2);       // dV^T += dO^T P
        if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
    };
    // a tile needs the mask if it reaches past row S-1 or (causal) crosses the diagonal of any of this workgroup's rows
    auto needs_mask = [&](int j) __attribute__((always_inline)) -> bool {
        if ((j + 1) * TS > S) return true;
        if (!causal) return false;
        return KEYS_RES ? j * TS < r0 + RM - 1 : (j + 1) * TS - 1 > r0;
    };
    if constexpr (!KEYS_RES) {
        // rows that see at most kBwdShortRow keys: Delta from its definition, before the pass proper.  Such rows are among
        // the first kBwdShortRow of a head, their keys too.
        if (!HAVE_STATS && r0 < kBwdShortRow && (causal || S <= kBwdShortRow)) {
            float sum = 0.f;
            for (int j = 0; j * TS < kBwdShortRow && j < j1; ++j) {
                load_tile(j, true, slots);
                TSDPA_WAIT_VMCNT0();
                __syncthreads();
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    f32x16 sacc, dpacc;
                    products(0, nb, false, sacc, nothing);
                    products(T2BASE, nb, true, dpacc, nothing);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int trow = j * TS + nb * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                        if (trow <= thi) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -lse_r)) * dpacc[i];
                    }
                }
                __syncthreads();
            }
            sum = pair_sum(sum);
            if (rrow < kBwdShortRow) delta_r = sum;
        }
        if constexpr (DELTA16) {
#pragma unroll
            for (int i = 0; i < 16; ++i) minus_delta[i] = -delta_r;
            TSDPA_OPAQUE(minus_delta);            // (left transparent, it is built again for every block)
        }
        if (!HAVE_STATS && stream == 0 && g == 0 && rrow < S) {
            stats[(size_t)head * S + rrow] = -delta_r;
            *(float *)((char *)stats + stat_bytes + ((size_t)head * S + rrow) * 4) = lse_r;
        }
    }
    constexpr bool HEADS = GRP && KEYS_RES;
    auto to_head = [&](int h) __attribute__((always_inline)) {     // descriptors of head h of the group
        t1_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(t1 + (size_t)h * S * D), (short)0, S * G::GROW, 0x00020000);
        t2_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(t2 + (size_t)h * S * D), (short)0, S * G::GROW, 0x00020000);
    };
    if constexpr (NS == 1) {
        for (int h = 0; h < (HEADS ? Gn : 1); ++h) {
            // next query head of the group: its Q, dO and statistics (the last barrier of the previous head's
            // loop has every wavefront past its last LDS read and every outstanding load landed)
            if (HEADS && h > 0) to_head(h);
            // (into the slot that the pointers stand at)
            load_stats(h * S + j0 * TS, shift > 0 ? 0 : 1);
            load_tile(j0, true, slots + (shift > 0 ? 0 : TILE));
            TSDPA_WAIT_VMCNT0();
            __syncthreads();
            for (int j = j0; j < j1; ++j) {
                tile(j, needs_mask(j), j + 1, h * S + (j + 1) * TS, j + 1 < j1);
                TSDPA_WAIT_VMCNT0();
                __syncthreads();
                other_slot();
            }
        }
    } else {
        // The tiles of this stream: every NS-th of the sequence (head of the group, tile), the next one's loads always a
        // step ahead, also across heads.
        const int nj = j1 - j0;
        int jn = j0 + stream, hn = 0;             // tile whose loads go out next, and its head within the group
        auto settle = [&]() __attribute__((always_inline)) {
            if constexpr (HEADS) {
                bool moved = false;
                while (jn >= j1 && hn < Gn) {
                    jn -= nj;
                    ++hn;
                    moved = true;
                }
                if (moved && hn < Gn) to_head(hn);
            }
        };
        auto valid = [&]() __attribute__((always_inline)) -> bool { return HEADS ? hn < Gn : jn < j1; };
        settle();
        load_stats(hn * S + jn * TS, 0);
        load_tile(jn, valid(), slots);
        int j = jn;
        bool here = valid();
        jn += NS;
        settle();
        TSDPA_WAIT_VMCNT0();
        __syncthreads();
        const int steps = ((HEADS ? Gn * nj : nj) + NS - 1) / NS;
        for (int step = 0; step < steps; ++step) {
            if (here) tile(j, needs_mask(j), jn, hn * S + jn * TS, valid());
            TSDPA_WAIT_VMCNT0();
            if constexpr (NW > 1) __syncthreads();    // (a wavefront that streams alone waits for nobody)
            other_slot();
            j = jn;
            here = valid();
            jn += NS;
            settle();
        }
    }

    // ---- the streams' sums, added in the order of the streams by the wavefronts of the first one
    if constexpr (NS > 1) {
        auto gather = [&](f32x16 (&acc)[DB]) __attribute__((always_inline)) {
            __syncthreads();                      // (the region's last readers are through)
            const lds_ptr at = lds + wave * (32 * D * 4) + lane * 16;
            constexpr int DIST = NW * 32 * D * 4;
            if (stream > 0) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        f32x4 part;
#pragma unroll
                        for (int e = 0; e < 4; ++e) part[e] = acc[db][q4 * 4 + e];
                        *(TSDPA_LDS f32x4 *)(at + (stream - 1) * DIST + (db * 4 + q4) * 1024) = part;
                    }
            }
            __syncthreads();
            if (stream == 0) {
#pragma unroll
                for (int s = 0; s < NS - 1; ++s)
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4) {
                            const f32x4 part = *(TSDPA_LDS f32x4 *)(at + s * DIST + (db * 4 + q4) * 1024);
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[db][q4 * 4 + e] += part[e];
                        }
            }
        };
        gather(oacc);
        if constexpr (FUSED) gather(oacc2);
        __syncthreads();
        if (stream != 0) return;
    }

    // ---- store: out^T tiles are turned through LDS (as the forward kernel's O) and written as whole
    // rows; dQ and dK carry the factor `scale` of the score, dV none.  The last barrier of the loop has
    // every wavefront past its last LDS read.
    auto store = [&](const f32x16 (&acc)[DB], float factor, T *dst) __attribute__((always_inline)) {
        constexpr int OCPR = G::OROW / 16, CMASK = OCPR - 1;
        const lds_ptr ow = lds + wave * (32 * G::OROW);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                vec4 val;
#pragma unroll
                for (int e = 0; e < 4; ++e) val[e] = (T)(acc[db][q4 * 4 + e] * factor);
                const int chunk = db * 4 + q4;
                *(TSDPA_LDS vec4 *)(ow + l32 * G::OROW + ((chunk ^ (l32 & CMASK)) << 4) + g * 8) = val;
            }
        constexpr int RPI = 64 / OCPR;
        const int row0 = r0 + wave * 32;
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int r = i * RPI + lane / OCPR, cc = lane % OCPR;
            const u32x4 val = lds_read128(ow + r * G::OROW + ((cc ^ (r & CMASK)) << 4));
            if (row0 + r < S && cc < G::CPR) *(u32x4 *)(dst + head_off + (size_t)(row0 + r) * D + cc * 8) = val;
        }
    };
    // (the launcher sizes the dynamic LDS for the larger of the tile slots and this staging area)
    store(oacc, scale, out);
    if constexpr (FUSED) store(oacc2, 1.0f, out2);   // same staging region: it is private to the wavefront, whose LDS operations complete in order
#endif
}

template <typename T, int D, int NW, int NS, int TS, int WPS, int MODE, bool GRP, bool R2LDS>
__global__ void __launch_bounds__(NW * NS * 64, WPS)
sdpa_bwd_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                const T *__restrict__ o, const float *__restrict__ lse, float *__restrict__ stats, T *__restrict__ out,
                T *__restrict__ out2, int S, int nR, int N, float c, float scale, uint32_t rsign, int causal,
                unsigned stat_bytes, int group, TileOrder order)
{
    bwd_pass<T, D, NW, NS, TS, MODE, GRP, R2LDS, false>(q, k, v, dout, o, lse, stats, out, out2, S, nR, N, c, scale, rsign,
                                                        causal, stat_bytes, group, order, blockIdx.x);
}

// LDS of one instantiation: slots and statistics of every stream during the loop (and the resident operand kept there), then
// the sums of the streams, then one 32 x D block per wavefront of a stream for the output transpose.
template <int D, int NW, int NS, int TS, int MODE, bool R2LDS> constexpr int bwd_lds_bytes()
{
    const int loop = NS * bwd_stream_bytes<D, TS, MODE>() + (R2LDS ? NW * (D / 16) * 1024 : 0);
    const int sums = (NS - 1) * NW * 32 * D * 4;
    const int stage = NW * 32 * BwdGeom<D>::OROW;
    const int most = loop > sums ? loop : sums;
    return most > stage ? most : stage;
}

}  // namespace tsdpa
