// Backward pass of short sequences (S <= 256, one query head per key/value head): one workgroup per head computes dQ, dK
// and dV in one launch.
//
// The general passes (sdpa_bwd_kernel.h) compute scores and dP twice, once with the queries resident and once with the keys,
// because a head's sums are spread over workgroups; they read Q, K, V and dO twice and are launches of their own.  A
// sequence of up to 256 keys fits one workgroup: wavefront w owns the keys 32w ... 32w + 31 (K and V rows as MFMA operands
// and the dK, dV accumulators in registers), Q and dO stream through the LDS in tiles of 32 rows, and dS of a tile (keys x 32
// queries, 16 bits) goes through the LDS to the wavefronts that share out its dQ tile in blocks of 16 x 16.  Five products
// instead of seven, every input read once, one barrier per tile: a wavefront does the dQ blocks of tile j after the barrier
// that ends its part of tile j, while others are already in tile j + 1 (two dS buffers).
// What bounds it: per tile and wavefront about 640 cycles of MFMA and 500 of vector work at D = 64 that overlap only across
// the two wavefronts of a SIMD (more would not fit 256 registers), and prologue and epilogue, which nothing overlaps where
// eight wavefronts fill the CU; with more such heads than CUs sdpa_bwd_heads_kernel below overlaps them.
#pragma once
#include <mutex>

#include "sdpa_bwd_kernel.h"
#include "sdpa_decode_kernel.h"

namespace tsdpa {

template <int D, int NW> struct BwdShortGeom {
    using G = BwdGeom<D>;
    static constexpr int TASKS = 2 * (D / 16);    // 16 x 16 blocks of a dQ tile
    static constexpr int NTASK = (TASKS + NW - 1) / NW;
    // K^T of a wavefront's blocks stays in registers where the wavefronts divide the 16-column blocks evenly
    static constexpr int NDB = (D / 16) / NW > 1 ? (D / 16) / NW : 1;       // distinct column blocks per wavefront
    static constexpr bool KTREG = D == 64;
    static constexpr int NSLOT = KTREG ? 4 : 2;   // tiles in the LDS: the present one and those on their way
    static constexpr int LPT = 2 * (32 * G::CPR / 64) / NW;                 // load instructions per wavefront and tile (KTREG: NW divides)
    // from 0 on: NSLOT Q tiles, NSLOT dO tiles
    static constexpr int STATS = 2 * NSLOT * G::bytes(32);                  // LSE in log2 units, then -Delta, of NW * 32 rows
    static constexpr int DSBUF = NW * 32 * 64;    // dS^T: a row of 32 queries (64 bytes) per key
    static constexpr int KBASE = STATS + 2 * NW * 32 * 4;
    static constexpr int KBYTES = G::bytes(NW * 32);
    static constexpr int DSBASE = KTREG ? KBASE : KBASE + KBYTES;           // (K is through once it is in registers)
    static constexpr int LOOP = (KTREG ? (KBYTES > 2 * DSBUF ? KBYTES : 2 * DSBUF) : KBYTES + 2 * DSBUF) + KBASE;
    static constexpr int STAGE = NW * 32 * G::OROW;
    static constexpr int LDS_BYTES = LOOP > STAGE ? LOOP : STAGE;
    // Byte offset of queries 4*q4 ... 4*q4 + 3 of key row `key` in a dS buffer.  Written as 8 bytes per lane by 32 consecutive
    // keys (all 64 banks), read transposed, 32 bytes of 8 consecutive keys at a time: both free of bank conflicts.
    static __host__ __device__ constexpr int ds_at(int key, int q4) {
        const int f = (((key >> 2) & 1) << 1) | ((key >> 3) & 1);
        return key * 64 + (((q4 >> 1) ^ f) << 4) + (((q4 & 1) ^ ((key >> 4) & 1)) << 3);
    }
};

// LDS of sdpa_bwd_heads_kernel: three Q tiles, three dO tiles, LSE in log2 units and -Delta of 256 rows, two dS buffers, K, V and O of a head.
struct BwdHeadsGeom {
    using G = BwdGeom<64>;
    static constexpr int U = 4, TILE = G::bytes(32), BLOCK = G::bytes(256), DSBUF = 256 * 64;
    static constexpr int DO = 3 * TILE, STATS = 6 * TILE, DS = STATS + 2 * 256 * 4, HEAD = DS + 2 * DSBUF;
    static constexpr int LDS_BYTES = HEAD + 3 * BLOCK;
    static __host__ __device__ constexpr int ds_at(int key, int q4) { return BwdShortGeom<64, 8>::ds_at(key, q4); }
    static_assert(256 * G::OROW <= 2 * DSBUF && DS % 1024 == 0, "dK and dV are turned where dS was; its chunks are XORed");
};

// Sixteen (or eight) transposing reads and the wait for them in one block of inline assembly.  Left to the compiler, which
// cannot tell the slots apart, the first such read of a tile waits for every tile on its way.  (One block: the compiler
// takes an output for written when its block ends; early clobbers because the addresses are read until the last of them.)
#define TSDPA_RD_TR(i, a, n) "ds_read_b64_tr_b16 %" #i ", %" #a " offset:%" #n "\n\t"
// x[0..7] at dO, x[8..15] at Q: [ks][db][lo, hi], O apart
template <int O, int R> __device__ __forceinline__ void short_read_tiles(i16x4 (&x)[16], uint32_t lo0, uint32_t hi0, uint32_t lo1, uint32_t hi1)
{
    asm volatile(TSDPA_RD_TR(0, 16, 20) TSDPA_RD_TR(1, 17, 20) TSDPA_RD_TR(2, 18, 20) TSDPA_RD_TR(3, 19, 20)
                 TSDPA_RD_TR(4, 16, 21) TSDPA_RD_TR(5, 17, 21) TSDPA_RD_TR(6, 18, 21) TSDPA_RD_TR(7, 19, 21)
                 TSDPA_RD_TR(8, 16, 22) TSDPA_RD_TR(9, 17, 22) TSDPA_RD_TR(10, 18, 22) TSDPA_RD_TR(11, 19, 22)
                 TSDPA_RD_TR(12, 16, 23) TSDPA_RD_TR(13, 17, 23) TSDPA_RD_TR(14, 18, 23) TSDPA_RD_TR(15, 19, 23)
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7]),
                   "=&v"(x[8]), "=&v"(x[9]), "=&v"(x[10]), "=&v"(x[11]), "=&v"(x[12]), "=&v"(x[13]), "=&v"(x[14]), "=&v"(x[15])
                 : "v"(lo0), "v"(hi0), "v"(lo1), "v"(hi1), "n"(O), "n"(O + R), "n"(0), "n"(R)
                 : "memory");
}
// x[2i], x[2i + 1]: lo and hi + i * STRIDE, i < 4 (TWO: i < 2, twice)
template <int STRIDE, bool TWO> __device__ __forceinline__ void short_read_blocks(i16x4 *x, uint32_t lo, uint32_t hi)
{
    asm volatile(TSDPA_RD_TR(0, 8, 10) TSDPA_RD_TR(1, 9, 10) TSDPA_RD_TR(2, 8, 11) TSDPA_RD_TR(3, 9, 11)
                 TSDPA_RD_TR(4, 8, 12) TSDPA_RD_TR(5, 9, 12) TSDPA_RD_TR(6, 8, 13) TSDPA_RD_TR(7, 9, 13)
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                 : "v"(lo), "v"(hi), "n"(0), "n"(STRIDE), "n"(TWO ? 0 : 2 * STRIDE), "n"(TWO ? STRIDE : 3 * STRIDE)
                 : "memory");
}
#undef TSDPA_RD_TR

template <typename T, int D, int NW, bool CAUSAL>
__global__ void __launch_bounds__(NW * 64, 2)
sdpa_bwd_short_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                      const T *__restrict__ o, const float *__restrict__ lse, T *__restrict__ dq, T *__restrict__ dk,
                      T *__restrict__ dv, int S, float c, float scale, uint32_t rsign)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    using vec4 = typename E::vec4;
    using G = BwdGeom<D>;
    using W = BwdShortGeom<D, NW>;
    constexpr int KK = D / 16, DB = D / 32, U = 32 * G::CPR / 64;          // U: load units per tile of one tensor
    constexpr int TILE = G::bytes(32), ROW16 = G::bytes(16);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, l32 = lane & 31, t = lane >> 4, l16 = lane & 15;

    const size_t head = blockIdx.x, off = head * (size_t)S * D;
    const int row = wave * 32 + l32, row_c = row < S ? row : S - 1;        // this lane's key, and its query in the prologue
    const int nb = (S + 31) / 32;                 // 32-row blocks of the sequence
    auto rsrc_of = [&](const T *p) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(p + off), (short)0, S * G::GROW, 0x00020000);
    };
    const auto q_rsrc = rsrc_of(q), do_rsrc = rsrc_of(dout);
    // unit u (64 chunks) of rows from row0 on, of the tensor behind rsrc
    auto load_unit = [&](decltype(q_rsrc) rsrc, lds_ptr dst, int u, int row0) __attribute__((always_inline)) {
        const int p = u * 64 + lane, r = p / G::CPR, cp = p % G::CPR;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(dst + u * G::UNIT), 16,
                                                 r * G::GROW + ((cp ^ G::swz(r)) << 4), row0 * G::GROW, 0, 0);
    };
    // Q and dO of tile j, their 2U units dealt over the wavefronts (rows past the end, also of a tile past it: zeros)
    auto load_tile = [&](int j, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (2 * U + NW - 1) / NW; ++i) {
            const int u = i * NW + wave;
            if (2 * U % NW != 0 && u >= 2 * U) break;
            const bool first = u < U;
            load_unit(first ? q_rsrc : do_rsrc, lds + (first ? 0 : W::NSLOT * TILE) + slot * TILE, first ? u : u - U, j * 32);
        }
    };
    const bool short_rows = CAUSAL || S <= kBwdShortRow;       // (their Delta comes from its definition: see the general kernel)

    // ---- prologue: K into the LDS, the first tile (or the first rows of V, for the short rows' Delta) beside it
    {
        const auto k_rsrc = rsrc_of(k);
#pragma unroll
        for (int u = 0; u < U; ++u) load_unit(k_rsrc, lds + W::KBASE + wave * TILE, u, wave * 32);
        if (short_rows) {
            const auto v_rsrc = rsrc_of(v);
#pragma unroll
            for (int i = 0; i < (2 * U + NW - 1) / NW; ++i) {
                const int u = i * NW + wave;
                if (2 * U % NW != 0 && u >= 2 * U) break;
                load_unit(v_rsrc, lds, u, 0);
            }
        } else {
            load_tile(0, 0);
        }
    }
    vec8 rf1[KK], rf2[KK];                        // K and V rows of this wavefront; the sign of a negative scale goes into K's
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        u32x4 raw = *(const u32x4 *)(k + off + (size_t)row_c * D + kk * 16 + g * 8);
        raw ^= rsign;
        rf1[kk] = __builtin_bit_cast(vec8, raw);
        rf2[kk] = *(const vec8 *)(v + off + (size_t)row_c * D + kk * 16 + g * 8);
    }
    // per-lane pointers, as in the general kernel
    lds_ptr row_ptr[G::NRP];
#pragma unroll
    for (int i = 0; i < G::NRP; ++i) {
        row_ptr[i] = lds + G::at(l32, 2 * G::rp_kk(i) + g);
        TSDPA_OPAQUE(row_ptr[i]);
    }
    auto products = [&](int at, const vec8 (&rf)[KK], f32x16 &acc) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const u32x4 raw = lds_read128(row_ptr[G::rp(kk)] + at + G::rp_imm(kk));
            acc = E::mfma(__builtin_bit_cast(vec8, raw), rf[kk], acc);
        }
    };
    {
        // statistics of the query rows 32w ...: LSE in log2 units (+inf past the end: weight 0) and Delta
        float lse_r = lse[head * S + row_c] * 1.44269504088896340736f, delta_r = 0.f;
        const T *orow = o + off + (size_t)row_c * D + g * 8, *drow = dout + off + (size_t)row_c * D + g * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const vec8 x = *(const vec8 *)(orow + kk * 16), y = *(const vec8 *)(drow + kk * 16);
#pragma unroll
            for (int e = 0; e < 8; ++e) delta_r += (float)x[e] * (float)y[e];
        }
        delta_r = pair_sum(delta_r);
        if (short_rows) {
            TSDPA_WAIT_VMCNT0();
            __syncthreads();
            if (wave * 32 < kBwdShortRow && wave < nb) {
                vec8 qf[KK], df[KK];
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    u32x4 raw = *(const u32x4 *)(q + off + (size_t)row_c * D + kk * 16 + g * 8);
                    raw ^= rsign;
                    qf[kk] = __builtin_bit_cast(vec8, raw);
                    df[kk] = *(const vec8 *)(drow + kk * 16);
                }
                const int thi = CAUSAL ? row_c : S - 1;
                float sum = 0.f;
                for (int j = 0; j < kBwdShortRow / 32 && j < nb; ++j) {
                    f32x16 sacc, dpacc;
#pragma unroll
                    for (int i = 0; i < 16; ++i) sacc[i] = dpacc[i] = 0.f;
                    products(W::KBASE + j * TILE, qf, sacc);
                    products(j * TILE, df, dpacc);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int key = j * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                        if (key <= thi) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -lse_r)) * dpacc[i];
                    }
                }
                delta_r = pair_sum(sum);
            }
            __syncthreads();                      // (V's rows are through: the slots take the first tile)
            load_tile(0, 0);
        }
        // (behind everything that is waited for here)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 1; i < W::NSLOT - 1; ++i) load_tile(i, i);
        if (g == 0) {
            TSDPA_LDS float *st = (TSDPA_LDS float *)(lds + W::STATS);
            st[row] = row < S ? lse_r : INFINITY;
            st[NW * 32 + row] = row < S ? -delta_r : 0.f;
        }
    }
    // The barrier that ends a tile: the next one has landed in the LDS, this one's dS is written.
    auto tile_barrier = [&]() __attribute__((always_inline)) {
        if constexpr (W::KTREG) {
            // the next tile has landed when at most the two after it are outstanding (stores of dQ may count as well: then
            // more has landed than needed); __syncthreads would wait for all of them
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(2 * W::LPT) : "memory");
        } else {
            TSDPA_WAIT_VMCNT0();
            __syncthreads();
        }
    };
    tile_barrier();

    // ---- this wavefront's share of the dQ tiles: blocks `task` = 16 queries (half of the tile) x 16 columns
    // transposing reads, 16 lanes x 4 values: key row 4t + l16/4 (+16), 8 bytes l16%4 of the 32 of the block
    const int k_row = 4 * t + (l16 >> 2);
    vec8 kt[W::KTREG ? W::NDB : 1][W::KTREG ? NW : 1];         // K^T of the wavefront's column blocks, 32 keys each
    auto read_kt = [&](int db, int kb) __attribute__((always_inline)) {
        const lds_ptr p = lds + W::KBASE + G::at(k_row, db * 2 + ((l16 & 3) >> 1)) + (l16 & 1) * 8 + kb * 2 * ROW16;
        const i16x4 lo = lds_read_tr16(p), hi = lds_read_tr16(p + ROW16);
        return __builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    if constexpr (W::KTREG) {
#pragma unroll
        for (int i = 0; i < W::NDB; ++i) {
            constexpr int NKB = NW < 4 ? 4 : NW;
            const int db = (wave + i * NW) % (D / 16);
            const uint32_t lo = __builtin_bit_cast(uint32_t, lds) + W::KBASE + G::at(k_row, db * 2 + ((l16 & 3) >> 1)) + (l16 & 1) * 8;
            i16x4 x[2 * NKB];
#pragma unroll
            for (int n = 0; n < NKB; n += 4)
                short_read_blocks<2 * ROW16, NW == 2>(x + 2 * n, lo + n * 2 * ROW16, lo + (n * 2 + 1) * ROW16);
#pragma unroll
            for (int kb = 0; kb < NW; ++kb)
                kt[i][kb] = __builtin_bit_cast(vec8, __builtin_shufflevector(x[2 * kb], x[2 * kb + 1], 0, 1, 2, 3, 4, 5, 6, 7));
        }
        __syncthreads();                          // (the dS buffers take K's place)
    }

    f32x16 acc_k[DB], acc_v[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc_k[db][i] = acc_v[db][i] = 0.f;
    const int t_row = g * 4 + ((lane & 15) >> 2), t_chunk = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    lds_ptr tr_lo[G::NTP], tr_hi[G::NTP];
#pragma unroll
    for (int i = 0; i < G::NTP; ++i) {
        tr_lo[i] = lds + G::at(t_row, i * 4 + t_chunk) + (lane & 1) * 8;
        tr_hi[i] = lds + G::at(t_row + 8, i * 4 + t_chunk) + (lane & 1) * 8;
        TSDPA_OPAQUE(tr_lo[i]);
        TSDPA_OPAQUE(tr_hi[i]);
    }
    auto accumulate = [&](int at, const vec8 (&x)[2], f32x16 (&acc)[DB]) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int imm = at + ks * ROW16 + G::tp_imm(db);
                const i16x4 lo = lds_read_tr16(tr_lo[G::tp(db)] + imm), hi = lds_read_tr16(tr_hi[G::tp(db)] + imm);
                acc[db] = E::mfma(__builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)), x[ks], acc[db]);
            }
    };
    // Keys past the end (lanes of the last block, with copies of the last key's rows): their rows of dK and dV are not stored, and
    // their dS, which other lanes' dQ would meet, is not written: the buffers hold zeros there.  (Under a mask per weight the
    // last block's wavefront took 160 vector instructions for the weights of a tile instead of 64, and held up the others at
    // every barrier: B=64 H=12 S=197 59.5 us.)
    vec8 pb[2], xb[2];
    auto weights = [&](int j, const f32x16 &sacc, const f32x16 &dpacc, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_tag)::value;
        const lds_ptr st = lds + W::STATS + (j * 32 + g * 4) * 4;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 st_lse = *(TSDPA_LDS f32x4 *)(st + r4 * 32);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = r4 * 4 + e, qrow = j * 32 + r4 * 8 + g * 4 + e;
                const bool masked = MASK && qrow < row;             // a key after the query
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -st_lse[e]));
                const float x = p * dpacc[i];
                pb[i >> 3][i & 7] = (T)(masked ? 0.f : p);
                xb[i >> 3][i & 7] = (T)(masked ? 0.f : x);
            }
        }
    };
    const int ds_w0 = W::DSBASE + W::ds_at(row, g);            // run r4 of this lane's key: chunk r4 ^ f, as an XOR of the address
    const lds_ptr ds_r = lds + W::DSBASE;
    if (row >= S)
#pragma unroll
        for (int i = 0; i < 8; ++i) *(TSDPA_LDS u32x2 *)(lds + (i >> 2) * W::DSBUF + (ds_w0 ^ ((i & 3) << 4))) = u32x2{0u, 0u};

    int slot = 0;
    const int qh0 = NW == 8 ? wave / 4 : 0;       // KTREG: the first half of the tile's queries that this wavefront has blocks in
    const uint32_t ds_lo = __builtin_bit_cast(uint32_t, ds_r) + W::ds_at(k_row, qh0 * 4 + (l16 & 3));
    const uint32_t ds_hi = __builtin_bit_cast(uint32_t, ds_r) + W::ds_at(k_row + 16, qh0 * 4 + (l16 & 3));
    for (int j = 0; j < nb; ++j) {
        const int ahead = j + W::NSLOT - 1, free_slot = (slot + W::NSLOT - 1) % W::NSLOT;
        if (W::KTREG || ahead < nb) load_tile(ahead, free_slot);   // (KTREG: also past the end, for the count of the wait below)
        const int at = slot * TILE, ds_buf = (j & 1) * W::DSBUF;
        if (wave < nb && (!CAUSAL || j >= wave)) {
            // (dP starts from -Delta; no branch between the two chains of MFMAs, which fill each other's waits)
            f32x16 sacc, dpacc;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4 md = *(TSDPA_LDS f32x4 *)(lds + W::STATS + (NW * 32 + j * 32 + g * 4) * 4 + r4 * 32);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sacc[r4 * 4 + e] = 0.f;
                    dpacc[r4 * 4 + e] = md[e];
                }
            }
            products(at, rf1, sacc);
            products(W::NSLOT * TILE + at, rf2, dpacc);
            if (CAUSAL && j == wave) weights(j, sacc, dpacc, std::true_type{});
            else                     weights(j, sacc, dpacc, std::false_type{});
            if (row < S)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    vec4 x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = xb[r4 >> 1][(r4 & 1) * 4 + e];
                    *(TSDPA_LDS vec4 *)(lds + ds_buf + (ds_w0 ^ (r4 << 4))) = x;
                }
            // dV^T += dO^T P, dK^T += Q^T dS
            if constexpr (W::KTREG) {
                i16x4 x[16];
                auto addr = [&](lds_ptr p) __attribute__((always_inline)) { return __builtin_bit_cast(uint32_t, p) + at; };
                short_read_tiles<W::NSLOT * TILE, ROW16>(x, addr(tr_lo[0]), addr(tr_hi[0]), addr(tr_lo[1]), addr(tr_hi[1]));
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        auto operand = [&](int i) __attribute__((always_inline)) {
                            return __builtin_bit_cast(vec8, __builtin_shufflevector(x[i], x[i + 1], 0, 1, 2, 3, 4, 5, 6, 7));
                        };
                        acc_v[db] = E::mfma(operand((ks * 2 + db) * 2), pb[ks], acc_v[db]);
                        acc_k[db] = E::mfma(operand(8 + (ks * 2 + db) * 2), xb[ks], acc_k[db]);
                    }
            } else {
                accumulate(W::NSLOT * TILE + at, pb, acc_v);
                accumulate(at, xb, acc_k);
            }
        }
        tile_barrier();
        // dQ of the tile: [16 columns][16 queries] += K^T dS^T over the keys (causal: up to the tile's own)
        const int kbs = CAUSAL ? j + 1 : nb;
        auto put = [&](const f32x4 &acc, int db, int qh) __attribute__((always_inline)) {
            const int qrow = j * 32 + qh * 16 + l16;
            vec4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (T)(acc[e] * scale);
            if (qrow < S) *(vec4 *)(dq + off + (size_t)qrow * D + db * 16 + t * 4) = out;
        };
        if constexpr (W::KTREG) {
            // (operands of key blocks without dS are read, not used)
            constexpr int NQH = NW == 8 ? 1 : 2, NKB = NW < 4 ? 4 : NW;
#pragma unroll
            for (int h = 0; h < NQH; ++h) {
                i16x4 x[2 * NKB];
                // (the other half: queries 16 further on, chunk ^ 2 of the dS row)
                const uint32_t lo = (ds_lo + ds_buf) ^ (h << 5), hi = (ds_hi + ds_buf) ^ (h << 5);
#pragma unroll
                for (int i = 0; i < NKB; i += 4) short_read_blocks<2048, NW == 2>(x + 2 * i, lo + i * 2048, hi + i * 2048);
                // two chains per block, even and odd key blocks; without the mask all of them in one run (dS past the end is zero)
                f32x4 acc[W::NDB][2];
#pragma unroll
                for (int d = 0; d < W::NDB; ++d) acc[d][0] = acc[d][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < NW; ++kb) {
                    if (CAUSAL && kb >= kbs) break;
                    const vec8 b = __builtin_bit_cast(vec8, __builtin_shufflevector(x[2 * kb], x[2 * kb + 1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                    for (int d = 0; d < W::NDB; ++d) acc[d][kb & 1] = Elem16<T>::mfma(kt[d][kb], b, acc[d][kb & 1]);
                }
#pragma unroll
                for (int d = 0; d < W::NDB; ++d) put(acc[d][0] + acc[d][1], (wave + d * NW) % (D / 16), qh0 + h);
            }
        } else {
#pragma unroll 1
            for (int i = 0; i < W::NTASK; ++i) {
                const int task = wave + i * NW;
                if (W::TASKS % NW != 0 && task >= W::TASKS) break;
                const int db = task % (D / 16), qh = task / (D / 16);
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < NW; ++kb) {
                    if (kb >= kbs) break;
                    const lds_ptr p = ds_r + ds_buf + kb * 2048;
                    const i16x4 lo = lds_read_tr16(p + W::ds_at(k_row, qh * 4 + (l16 & 3)));
                    const i16x4 hi = lds_read_tr16(p + W::ds_at(k_row + 16, qh * 4 + (l16 & 3)));
                    const vec8 b = __builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    acc = Elem16<T>::mfma(read_kt(db, kb), b, acc);
                }
                put(acc, db, qh);
            }
        }
        slot = (slot + 1) % W::NSLOT;
    }

    // ---- dK and dV through the LDS as whole rows (as in the general kernel)
    TSDPA_WAIT_VMCNT0();
    __syncthreads();
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
                *(TSDPA_LDS vec4 *)(ow + l32 * G::OROW + (((db * 4 + q4) ^ (l32 & CMASK)) << 4) + g * 8) = val;
            }
        constexpr int RPI = 64 / OCPR;
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int r = i * RPI + lane / OCPR, cc = lane % OCPR;
            const u32x4 val = lds_read128(ow + r * G::OROW + ((cc ^ (r & CMASK)) << 4));
            if (wave * 32 + r < S && cc < G::CPR) *(u32x4 *)(dst + off + (size_t)(wave * 32 + r) * D + cc * 8) = val;
        }
    };
    store(acc_k, scale, dk);
    store(acc_v, 1.0f, dv);                       // (same region: it is private to the wavefront, whose LDS operations complete in order)
#endif
}

template <typename T, int D, int NW, bool CAUSAL> int launch_bwd_short_mask(const BwdLaunchArgs &a)
{
    auto kern = sdpa_bwd_short_kernel<T, D, NW, CAUSAL>;
    constexpr int lds_bytes = BwdShortGeom<D, NW>::LDS_BYTES;
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.BH), dim3(NW * 64), lds_bytes, a.stream, (const T *)a.q, (const T *)a.k, (const T *)a.v,
                       (const T *)a.dout, (const T *)a.o, a.lse, (T *)a.dq, (T *)a.dk, (T *)a.dv, a.S, a.c, a.scale, a.rsign);
    return (int)hipGetLastError();
}

template <typename T, int D, int NW> int launch_bwd_short_nw(const BwdLaunchArgs &a)
{
    return a.causal ? launch_bwd_short_mask<T, D, NW, true>(a) : launch_bwd_short_mask<T, D, NW, false>(a);
}

// The same for sequences of 129 ... 256 rows at D = 64 and more heads than CUs: a workgroup per CU takes one head after another and
// fetches the next head's K, V and O into the LDS while it works on the present one, two load instructions per wavefront and tile; the
// next head's first tiles and dO rows are on their way while dK and dV are stored.  As a workgroup per head, whose eight wavefronts
// fill the CU, a head spent 13 of its 35 thousand clocks on the arrival of those, every CU at the same time, and 18 in the loop
// with the memory idle.  us per call, BF16, a workgroup per head -> this, the same tensors again and
// again (24 sets of them in turn, so that they come from memory): 768 heads of 197 rows 50.9 -> 44.9 (56.6 -> 51.7), causal 53.8 -> 47.4
// (60.1 -> 51.3), 1030 of 130 56.2 -> 51.3 (61.5 -> 52.7), 520 of 160 36.8 -> 33.7 (40.5 -> 36.3), 384 of 256 35.8 -> 34.4 (40.6 -> 38.3).
// What bounds it: the loop as above, now with the memory at work
// beside it, and the prologue of a workgroup's first head.
template <typename T, bool CAUSAL>
__global__ void __launch_bounds__(512, 2)
sdpa_bwd_heads_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                      const T *__restrict__ o, const float *__restrict__ lse, T *__restrict__ dq, T *__restrict__ dk,
                      T *__restrict__ dv, int heads, int S, float c, float scale, uint32_t rsign)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int D = 64, NW = 8;
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    using vec4 = typename E::vec4;
    using G = BwdGeom<D>;
    using W = BwdHeadsGeom;
    constexpr int KK = D / 16, DB = D / 32, U = W::U, TILE = W::TILE, ROW16 = G::bytes(16);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, l32 = lane & 31, t = lane >> 4, l16 = lane & 15;
    const int row = wave * 32 + l32, row_c = row < S ? row : S - 1;        // this lane's key, and its query in the statistics
    const int nb = (S + 31) / 32;                 // 32-row blocks of the sequence

    // (rows past the sequence read as zero and are not written)
    auto rsrc_of = [&](const T *p, int head) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(p + (size_t)head * S * D), (short)0, S * G::GROW, 0x00020000);
    };
    // a unit of eight rows; of a wavefront's units all have odd or all even numbers
    const int goff = (lane >> 3) * G::GROW + (((lane & 7) ^ G::swz((wave & 1) * 8 + (lane >> 3))) << 4);
    auto load_unit = [&](__amdgpu_buffer_rsrc_t rsrc, uint32_t dst, int unit) __attribute__((always_inline)) {
        lds_load16(rsrc, dst, goff, unit * 1024);
    };
    // Q and dO of tile j of the head behind rsrc: one unit per wavefront, of Q or of dO
    const T *const mine = wave < 4 ? q : dout;
    const uint32_t mine_at = lds0 + (wave < 4 ? 0 : W::DO) + (wave & 3) * 1024;
    auto load_tile = [&](__amdgpu_buffer_rsrc_t rsrc, int j, int slot) __attribute__((always_inline)) {
        load_unit(rsrc, mine_at + slot * TILE, j * U + (wave & 3));
    };
    // K, V and O of the head behind the three descriptors: part j of nb, two units per wavefront (the last ones more than once, so that
    // every part has two)
    auto fetch = [&](__amdgpu_buffer_rsrc_t k_rsrc, __amdgpu_buffer_rsrc_t v_rsrc, __amdgpu_buffer_rsrc_t o_rsrc, int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int at = j * 16 + i * 8 + wave, u = at < 12 * nb ? at : 12 * nb - 8 + wave;
            const int x = (u >= 4 * nb) + (u >= 8 * nb), uu = u - x * 4 * nb;
            load_unit(x == 0 ? k_rsrc : x == 1 ? v_rsrc : o_rsrc, lds0 + W::HEAD + x * W::BLOCK + uu * 1024, uu);
        }
    };
    lds_ptr row_ptr[G::NRP];
#pragma unroll
    for (int i = 0; i < G::NRP; ++i) {
        row_ptr[i] = lds + G::at(l32, 2 * G::rp_kk(i) + g);
        TSDPA_OPAQUE(row_ptr[i]);
    }
    auto operand = [&](int at, int kk) __attribute__((always_inline)) { return lds_read128(row_ptr[G::rp(kk)] + at + G::rp_imm(kk)); };
    auto products = [&](int at, const vec8 (&rf)[KK], f32x16 &acc) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) acc = E::mfma(__builtin_bit_cast(vec8, operand(at, kk)), rf[kk], acc);
    };
    const int t_row = g * 4 + (l16 >> 2), t_chunk = (t & 1) * 2 + ((lane & 3) >> 1), k_row = 4 * t + (l16 >> 2);
    uint32_t tr_lo[G::NTP], tr_hi[G::NTP];
#pragma unroll
    for (int i = 0; i < G::NTP; ++i) {
        tr_lo[i] = lds0 + G::at(t_row, i * 4 + t_chunk) + (lane & 1) * 8;
        tr_hi[i] = lds0 + G::at(t_row + 8, i * 4 + t_chunk) + (lane & 1) * 8;
        TSDPA_OPAQUE(tr_lo[i]);
        TSDPA_OPAQUE(tr_hi[i]);
    }
    // dQ: block of 16 columns wave % 4, queries (wave / 4) * 16 ...
    const int qh = wave / 4, cb = wave & 3;
    const uint32_t ds_lo = lds0 + W::DS + W::ds_at(k_row, qh * 4 + (l16 & 3)), ds_hi = lds0 + W::DS + W::ds_at(k_row + 16, qh * 4 + (l16 & 3));
    const uint32_t kt_at = lds0 + W::HEAD + G::at(k_row, cb * 2 + ((l16 & 3) >> 1)) + (l16 & 1) * 8;
    const int ds_w0 = W::DS + W::ds_at(row, g);   // run r4 of this lane's key: chunk r4 ^ f, as an XOR of the address

    int head = blockIdx.x;
    u32x4 drow[KK];                               // dO of the lane's row, and its LSE
    float lse_r;
    auto load_rows = [&](int h) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) drow[kk] = *(const u32x4 *)(dout + ((size_t)h * S + row_c) * D + kk * 16 + g * 8);
        lse_r = lse[(size_t)h * S + row_c];
    };
    auto t_rsrc = rsrc_of(mine, head);
    {
        const auto k_rsrc = rsrc_of(k, head), v_rsrc = rsrc_of(v, head), o_rsrc = rsrc_of(o, head);
        for (int j = 0; j < nb; ++j) fetch(k_rsrc, v_rsrc, o_rsrc, j);
    }
    load_tile(t_rsrc, 0, 0);
    load_tile(t_rsrc, 1, 1);
    load_rows(head);
    int slot = 0;                                 // of the head's first tile; tiles follow one another also across heads
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    for (;;) {
        const int next = head + (int)gridDim.x;
        const bool more = next < heads;
        const auto n_rsrc = rsrc_of(mine, next), k_rsrc = rsrc_of(k, next), v_rsrc = rsrc_of(v, next), o_rsrc = rsrc_of(o, next);
        const size_t off = (size_t)head * S * D;
        __syncthreads();
        // ---- K and V rows of this wavefront (the sign of a negative scale goes into K's), K^T of its dQ blocks
        vec8 rf1[KK], rf2[KK], kt[NW];
        float delta_r = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            rf1[kk] = __builtin_bit_cast(vec8, operand(W::HEAD + wave * TILE, kk) ^ rsign);
            rf2[kk] = __builtin_bit_cast(vec8, operand(W::HEAD + W::BLOCK + wave * TILE, kk));
            const vec8 x = __builtin_bit_cast(vec8, operand(W::HEAD + 2 * W::BLOCK + wave * TILE, kk)), y = __builtin_bit_cast(vec8, drow[kk]);
#pragma unroll
            for (int e = 0; e < 8; ++e) delta_r += (float)x[e] * (float)y[e];
        }
        delta_r = pair_sum(delta_r);
        const float lse2 = lse_r * 1.44269504088896340736f;
        {
            i16x4 x[2 * NW];
#pragma unroll
            for (int n = 0; n < NW; n += 4) short_read_blocks<2 * ROW16, false>(x + 2 * n, kt_at + n * 2 * ROW16, kt_at + (n * 2 + 1) * ROW16);
#pragma unroll
            for (int kb = 0; kb < NW; ++kb) {
                // (blocks past the end are whatever the LDS holds; their dS is zero)
                const u32x4 raw = __builtin_bit_cast(u32x4, __builtin_shufflevector(x[2 * kb], x[2 * kb + 1], 0, 1, 2, 3, 4, 5, 6, 7));
                kt[kb] = __builtin_bit_cast(vec8, kb < nb ? raw : u32x4{0u, 0u, 0u, 0u});
            }
        }
        if constexpr (CAUSAL) {
            // rows that see at most kBwdShortRow keys: Delta from its definition (see the general kernel); their Q is in the first tiles
            if (wave * 32 < kBwdShortRow) {
                vec8 qf[KK], df[KK];
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    qf[kk] = __builtin_bit_cast(vec8, operand((slot + wave) % 3 * TILE, kk) ^ rsign);
                    df[kk] = __builtin_bit_cast(vec8, drow[kk]);
                }
                float sum = 0.f;
                for (int j = 0; j < kBwdShortRow / 32; ++j) {
                    f32x16 sacc, dpacc;
#pragma unroll
                    for (int i = 0; i < 16; ++i) sacc[i] = dpacc[i] = 0.f;
                    products(W::HEAD + j * TILE, qf, sacc);
                    products(W::HEAD + W::BLOCK + j * TILE, df, dpacc);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int key = j * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                        if (key <= row_c) sum += __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -lse2)) * dpacc[i];
                    }
                }
                delta_r = pair_sum(sum);
            }
        }
        if (g == 0) {
            TSDPA_LDS float *st = (TSDPA_LDS float *)(lds + W::STATS);
            st[row] = row < S ? lse2 : INFINITY;
            st[NW * 32 + row] = row < S ? -delta_r : 0.f;
        }
        // dS of keys past the end is never written: zero
        if (row >= S)
#pragma unroll
            for (int i = 0; i < 8; ++i) *(TSDPA_LDS u32x2 *)(lds + (i >> 2) * W::DSBUF + (ds_w0 ^ ((i & 3) << 4))) = u32x2{0u, 0u};
        __syncthreads();                          // (K, V and O are through: the next head's may come)

        f32x16 acc_k[DB], acc_v[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc_k[db][i] = acc_v[db][i] = 0.f;
        vec8 pb[2], xb[2];
        auto weights = [&](int j, const f32x16 &sacc, const f32x16 &dpacc, auto mask_tag) __attribute__((always_inline)) {
            constexpr bool MASK = decltype(mask_tag)::value;
            const lds_ptr st = lds + W::STATS + (j * 32 + g * 4) * 4;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4 st_lse = *(TSDPA_LDS f32x4 *)(st + r4 * 32);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = r4 * 4 + e, qrow = j * 32 + r4 * 8 + g * 4 + e;
                    const bool masked = MASK && qrow < row;             // a key after the query
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], c, -st_lse[e]));
                    const float x = p * dpacc[i];
                    pb[i >> 3][i & 7] = (T)(masked ? 0.f : p);
                    xb[i >> 3][i & 7] = (T)(masked ? 0.f : x);
                }
            }
        };
        for (int j = 0; j < nb; ++j) {
            const bool own = j + 2 < nb;
            if (own || more) load_tile(own ? t_rsrc : n_rsrc, own ? j + 2 : j + 2 - nb, slot == 0 ? 2 : slot - 1);
            if (more) fetch(k_rsrc, v_rsrc, o_rsrc, j);
            const int at = slot * TILE, ds_buf = (j & 1) * W::DSBUF;
            if (wave < nb && (!CAUSAL || j >= wave)) {
                f32x16 sacc, dpacc;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 md = *(TSDPA_LDS f32x4 *)(lds + W::STATS + (NW * 32 + j * 32 + g * 4) * 4 + r4 * 32);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        sacc[r4 * 4 + e] = 0.f;
                        dpacc[r4 * 4 + e] = md[e];
                    }
                }
                products(at, rf1, sacc);
                products(W::DO + at, rf2, dpacc);
                if (CAUSAL && j == wave) weights(j, sacc, dpacc, std::true_type{});
                else                     weights(j, sacc, dpacc, std::false_type{});
                if (row < S)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        vec4 x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = xb[r4 >> 1][(r4 & 1) * 4 + e];
                        *(TSDPA_LDS vec4 *)(lds + ds_buf + (ds_w0 ^ (r4 << 4))) = x;
                    }
                // dV^T += dO^T P, dK^T += Q^T dS
                i16x4 x[16];
                short_read_tiles<W::DO, ROW16>(x, tr_lo[0] + at, tr_hi[0] + at, tr_lo[1] + at, tr_hi[1] + at);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        auto both = [&](int i) __attribute__((always_inline)) {
                            return __builtin_bit_cast(vec8, __builtin_shufflevector(x[i], x[i + 1], 0, 1, 2, 3, 4, 5, 6, 7));
                        };
                        acc_v[db] = E::mfma(both((ks * 2 + db) * 2), pb[ks], acc_v[db]);
                        acc_k[db] = E::mfma(both(8 + (ks * 2 + db) * 2), xb[ks], acc_k[db]);
                    }
            }
            // The next tile, requested a step ago, has landed when nothing but what was requested after it is outstanding: two units of
            // the next head then, the tile after the next and two more units now (a store of dQ may count as well: then more has landed).
            // In the last head the tile after the next is all there is.
            if (more) asm volatile("s_waitcnt vmcnt(5) lgkmcnt(0)" : : : "memory");
            else if (own) asm volatile("s_waitcnt vmcnt(1) lgkmcnt(0)" : : : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");
            __builtin_amdgcn_s_barrier();
            slot = slot == 2 ? 0 : slot + 1;
            // dQ of the tile: [16 columns][16 queries] += K^T dS^T over the keys (causal: up to the tile's own)
            i16x4 x[2 * NW];
#pragma unroll
            for (int i = 0; i < NW; i += 4) short_read_blocks<2048, false>(x + 2 * i, ds_lo + ds_buf + i * 2048, ds_hi + ds_buf + i * 2048);
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int kb = 0; kb < NW; ++kb) {
                if (CAUSAL && kb > j) break;
                const vec8 b = __builtin_bit_cast(vec8, __builtin_shufflevector(x[2 * kb], x[2 * kb + 1], 0, 1, 2, 3, 4, 5, 6, 7));
                acc[kb & 1] = Elem16<T>::mfma(kt[kb], b, acc[kb & 1]);
            }
            const int qrow = j * 32 + qh * 16 + l16;
            vec4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (T)((acc[0][e] + acc[1][e]) * scale);
            if (qrow < S) *(vec4 *)(dq + off + (size_t)qrow * D + cb * 16 + t * 4) = out;
        }
        // ---- the next head's rows, and dK and dV through the place of dS as whole rows (the barrier: dS is read)
        if (more) load_rows(next);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
        auto store = [&](const f32x16 (&acc)[DB], float factor, T *dst) __attribute__((always_inline)) {
            constexpr int OCPR = G::OROW / 16, CMASK = OCPR - 1;
            const lds_ptr ow = lds + W::DS + wave * (32 * G::OROW);
            const auto rsrc = rsrc_of(dst, head);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    vec4 val;
#pragma unroll
                    for (int e = 0; e < 4; ++e) val[e] = (T)(acc[db][q4 * 4 + e] * factor);
                    *(TSDPA_LDS vec4 *)(ow + l32 * G::OROW + (((db * 4 + q4) ^ (l32 & CMASK)) << 4) + g * 8) = val;
                }
            constexpr int RPI = 64 / OCPR;
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + lane / OCPR, cc = lane % OCPR;
                const u32x4 val = lds_read128(ow + r * G::OROW + ((cc ^ (r & CMASK)) << 4));
                __builtin_amdgcn_raw_buffer_store_b128(val, rsrc, r * G::GROW + cc * 16, wave * 32 * G::GROW, 0);        // (rows >= S: dropped)
            }
        };
        store(acc_k, scale, dk);
        store(acc_v, 1.0f, dv);                   // (same region: it is private to the wavefront, whose LDS operations complete in order)
        if (!more) break;
        // everything of the next head has landed; the eight stores may be on their way
        asm volatile("s_waitcnt vmcnt(8)" : : : "memory");
        head = next;
        t_rsrc = n_rsrc;
    }
#endif
}

template <typename T, bool CAUSAL> int launch_bwd_heads_mask(const BwdLaunchArgs &a)
{
    auto kern = sdpa_bwd_heads_kernel<T, CAUSAL>;
    static_assert(BwdHeadsGeom::LDS_BYTES <= 160 * 1024, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, BwdHeadsGeom::LDS_BYTES);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    hipLaunchKernelGGL(kern, dim3(256), dim3(512), BwdHeadsGeom::LDS_BYTES, a.stream, (const T *)a.q, (const T *)a.k, (const T *)a.v,
                       (const T *)a.dout, (const T *)a.o, a.lse, (T *)a.dq, (T *)a.dk, (T *)a.dv, a.BH, a.S, a.c, a.scale, a.rsign);
    return (int)hipGetLastError();
}

template <typename T> int launch_bwd_heads(const BwdLaunchArgs &a)
{
    return a.causal ? launch_bwd_heads_mask<T, true>(a) : launch_bwd_heads_mask<T, false>(a);
}

}  // namespace tsdpa
