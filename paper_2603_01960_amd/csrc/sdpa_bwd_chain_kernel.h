// Backward pass with five products per pair of tiles: scores and dP once, dV, dK and dQ from them.
//
// A workgroup owns 256 keys (K in the LDS, V in registers, dK and dV in accumulators) and streams Q and dO tiles of 32 rows, as the
// keys-resident pass of sdpa_bwd_kernel.h; it also multiplies the tile's dS (through the LDS, transposed) with its keys into the part of dQ
// that these keys give.  The parts of a query tile, one per block of keys, are summed in the order of the blocks: block b takes the sum of
// the blocks before it from the workspace (FP32), adds its own and leaves the result for block b + 1; the last block writes dQ.  The
// order is fixed, so results are deterministic.  Every block walks the query tiles in the same order, the last one first (causal: the
// diagonal last), so that block b runs a step or two behind block b - 1 and seldom waits.
//
// Who waits for whom: a workgroup takes its blocks by ticket, and waits only for blocks of lower tickets, which by then have a
// workgroup that runs.  Whatever the order and the number of workgroups on the card, the lowest unfinished block waits for nobody, so
// every wait ends.  The sums pass through the L2 of one XCD (8, 12 or 16 KB by head dim per step and workgroup each way: past the L2, at agent scope, the whole
// pass takes 1.3 to 1.5 times as long): an XCD claims whole key/value heads, and its workgroups, which ask the hardware where they
// are, take the blocks of its claims only.  A block starts by invalidating its CU's cache, in which a line of a sum could
// be left from an earlier block; within a block each line is read once.  Progress counters are written and read at agent scope, after the
// sums they stand for have been acknowledged.
//
// What bounds it: the matrix pipe under the power limit, with 5 instead of 7 products, at 0.57 of the pipe's cycles (64 heads S = 8192, D = 128).  One wavefront
// per SIMD (512 registers: 256 accumulators that only matrix instructions touch, 256 others) and 64 keys per wavefront halve the LDS
// reads per product against two wavefronts of 32 keys (which took 5.5 ms in the shape below, without the sums).  What a single wavefront
// issues beside its products is then what limits it (a vector instruction takes 5.8 clocks, an exponential 12, a scalar one 5, a transposing
// read 9, a product 32), so that the step is written out: reads two products ahead, the exponentials under the second half of
// the scores and the first half of dP, dS under the second half and dV, dQ's reads under dK.  Fences keep that order; the loads to the LDS are written in
// assembly, or the compiler would wait for all of them at the first transposing read.
// BF16, us per call, two passes -> this: D = 128, 64 heads S = 8192 6237 -> 5433, S = 2048 423 -> 369, 8 heads S = 16384 3107 -> 2613,
// 16 over 4 heads of four entries S = 4096 1572 -> 1334; causal 64 heads S = 8192 3263 -> 2820, S = 4096 855 -> 792; D = 96, 32 heads S = 4096
// 629 -> 546; D = 64, 64 heads S = 2048 233 -> 224.
#pragma once
#include <mutex>
#include "sdpa_bwd_joint_kernel.h"
#include "sdpa_bwd_pick.h"

namespace tsdpa {

template <int D> struct BwdChainGeom {
    using G = BwdGeom<D>;
    static constexpr int U = 32 * G::CPR / 64;                              // 1-KiB units of 32 rows of one tensor
    static constexpr int TILE = G::bytes(32), SLOT = 2 * TILE + 256;        // Q and dO of 32 rows, their statistics; three slots
    static constexpr int SLOTS = G::bytes(kChainKeys), DSB = kChainKeys * 64;       // K before them; dS of a tile, two of them
    static constexpr int DS = (SLOTS + 3 * SLOT + 1023) / 1024 * 1024, FLAGS = DS + 2 * DSB;
    static constexpr int LDS_BYTES = FLAGS + kChainWaves * 256 + 16;
    static_assert(TILE == U * G::UNIT, "Q's units, then dO's");
    // dQ of a tile: D = 128, 32 columns of all 32 queries per wavefront in one 32 x 32 product; D = 64 and 96, blocks of 16 x 16.  Sums of four
    // floats per lane and wavefront either way:
    static constexpr int PARTS = D / 32;
};

// what a launch shares, zero at its start
struct ChainQueue {
    unsigned next, pad[31];                       // claim that is handed out next
    struct { unsigned ticket, pad[31]; } xcd[kChainXcds];
};
static_assert(sizeof(ChainQueue) == kChainQueueBytes, "");

// arguments, read where they are needed (all of them in scalar registers at once, half would be spilled)
struct ChainArgs {
    const void *q, *k, *v, *dout;
    const float *stats;
    void *dq, *dk, *dv;
    float *part;
    unsigned *progress;
    ChainQueue *queue;
    unsigned *claims;
    int S, nB, HK, per_claim, nclaims, max_slots, causal, group;
    unsigned stat_bytes;
    float c, scale;
};

// all but the last N vector memory operations are complete
template <int N> __device__ __forceinline__ void wait_all_but() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
__device__ __forceinline__ void wait_all()
{
    asm volatile("" ::: "memory");
    TSDPA_WAIT_VMCNT0();
    asm volatile("" ::: "memory");
}

// acc0 += a b0, acc1 += a b1 with the accumulators in the registers that only matrix instructions reach.  A matrix instruction must not
// read a register less than two wait states after a vector instruction has written it, and the compiler, which may put a copy of an
// operand anywhere, does not look into assembly: the instruction before the products makes two.  (It costs 7 clocks: by pairs of
// products 0.6 % of a call, one by one 2 to 3 % at D = 64.)
//   * Of the 64 keys only the first `keys`, a multiple of 32 or less than one.  (As a branch of the compiler's, the accumulators moved at every join.)
template <typename T> struct AccMfma;
template <> struct AccMfma<_Float16> {
    static __device__ __forceinline__ void run(f32x16 &acc0, f32x16 &acc1, f16x8 a, f16x8 b0, f16x8 b1) {
        asm("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %2, %3, %0\n\tv_mfma_f32_32x32x16_f16 %1, %2, %4, %1" : "+a"(acc0), "+a"(acc1) : "v"(a), "v"(b0), "v"(b1));
    }
    static __device__ __forceinline__ void run(f32x16 &acc0, f32x16 &acc1, f16x8 a, f16x8 b0, f16x8 b1, int keys) {
        asm("s_cmp_lt_i32 %5, 32\n\ts_cbranch_scc1 .Lhidden%=\n\tv_mfma_f32_32x32x16_f16 %0, %2, %3, %0\n\t"
            "s_cmp_lt_i32 %5, 64\n\ts_cbranch_scc1 .Lhidden%=\n\tv_mfma_f32_32x32x16_f16 %1, %2, %4, %1\n.Lhidden%=:"
            : "+a"(acc0), "+a"(acc1) : "v"(a), "v"(b0), "v"(b1), "s"(keys) : "scc");
    }
};
template <> struct AccMfma<__bf16> {
    static __device__ __forceinline__ void run(f32x16 &acc0, f32x16 &acc1, bf16x8 a, bf16x8 b0, bf16x8 b1) {
        asm("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %2, %3, %0\n\tv_mfma_f32_32x32x16_bf16 %1, %2, %4, %1" : "+a"(acc0), "+a"(acc1) : "v"(a), "v"(b0), "v"(b1));
    }
    static __device__ __forceinline__ void run(f32x16 &acc0, f32x16 &acc1, bf16x8 a, bf16x8 b0, bf16x8 b1, int keys) {
        asm("s_cmp_lt_i32 %5, 32\n\ts_cbranch_scc1 .Lhidden%=\n\tv_mfma_f32_32x32x16_bf16 %0, %2, %3, %0\n\t"
            "s_cmp_lt_i32 %5, 64\n\ts_cbranch_scc1 .Lhidden%=\n\tv_mfma_f32_32x32x16_bf16 %1, %2, %4, %1\n.Lhidden%=:"
            : "+a"(acc0), "+a"(acc1) : "v"(a), "v"(b0), "v"(b1), "s"(keys) : "scc");
    }
};

// Accumulators of such products, for others to read from here on: no product moves behind the wait and no reader ahead of it, which is
// longer than the 19 states that the longest product takes.
template <int N> __device__ __forceinline__ void settle(f32x16 (&a)[2][N], f32x16 (&b)[2][N])
{
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) asm volatile("" : "+a"(a[i / N][i % N]), "+a"(b[i / N][i % N]));
    asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) asm volatile("" : "+a"(a[i / N][i % N]), "+a"(b[i / N][i % N]));
}

template <typename T, int D>
__global__ void __launch_bounds__(kChainWaves * 64, 1)
sdpa_bwd_chain_kernel(const ChainArgs by_value)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    using vec4 = typename E::vec4;
    using G = BwdGeom<D>;
    using C = BwdChainGeom<D>;
    constexpr int NW = kChainWaves, KEYS = kChainKeys, TS = 32;
    constexpr int KK = D / 16, DB = D / 32, U = C::U, TILE = C::TILE, SLOT = C::SLOT, PARTS = C::PARTS;
    constexpr int ROW16 = G::bytes(16);
    constexpr int TILE_FLOATS = TS * D, TILE_BYTES = TS * G::GROW;
    constexpr int NLD = 2 * U / NW;               // load instructions per wavefront and tile
    constexpr bool SMALL = D != 128;              // dQ in 16 x 16 blocks
    static_assert(2 * U % NW == 0 && KK >= 4, "");

    typedef const __attribute__((address_space(4))) ChainArgs *args_ptr;
    args_ptr args = (args_ptr)__builtin_amdgcn_kernarg_segment_ptr();

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    TSDPA_LDS int *const s_work = (TSDPA_LDS int *)(lds + C::LDS_BYTES - 16);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (;;) {
        asm volatile("" : "+s"(args));
        const int S = args->S, nB = args->nB, group = args->group, causal = args->causal;
        const int nT = (S + TS - 1) / TS;
        // ---- the next block of keys: tickets of an XCD run through its claims, per_claim heads each, block after block and within
        // a block number head after head
        if (tid == 0) {
            unsigned xcd;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(xcd));
            const unsigned per_claim = args->per_claim, per_slot = per_claim * nB;
            const unsigned t = __hip_atomic_fetch_add(&args->queue->xcd[xcd].ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned slot = t / per_slot, idx = t - slot * per_slot;
            unsigned *at = args->claims + xcd * (unsigned)args->max_slots + slot;
            unsigned claim;
            if (idx == 0) {
                claim = __hip_atomic_fetch_add(&args->queue->next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
                __hip_atomic_store(at, claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                while ((claim = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) __builtin_amdgcn_s_sleep(8);
            }
            claim -= 1;
            const unsigned h = claim * per_claim + idx % per_claim;
            *s_work = claim >= (unsigned)args->nclaims ? -1 : h >= (unsigned)args->HK ? -2 : (int)(h * (unsigned)nB + idx / per_claim);
        }
        __syncthreads();
        const int work = __builtin_amdgcn_readfirstlane(*s_work);
        if (work == -1) return;                   // no claims left
        __syncthreads();
        if (work == -2) continue;                 // (the last claim may have fewer heads)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const int head = work / nB, b = work - head * nB;
        // (what depends on the lane is made anew for every block, or it would live in registers across the loop)
        int lane = tid & 63;
        TSDPA_OPAQUE(lane);
        const int g = lane >> 5, l32 = lane & 31, g16 = lane >> 4, l16 = lane & 15;

        const int r0 = b * KEYS, w0 = r0 + wave * 64;            // first key of the block, of the wavefront
        const size_t head_off = (size_t)head * (size_t)S * D;
        // ---- K of the block into the LDS, V of the wavefront's 64 keys into registers (rows >= S: zeros)
        {
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)args->k + head_off), (short)0, S * G::GROW, 0x00020000);
#pragma unroll
            for (int u = 0; u < 2 * U; ++u) {
                const int p = u % U * 64 + lane, r = p / G::CPR, cp = p % G::CPR;
                lds_load16(rsrc, lds0 + (wave * 2 + u / U) * TILE + u % U * G::UNIT, r * G::GROW + ((cp ^ G::swz(r)) << 4), (w0 + u / U * 32) * G::GROW);
            }
        }
        vec8 vf[2][KK];
        {
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const T *)args->v + head_off), (short)0, S * G::GROW, 0x00020000);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
                    vf[kb][kk] = __builtin_bit_cast(vec8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, l32 * G::GROW + g * 16, (w0 + kb * 32) * G::GROW + kk * 32, 0));
        }
        const int j0 = causal ? r0 / TS : 0;      // query tiles nT - 1 ... j0
        const size_t shead0 = (size_t)head * group;
        const T *const t1 = (const T *)args->q + shead0 * (size_t)S * D, *const t2 = (const T *)args->dout + shead0 * (size_t)S * D;
        auto t1_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)t1, (short)0, S * G::GROW, 0x00020000);
        auto t2_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)t2, (short)0, S * G::GROW, 0x00020000);
        // statistics (-Delta of all heads, then LSE, 32 rows per tile) and sums of the group's query heads, tile after tile
        const int tiles = group * nT;
        const auto stat_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)args->stats + shead0 * nT * 128), (short)0,
                                                                 (int)(args->stat_bytes + tiles * 128u), 0x00020000);
        const auto part_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(args->part + shead0 * (size_t)(nT * TILE_FLOATS)), (short)0, tiles * TILE_FLOATS * 4, 0x00020000);
        // global offsets of the lane in load i: unit 4 i + wave of the pair Q, dO (D = 128: the same in every unit)
        constexpr int NGO = D == 96 ? NLD : 1;
        int goff[NGO];
#pragma unroll
        for (int i = 0; i < NGO; ++i) {
            const int p = (D == 128 ? 0 : (i * NW + wave) % U) * 64 + lane, r = p / G::CPR, cp = p % G::CPR;
            goff[i] = r * G::GROW + ((cp ^ G::swz(r)) << 4);
            TSDPA_OPAQUE(goff[i]);
        }
        int stat_goff = (lane >= 32 ? 0 : (int)args->stat_bytes) + (lane & 31) * 4;      // LSE, then -Delta
        TSDPA_OPAQUE(stat_goff);
        int lane16 = lane * 16;
        TSDPA_OPAQUE(lane16);
        // the tile whose loads go out next: its place in its head and among the group's tiles, its slot
        int lj = nT - 1, lh = 0, l_off = (nT - 1) * TILE_BYTES, l_tile = nT - 1;
        uint32_t l_slot = lds0 + C::SLOTS;
        auto load_part = [&](int i) __attribute__((always_inline)) {
            const int u = i * NW + wave;
            const bool first = D == 96 && i == 1 ? u < U : i < NLD / 2;
            lds_load16(first ? t1_rsrc : t2_rsrc, l_slot + u * G::UNIT, goff[NGO == 1 ? 0 : i], l_off + (D == 128 ? (u - (i < NLD / 2 ? 0 : U)) * 1024 : 0));
        };
        auto load_stats = [&]() __attribute__((always_inline)) {
            if (wave == 0) lds_load4(stat_rsrc, l_slot + 2 * TILE, stat_goff, l_tile * 128);
        };
        auto load_next = [&]() __attribute__((always_inline)) {
            l_off -= TILE_BYTES;
            --l_tile;
            l_slot = l_slot == lds0 + C::SLOTS + 2 * SLOT ? l_slot - 2 * SLOT : l_slot + SLOT;
            if (lj-- == j0) {
                if (++lh < group) {
                    lj = nT - 1;
                    l_off = (nT - 1) * TILE_BYTES;
                    l_tile += 2 * nT - j0;
                    t1_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(t1 + (size_t)lh * S * D), (short)0, S * G::GROW, 0x00020000);
                    t2_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(t2 + (size_t)lh * S * D), (short)0, S * G::GROW, 0x00020000);
                } else {
                    l_off = (nT + 2) * TILE_BYTES;        // no such tile (asked for up to three times): outside the descriptors, zeros
                    l_tile = 2;
                }
            }
        };
        f32x16 dk[2][DB], dv[2][DB];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) dk[kb][db][i] = dv[kb][db][i] = 0.f;

        // ---- LDS pointers (as in bwd_pass)
        lds_ptr row_ptr[G::NRP], k_ptr[G::NRP];
#pragma unroll
        for (int i = 0; i < G::NRP; ++i) {
            row_ptr[i] = lds + C::SLOTS + G::at(l32, 2 * G::rp_kk(i) + g);
            k_ptr[i] = lds + 2 * wave * TILE + G::at(l32, 2 * G::rp_kk(i) + g);
            TSDPA_OPAQUE(row_ptr[i]);
            TSDPA_OPAQUE(k_ptr[i]);
        }
        const int t_row = g * 4 + (l16 >> 2), t_chunk = (g16 & 1) * 2 + ((lane & 3) >> 1);
        lds_ptr tr_lo[G::NTP], tr_hi[D == 128 ? 1 : G::NTP];
#pragma unroll
        for (int i = 0; i < G::NTP; ++i) {
            tr_lo[i] = lds + C::SLOTS + G::at(t_row, i * 4 + t_chunk) + (lane & 1) * 8;
            TSDPA_OPAQUE(tr_lo[i]);
            if constexpr (D != 128) {
                tr_hi[i] = lds + C::SLOTS + G::at(t_row + 8, i * 4 + t_chunk) + (lane & 1) * 8;
                TSDPA_OPAQUE(tr_hi[i]);
            }
        }
        lds_ptr st_ptr = lds + C::SLOTS + 2 * TILE + g * 16;
        TSDPA_OPAQUE(st_ptr);
        // dQ.  D = 128: 32 columns of the wavefront, 32 queries; k-steps of 16 keys, the lane's keys g*4 ... + 3 and 8 further.  Else blocks i
        // of 16 columns `column(i)` and 16 queries `half(i)`; k-steps of 32 keys, the lane's keys g16*8 ... + 7.
        // dS in the LDS: 64 bytes (32 queries) per key, 8-byte slot s at s ^ x(key), x so that 16 or 32 lanes of a
        // transposing read (32 or 64 bytes of 4 consecutive keys) meet no bank twice, and those of a write (one slot of 32 keys) two at most.
        auto half = [&](int i) { return D == 64 ? i : wave & 1; };
        auto column = [&](int i) { return D == 64 ? wave : (wave >> 1) * 3 + i; };
        constexpr int NKP = D == 96 ? 3 : 1, NDP = D == 96 ? 1 : 2;
        lds_ptr kt_lo[NKP], kt_hi[NKP], ds_r[NDP];
        int ds_w;                                 // slot 2 * r4 + g of the lane's key: this ^ r4 << 4
        if constexpr (SMALL) {
            const int k_row = g16 * 8 + (l16 >> 2);
#pragma unroll
            for (int i = 0; i < NKP; ++i) {
                kt_lo[i] = lds + G::at(k_row, column(i) * 2 + ((lane & 3) >> 1)) + (lane & 1) * 8;
                kt_hi[i] = lds + G::at(k_row + 4, column(i) * 2 + ((lane & 3) >> 1)) + (lane & 1) * 8;
                TSDPA_OPAQUE(kt_lo[i]);
                TSDPA_OPAQUE(kt_hi[i]);
            }
#pragma unroll
            for (int i = 0; i < NDP; ++i)         // x = bit 3 of the key << 2 | bit 4 << 1
                ds_r[i] = lds + C::DS + k_row * 64 + (((half(i) * 4 + (lane & 3)) ^ ((g16 & 1) << 2 | (g16 >> 1) << 1)) << 3);
            ds_w = C::DS + (wave * 64 + l32) * 64 + ((l32 >> 3 & 1) << 5 | (l32 >> 4 & 1) << 4) + g * 8;
        } else {
            kt_lo[0] = lds + G::at(t_row, wave * 4 + t_chunk) + (lane & 1) * 8;
            TSDPA_OPAQUE(kt_lo[0]);
#pragma unroll
            for (int i = 0; i < NDP; ++i)         // x = bit 2 of the key | bit 4 << 1: even and odd k-steps
                ds_r[i] = lds + C::DS + t_row * 64 + ((((g16 & 1) * 4 + (lane & 3)) ^ g ^ i << 1) << 3);
            ds_w = C::DS + (wave * 64 + l32) * 64 + ((g ^ (l32 >> 2 & 1) ^ (l32 >> 4 & 1) << 1) << 3);
        }
        TSDPA_OPAQUE(ds_w);
#pragma unroll
        for (int i = 0; i < NDP; ++i) TSDPA_OPAQUE(ds_r[i]);

        // ---- the chain of sums: steps that the same wavefront of block b - 1 has done, counted as it publishes them
        const int n = nT - j0, steps = n * group;
        unsigned *const mine = args->progress + (((size_t)head * nB + b) * NW + wave) * kChainFlag;
        const auto flag_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(mine - (b > 0 ? NW * kChainFlag : 0)), (short)0, 4, 0x00020000);
        const int n_before = causal ? n + KEYS / TS : n;         // tiles per head of block b - 1
        unsigned seen = b == 0 ? 0xffffffffu : 0u, need = 1;
        const lds_ptr flag_ptr = lds + C::FLAGS + wave * 256;
        if (lane == 0) *(TSDPA_LDS unsigned *)flag_ptr = 0;
        const float c = args->c;
        // (block 0 reads its sums outside the descriptor: zeros)
        int p_off = (nT - 1) * TILE_FLOATS * 4 + wave * (PARTS * 1024), p_read = p_off + (b == 0 ? 1 << 30 : 0);

#pragma unroll
        for (int t = 0; t < 2; ++t) {
            load_stats();
#pragma unroll
            for (int i = 0; i < NLD; ++i) load_part(i);
            load_next();
        }
        wait_all();
        __syncthreads();
        int slot = 0, dsbuf = C::DSB;             // from this step's dS to the next one's
        int j = nT - 1, it = 0;

        // One query tile.  Vector memory operations of a step, in their order: PARTS loads of sums, the counter's store, the flag's load, the loads
        // of the tile after the next (NLD, and one of wavefront 0), PARTS stores.
        // Masks: none; the diagonal (and the end of the keys); the end of the keys, past which a lane's rows of dK and dV are garbage that is not
        // stored, so that only its dS has to be zero; the diagonal in a ragged last tile of queries, whose rows past the end have weights of zero
        // by their LSE, but a score of 0 * inf with a key of infinities.
        enum { NONE, DIAGONAL, END, TAIL };
        auto step = [&](auto mask_tag) __attribute__((always_inline)) {
            constexpr bool ROWS = decltype(mask_tag)::value == TAIL, MASK = ROWS || decltype(mask_tag)::value == DIAGONAL;
            constexpr bool LAST = decltype(mask_tag)::value == END;
            f32x16 s[2], dp[2], delta;
#pragma unroll
            for (int i = 0; i < 16; ++i) s[0][i] = s[1][i] = 0.f;
            u32x4 qf[KK], kf[2][KK], of[KK];
            f32x4 lse[4], sum[PARTS];
            auto read_q = [&](int kk) __attribute__((always_inline)) {
                qf[kk] = lds_read128(row_ptr[G::rp(kk)] + G::rp_imm(kk));
                kf[0][kk] = lds_read128(k_ptr[G::rp(kk)] + G::rp_imm(kk));
            };
            auto read_k1 = [&](int kk) __attribute__((always_inline)) { kf[1][kk] = lds_read128(k_ptr[G::rp(kk)] + G::rp_imm(kk) + TILE); };
            auto read_o = [&](int kk) __attribute__((always_inline)) { of[kk] = lds_read128(row_ptr[G::rp(kk)] + TILE + G::rp_imm(kk)); };
            auto read_lse = [&](int r4) __attribute__((always_inline)) { lse[r4] = *(TSDPA_LDS f32x4 *)(st_ptr + r4 * 32); };
            auto read_delta = [&](int r4) __attribute__((always_inline)) {
                const f32x4 md = *(TSDPA_LDS f32x4 *)(st_ptr + (TS + r4 * 8) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) delta[r4 * 4 + e] = md[e];
            };
            auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
            // ---- scores of the first 32 keys
            read_q(0);
            read_q(1);
            wait_all_but<NLD + PARTS>();          // the flag has landed
            const unsigned flag = *(TSDPA_LDS volatile unsigned *)flag_ptr;
            fence();
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (kk + 2 < KK) read_q(kk + 2);
                else read_k1(kk + 2 - KK);
                if (kk >= KK - 4) read_lse(kk - (KK - 4));
                s[0] = E::mfma(__builtin_bit_cast(vec8, qf[kk]), __builtin_bit_cast(vec8, kf[0][kk]), s[0]);
                fence();
            }
            // ---- what the blocks before have summed up for this tile
            if (seen < need) {
                seen = (unsigned)__builtin_amdgcn_readfirstlane((int)flag);
                while (seen < need) {
                    seen = (unsigned)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(mine - NW * kChainFlag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    if (seen < need) __builtin_amdgcn_s_sleep(1);
                }
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < PARTS; ++i)
                sum[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part_rsrc, lane16 + i * 1024, p_read, 0));
            fence();
            // ---- scores of the other 32 keys, and dP; the weights under these products
            u32x2 pw[2][4], xw[2][4];
            f32x4 p4[2][4];
            // queries before this one of the tile do not see the lane's key (past the end: none does)
            auto hidden = [&](int kb) __attribute__((always_inline)) -> int {
                const int key = w0 + kb * 32 + (lane & 31);
                return (key >= S ? 0x7fffffff : causal ? key : 0) - (lane >> 5) * 4;
            };
            // ... and of those that do, the first this many exist
            auto seeing = [&](int kb) __attribute__((always_inline)) -> unsigned {
                const int key = w0 + kb * 32 + (lane & 31);
                return key >= S ? 0u : causal ? S - key : S;
            };
            auto weight = [&](int kb, int r4) __attribute__((always_inline)) {
                const int lo = MASK ? hidden(kb) : 0;
                const unsigned row = ROWS ? (unsigned)(j * TS + r4 * 8) - (unsigned)lo : 0u, rows = ROWS ? seeing(kb) : 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][r4 * 4 + e], c, -lse[r4][e]));
                    p4[kb][r4][e] = (ROWS ? row + e >= rows : MASK && j * TS + r4 * 8 + e < lo) ? 0.f : p;
                }
                pw[kb][r4] = __builtin_bit_cast(u32x2, __builtin_convertvector(p4[kb][r4], vec4));
            };
            auto grad = [&](int kb, int r4) __attribute__((always_inline)) {
                const int lo = MASK ? hidden(kb) : 0;
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = p4[kb][r4][e] * dp[kb][r4 * 4 + e];
                    if (MASK && j * TS + r4 * 8 + e < lo) x[e] = 0.f;
                }
                xw[kb][r4] = __builtin_bit_cast(u32x2, __builtin_convertvector(x, vec4));
                u32x2 w = xw[kb][r4];
                if (LAST && w0 + kb * 32 + (lane & 31) >= S) w = u32x2{0u, 0u};
                *(TSDPA_LDS u32x2 *)(lds + (ds_w ^ (r4 << 4)) + kb * 2048) = w;
            };
            vec8 tf[2 * DB], hf[2 * DB];
            auto both = [](i16x4 lo, i16x4 hi) __attribute__((always_inline)) -> vec8 {
                return __builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            };
            auto tr_frag = [&](int base, int i) __attribute__((always_inline)) -> vec8 {     // i = k-step * DB + db
                const int off = base + i / DB * ROW16 + G::tp_imm(i % DB), p = G::tp(i % DB);
                return both(lds_read_tr16(tr_lo[p] + off), lds_read_tr16(D == 128 ? tr_lo[p] + off + 2 * G::UNIT : tr_hi[D == 128 ? 0 : p] + off));
            };
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (kk + 2 < KK) read_k1(kk + 2);
                else read_o(kk + 2 - KK);
                if (kk < 4) read_delta(kk);
                s[1] = E::mfma(__builtin_bit_cast(vec8, qf[kk]), __builtin_bit_cast(vec8, kf[1][kk]), s[1]);
#pragma unroll
                for (int r4 = kk * 4 / KK; r4 < (kk + 1) * 4 / KK; ++r4) weight(0, r4);
                fence();
            }
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (kk + 2 < KK) read_o(kk + 2);
                dp[0] = E::mfma(__builtin_bit_cast(vec8, of[kk]), vf[0][kk], kk == 0 ? delta : dp[0]);
#pragma unroll
                for (int r4 = kk * 4 / KK; r4 < (kk + 1) * 4 / KK; ++r4) weight(1, r4);
                fence();
            }
            // the sums of the tile before have been stored (and the next tile's loads are through): block b + 1 may have them
            wait_all_but<PARTS>();
            __hip_atomic_store(mine, (unsigned)it, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (kk >= KK - 2) tf[kk - (KK - 2)] = tr_frag(TILE, kk - (KK - 2));
                dp[1] = E::mfma(__builtin_bit_cast(vec8, of[kk]), vf[1][kk], kk == 0 ? delta : dp[1]);
#pragma unroll
                for (int r4 = kk * 4 / KK; r4 < (kk + 1) * 4 / KK; ++r4) grad(0, r4);
                fence();
            }
            // ---- dV, the rest of dS under its products
            auto frag = [&](const u32x2 (&w)[4], int ks) __attribute__((always_inline)) -> vec8 {
                return __builtin_bit_cast(vec8, u32x4{w[2 * ks][0], w[2 * ks][1], w[2 * ks + 1][0], w[2 * ks + 1][1]});
            };
            // products of dV or dK with the wavefront's 64 keys.  Without the blocks of 32 that no query of the tile sees: their weights are
            // zero, which a row of infinities would turn into NaN.
            const int visible_keys = causal ? j * TS + TS - w0 : 64;
            auto add = [&](f32x16 (&acc)[2][DB], int db, vec8 a, const u32x2 (&w)[2][4], int ks) __attribute__((always_inline)) {
                if constexpr (MASK) AccMfma<T>::run(acc[0][db], acc[1][db], a, frag(w[0], ks), frag(w[1], ks), visible_keys);
                else                AccMfma<T>::run(acc[0][db], acc[1][db], a, frag(w[0], ks), frag(w[1], ks));
            };
            constexpr int KS = SMALL ? KEYS / 32 : KEYS / 16;
            vec8 qk[KS][NKP], qd[KS][SMALL ? NDP : 1];
            auto read_qk = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < NKP; ++i)
                    if constexpr (SMALL) qk[ks][i] = both(lds_read_tr16(kt_lo[i] + ks * TILE), lds_read_tr16(kt_hi[i] + ks * TILE));
                    else qk[ks][i] = both(lds_read_tr16(kt_lo[i] + ks * ROW16), lds_read_tr16(kt_lo[i] + ks * ROW16 + 2 * G::UNIT));
            };
            auto read_qd = [&](int ks) __attribute__((always_inline)) {
                if constexpr (SMALL) {
#pragma unroll
                    for (int i = 0; i < NDP; ++i) qd[ks][i] = both(lds_read_tr16(ds_r[i] + ks * 2048), lds_read_tr16(ds_r[i] + ks * 2048 + 256));
                } else {
                    qd[ks][0] = both(lds_read_tr16(ds_r[ks & 1] + ks * 1024), lds_read_tr16(ds_r[ks & 1] + ks * 1024 + 512));
                }
            };
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) {
                if (i + 2 < 2 * DB) {
                    tf[i + 2] = tr_frag(TILE, i + 2);
                } else {
                    hf[i + 2 - 2 * DB] = tr_frag(0, i + 2 - 2 * DB);
                    read_qk(i + 2 - 2 * DB);
                }
                add(dv, i % DB, tf[i], pw, i / DB);
                if (i < 4) grad(1, i);
                fence();
            }
            // ---- dS of all keys is in the LDS, and so is the next tile
#pragma unroll
            for (int i = 0; i < PARTS; ++i) TSDPA_OPAQUE(sum[i]);        // (waited for here, before loads that the compiler does not count)
            __syncthreads();
            // ---- dQ and dK
            f32x16 qacc;
            if constexpr (!SMALL) {
#pragma unroll
                for (int i = 0; i < 16; ++i) qacc[i] = sum[i / 4 % PARTS][i & 3];
            }
            int visible = causal ? j * TS + TS - r0 : KEYS;      // keys of the block that a query of the tile sees
            read_qd(0);
            read_qd(1);
            lds_load4_agent(flag_rsrc, lds0 + C::FLAGS + wave * 256);
            load_stats();
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks < NLD) load_part(ks);
                if (ks + 2 < KS) {
                    read_qk(ks + 2);
                    read_qd(ks + 2);
                }
                constexpr int NDK = 4 * DB;       // dK products: key block i & 1, fragment i / 2, by pairs
#pragma unroll
                for (int i = ks * NDK / KS; i < (ks + 1) * NDK / KS; ++i)
                    if (i % 2 == 0 && i / 2 + 2 < 2 * DB) hf[i / 2 + 2] = tr_frag(0, i / 2 + 2);
                if constexpr (MASK) asm volatile("" : "+s"(visible));
                if (!MASK || ks * (KEYS / KS) < visible) {
                    if constexpr (SMALL) {
#pragma unroll
                        for (int i = 0; i < PARTS; ++i)
                            sum[i] = Elem16<T>::mfma(qk[ks][D == 96 ? i : 0], qd[ks][D == 96 ? 0 : i % NDP], sum[i]);
                    } else {
                        qacc = E::mfma(qk[ks][0], qd[ks][0], qacc);
                    }
                }
#pragma unroll
                for (int i = ks * NDK / KS; i < (ks + 1) * NDK / KS; ++i)
                    if (i % 2 == 1) add(dk, i / 2 % DB, hf[i / 2], xw, i / 2 / DB);
                if (ks == KS - 4) load_next();
                fence();
            }
            if constexpr (!SMALL) {
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[i / 4 % PARTS][i & 3] = qacc[i];
            }
            if (b == (causal ? j / (KEYS / TS) : nB - 1)) {
                // the last block that this tile sees: dQ (rows >= S fall outside the descriptor; PARTS stores, as below)
                asm volatile("" : "+s"(args));
                const float scale = args->scale;
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((T *)args->dq + (shead0 + it / n) * (size_t)S * D), (short)0, S * G::GROW, 0x00020000);
#pragma unroll
                for (int i = 0; i < PARTS; ++i) {
                    vec4 x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = (T)(sum[i][e] * scale);
                    const int at = SMALL ? (half(i) * 16 + (lane & 15)) * G::GROW + column(i) * 32 + (lane >> 4) * 8
                                         : (lane & 31) * G::GROW + wave * 64 + (lane >> 5) * 8 + i * 16;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), rsrc, at, j * TILE_BYTES, 0);
                }
            } else {
#pragma unroll
                for (int i = 0; i < PARTS; ++i)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum[i]), part_rsrc, lane16 + i * 1024, p_off, 0);
            }
            const int shift = slot == 2 ? -2 * SLOT : SLOT;
            slot = slot == 2 ? 0 : slot + 1;
#pragma unroll
            for (int i = 0; i < G::NRP; ++i) row_ptr[i] += shift;
#pragma unroll
            for (int i = 0; i < G::NTP; ++i) {
                tr_lo[i] += shift;
                if constexpr (D != 128) tr_hi[i] += shift;
            }
            st_ptr += shift;
#pragma unroll
            for (int i = 0; i < NDP; ++i) ds_r[i] += dsbuf;
            ds_w += dsbuf;
            dsbuf = -dsbuf;
            --j;
            ++it;
            ++need;
            p_off -= TILE_FLOATS * 4;
            p_read -= TILE_FLOATS * 4;
        };
        // (causal, the tiles of the last block are all on the diagonal)
        const bool end = !causal && r0 + KEYS > S;
        const int jd = causal ? j0 + KEYS / TS : j0;             // tiles from here on are behind the diagonal
        for (int h = 0; h < group; ++h) {
            if (S % TS != 0) step(std::integral_constant<int, TAIL>{});
            if (end)
                while (j >= j0) step(std::integral_constant<int, END>{});
            while (j >= jd) step(std::integral_constant<int, NONE>{});
            while (j >= j0) step(std::integral_constant<int, DIAGONAL>{});
            j = nT - 1;
            need += (unsigned)(n_before - n);
            p_off += (2 * nT - j0) * TILE_FLOATS * 4;
            p_read += (2 * nT - j0) * TILE_FLOATS * 4;
        }
        wait_all();
        __hip_atomic_store(mine, (unsigned)steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();                          // every wavefront past its last LDS read

        // ---- dK and dV, turned through the LDS
        settle(dk, dv);
        auto store = [&](const f32x16 (&acc)[DB], int kb, float factor, T *dst) __attribute__((always_inline)) {
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
                    *(TSDPA_LDS vec4 *)(ow + (lane & 31) * G::OROW + ((chunk ^ (lane & 31 & CMASK)) << 4) + (lane >> 5) * 8) = val;
                }
            constexpr int RPI = 64 / OCPR;
            const int row0 = w0 + kb * 32;
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + lane / OCPR, cc = lane % OCPR;
                const u32x4 val = lds_read128(ow + r * G::OROW + ((cc ^ (r & CMASK)) << 4));
                if (row0 + r < S && cc < G::CPR) *(u32x4 *)(dst + head_off + (size_t)(row0 + r) * D + cc * 8) = val;
            }
        };
        asm volatile("" : "+s"(args));
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            store(dk[kb], kb, args->scale, (T *)args->dk);
            store(dv[kb], kb, 1.0f, (T *)args->dv);
        }
        __syncthreads();
    }
#endif
}

// One workgroup per CU, which takes blocks until no claim is left: which XCD a workgroup runs on is known only there.  Where the
// heads that an XCD gets have fewer blocks, as many (the others would claim heads that another XCD is to have: 46 key/value heads of S = 1216 with
// eight query heads each, D = 96, 941 us instead of 660).
template <typename T, int D> int launch_bwd_chain(const BwdLaunchArgs &a, int per_claim)
{
    auto kern = sdpa_bwd_chain_kernel<T, D>;
    constexpr int lds_bytes = BwdChainGeom<D>::LDS_BYTES;
    static_assert(lds_bytes <= 160 * 1024 && kChainWaves * 32 * BwdGeom<D>::OROW <= BwdChainGeom<D>::FLAGS, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    const ChainLayout l = chain_layout(a.BH, a.group, a.S, D, per_claim);
    char *const ws = (char *)a.chain;
    unsigned *const claims = (unsigned *)(ws + kChainQueueBytes);
    BwdLaunchArgs st = a;
    st.stats = (float *)(ws + l.stats_at);
    st.stat_bytes = l.stat_bytes;
    const int err = launch_bwd_stats<T, D, true>(st, (unsigned *)ws, (int)(l.zero_bytes / 4), l.nT * 32);
    if (err != 0) return err;
    const ChainArgs args{a.q, a.k, a.v, a.dout, st.stats, a.dq, a.dk, a.dv, (float *)(ws + l.part_at), claims + (size_t)kChainXcds * l.max_slots,
                         (ChainQueue *)ws, claims, a.S, l.nB, a.BH / a.group, per_claim, l.nclaims, l.max_slots, a.causal, a.group, l.stat_bytes,
                         a.rsign ? -a.c : a.c, a.scale};
    const long long blocks = 8ll * ((l.nclaims + 7) / 8) * per_claim * l.nB;
    hipLaunchKernelGGL(kern, dim3(blocks < kChainGroups ? (unsigned)blocks : kChainGroups), dim3(kChainWaves * 64), lds_bytes, a.stream, args);
    return (int)hipGetLastError();
}

}  // namespace tsdpa
