// Decoding steps: a few query rows (at most 32, the grouped query heads' rows together) against a long cache.
//
// Such a call is bound by reading the cache once, so the kernel is built around loads: each of a workgroup's four
// wavefronts streams K/V tiles of its own (32 keys) through LDS slots of its own, with no barrier in the loop.  A
// wavefront has one slot for K and one for V and refills each as soon as it has read it into registers: the next K tile
// is requested before the scores of this one are computed, the next V tile before its output products, so that one or
// two tiles per wavefront are always in flight; eight wavefronts per CU (64-80 KiB per workgroup from D = 128) keep
// about 100 KB per CU in flight.  Scores and output are 16x16x32 MFMAs on 16 query rows (32: two of each): half the
// matrix work of the 32x32 tiles on the same rows, and half the registers.  At the end the four states (o, m, l of
// Eqs. 2-4) meet in the LDS.
// The keys of the longest entry are cut into `splits` runs of equal length, and the other entries into runs of that length;
// an entry of fewer keys has fewer runs, so that workgroups do the same work each and the long entries do not finish last.
// (Runs that are a share of the CAPACITY, as they were, leave most workgroups without keys while little of a large cache is
// filled: BF16, us, capacity 32768, such runs / these: 4 entries of 8 heads, 819 ... 3276 keys, D = 128 in pages 24.3 / 12.9, D =
// 160 34.6 / 15.3; 2457 ... 9830 keys 43.5 / 22.4, 56.3 / 28.2; 1 entry of 8 heads, 655 keys, D = 128 10.8 / 8.5; a full
// cache is level.  A share of each entry's OWN keys is level with these but for large entries of unequal length: 8192 ... 32768
// keys, D = 160 84 / 77.)
// The forward kernel, which ran these shapes before (32 x 32 tiles, all wavefronts on the same tile, a barrier per tile, one
// of its two wavefronts without rows), against this one, BF16, cold cache, us per call with the states' combination:
// 8 key/value heads of 1024 keys 11.5 / 7.9, of 8192 keys 14.2 / 13.3; 32 heads of 8192 keys 34.1 / 27.5; 96 heads of 3000
// keys at D = 96 36.4 / 24.2; 256 heads of 2048 keys 51.3 / 48.4 and of 200 ... 2048 keys 35.1 / 29.6; 256 heads of 8192
// keys 187 / 177 (6.06 TB/s), of 2048 ... 8192 keys in pages 135.6 / 127.8.
#pragma once
#include "sdpa_fwd_kernel.h"
#include "sdpa_fwd_launch.h"

namespace tsdpa {

constexpr int kDecodeTile = 32;                   // keys per tile

// LDS layout of a K or V tile: 32 rows of D values, unpadded; 16-byte chunks are permuted within each row.
//   K (16 lanes read one chunk of 16 consecutive rows): as in the forward kernel.
//   V (the transposing read has 32 lanes fetch the same 32 bytes of 8 consecutive rows): 32-byte block b of row r at
//   b ^ vx(r), which puts eight consecutive rows on eight different 32-byte slots of the 256 bytes of the banks.
template <int D> struct DecodeGeom {
    static constexpr int ROW = D * 2, CPR = D / 8;
    static constexpr int TILE = kDecodeTile * ROW;
    static constexpr int UNITS = D / 16;          // direct-to-LDS load instructions (1 KiB each) per tile
    static __host__ __device__ constexpr int kswz(int r) { return TileGeom<D, 32>::kswz(r); }
    static __host__ __device__ constexpr int vx(int r) { return D == 128 ? ((r & 3) << 1) | ((r >> 2) & 1) : D == 64 ? (r >> 1) & 3 : (r >> 2) & 1; }
    static constexpr int KP = D == 128 ? 4 : D == 64 ? 2 : CPR / 4;       // the lanes' offsets of K repeat every KP units
    static constexpr int VP = D == 128 ? 2 : D == 64 ? 1 : CPR / 4;       // ... of V every VP
    static constexpr int NKP = D == 128 ? 4 : D == 64 ? 2 : 1;            // row pointers: one per 64-byte step ks (or immediates)
    static constexpr int NVP = D == 128 ? 8 : D == 64 ? 4 : 2;            // transposing pointers: one per 32-byte block db (or per parity)
};

// The operand reads of one tile and the wait for them, in ONE block of inline assembly each: left to the compiler, which
// cannot tell the slots apart, the first read waits for every outstanding load, the next tile's included.  (One block:
// the compiler takes an output for written when its block ends, so none may still be on its way then; outputs are early
// clobbers because the pointers are read until the last of them.)
//   keys:   x[b][ks] = 16 bytes at kptr[NKP == 1 ? 0 : ks] + b * 16 * ROW (+ ks * 64 where one pointer serves every ks)
//   values: x[db][b] = transposing read at vptr[NVP == 2 ? db & 1 : db] + b * 16 * ROW (+ (db >> 1) * 64 where two serve)
#define TSDPA_RD_K(i, a, off) "ds_read_b128 %" #i ", %" #a " offset:" #off "\n\t"
#define TSDPA_RD_V(i, a, off) "ds_read_b64_tr_b16 %" #i ", %" #a " offset:" #off "\n\t"
#define TSDPA_RD_WAIT "s_waitcnt lgkmcnt(0)"
template <int D> struct DecodeRead;
template <> struct DecodeRead<64> {
    static __device__ __forceinline__ void keys(u32x4 (&x)[2][2], const uint32_t (&p)[2])
    {
        asm volatile(TSDPA_RD_K(0, 4, 0) TSDPA_RD_K(1, 5, 0) TSDPA_RD_K(2, 4, 2048) TSDPA_RD_K(3, 5, 2048) TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1])
                     : "v"(p[0]), "v"(p[1])
                     : "memory");
    }
    static __device__ __forceinline__ void values(i16x4 (&x)[4][2], const uint32_t (&p)[4])
    {
        asm volatile(TSDPA_RD_V(0, 8, 0) TSDPA_RD_V(1, 8, 2048) TSDPA_RD_V(2, 9, 0) TSDPA_RD_V(3, 9, 2048)
                     TSDPA_RD_V(4, 10, 0) TSDPA_RD_V(5, 10, 2048) TSDPA_RD_V(6, 11, 0) TSDPA_RD_V(7, 11, 2048) TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), "=&v"(x[2][1]),
                       "=&v"(x[3][0]), "=&v"(x[3][1])
                     : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3])
                     : "memory");
    }
};
template <> struct DecodeRead<96> {
    static __device__ __forceinline__ void keys(u32x4 (&x)[2][3], const uint32_t (&p)[1])
    {
        asm volatile(TSDPA_RD_K(0, 6, 0) TSDPA_RD_K(1, 6, 64) TSDPA_RD_K(2, 6, 128) TSDPA_RD_K(3, 6, 3072)
                     TSDPA_RD_K(4, 6, 3136) TSDPA_RD_K(5, 6, 3200) TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[1][2])
                     : "v"(p[0])
                     : "memory");
    }
    static __device__ __forceinline__ void values(i16x4 (&x)[6][2], const uint32_t (&p)[2])
    {
        asm volatile(TSDPA_RD_V(0, 12, 0) TSDPA_RD_V(1, 12, 3072) TSDPA_RD_V(2, 13, 0) TSDPA_RD_V(3, 13, 3072)
                     TSDPA_RD_V(4, 12, 64) TSDPA_RD_V(5, 12, 3136) TSDPA_RD_V(6, 13, 64) TSDPA_RD_V(7, 13, 3136)
                     TSDPA_RD_V(8, 12, 128) TSDPA_RD_V(9, 12, 3200) TSDPA_RD_V(10, 13, 128) TSDPA_RD_V(11, 13, 3200)
                     TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), "=&v"(x[2][1]),
                       "=&v"(x[3][0]), "=&v"(x[3][1]), "=&v"(x[4][0]), "=&v"(x[4][1]), "=&v"(x[5][0]), "=&v"(x[5][1])
                     : "v"(p[0]), "v"(p[1])
                     : "memory");
    }
};
template <> struct DecodeRead<128> {
    static __device__ __forceinline__ void keys(u32x4 (&x)[2][4], const uint32_t (&p)[4])
    {
        asm volatile(TSDPA_RD_K(0, 8, 0) TSDPA_RD_K(1, 9, 0) TSDPA_RD_K(2, 10, 0) TSDPA_RD_K(3, 11, 0) TSDPA_RD_K(4, 8, 4096)
                     TSDPA_RD_K(5, 9, 4096) TSDPA_RD_K(6, 10, 4096) TSDPA_RD_K(7, 11, 4096) TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[1][0]), "=&v"(x[1][1]),
                       "=&v"(x[1][2]), "=&v"(x[1][3])
                     : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3])
                     : "memory");
    }
    static __device__ __forceinline__ void values(i16x4 (&x)[8][2], const uint32_t (&p)[8])
    {
        asm volatile(TSDPA_RD_V(0, 16, 0) TSDPA_RD_V(1, 16, 4096) TSDPA_RD_V(2, 17, 0) TSDPA_RD_V(3, 17, 4096)
                     TSDPA_RD_V(4, 18, 0) TSDPA_RD_V(5, 18, 4096) TSDPA_RD_V(6, 19, 0) TSDPA_RD_V(7, 19, 4096)
                     TSDPA_RD_V(8, 20, 0) TSDPA_RD_V(9, 20, 4096) TSDPA_RD_V(10, 21, 0) TSDPA_RD_V(11, 21, 4096)
                     TSDPA_RD_V(12, 22, 0) TSDPA_RD_V(13, 22, 4096) TSDPA_RD_V(14, 23, 0) TSDPA_RD_V(15, 23, 4096)
                     TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), "=&v"(x[2][1]),
                       "=&v"(x[3][0]), "=&v"(x[3][1]), "=&v"(x[4][0]), "=&v"(x[4][1]), "=&v"(x[5][0]), "=&v"(x[5][1]),
                       "=&v"(x[6][0]), "=&v"(x[6][1]), "=&v"(x[7][0]), "=&v"(x[7][1])
                     : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "v"(p[4]), "v"(p[5]), "v"(p[6]), "v"(p[7])
                     : "memory");
    }
};
template <> struct DecodeRead<160> {
    static __device__ __forceinline__ void keys(u32x4 (&x)[2][5], const uint32_t (&p)[1])
    {
        asm volatile(TSDPA_RD_K(0, 10, 0) TSDPA_RD_K(1, 10, 64) TSDPA_RD_K(2, 10, 128) TSDPA_RD_K(3, 10, 192)
                     TSDPA_RD_K(4, 10, 256) TSDPA_RD_K(5, 10, 5120) TSDPA_RD_K(6, 10, 5184) TSDPA_RD_K(7, 10, 5248)
                     TSDPA_RD_K(8, 10, 5312) TSDPA_RD_K(9, 10, 5376) TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[0][2]), "=&v"(x[0][3]), "=&v"(x[0][4]), "=&v"(x[1][0]),
                       "=&v"(x[1][1]), "=&v"(x[1][2]), "=&v"(x[1][3]), "=&v"(x[1][4])
                     : "v"(p[0])
                     : "memory");
    }
    static __device__ __forceinline__ void values(i16x4 (&x)[10][2], const uint32_t (&p)[2])
    {
        asm volatile(TSDPA_RD_V(0, 20, 0) TSDPA_RD_V(1, 20, 5120) TSDPA_RD_V(2, 21, 0) TSDPA_RD_V(3, 21, 5120)
                     TSDPA_RD_V(4, 20, 64) TSDPA_RD_V(5, 20, 5184) TSDPA_RD_V(6, 21, 64) TSDPA_RD_V(7, 21, 5184)
                     TSDPA_RD_V(8, 20, 128) TSDPA_RD_V(9, 20, 5248) TSDPA_RD_V(10, 21, 128) TSDPA_RD_V(11, 21, 5248)
                     TSDPA_RD_V(12, 20, 192) TSDPA_RD_V(13, 20, 5312) TSDPA_RD_V(14, 21, 192) TSDPA_RD_V(15, 21, 5312)
                     TSDPA_RD_V(16, 20, 256) TSDPA_RD_V(17, 20, 5376) TSDPA_RD_V(18, 21, 256) TSDPA_RD_V(19, 21, 5376)
                     TSDPA_RD_WAIT
                     : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[1][0]), "=&v"(x[1][1]), "=&v"(x[2][0]), "=&v"(x[2][1]),
                       "=&v"(x[3][0]), "=&v"(x[3][1]), "=&v"(x[4][0]), "=&v"(x[4][1]), "=&v"(x[5][0]), "=&v"(x[5][1]),
                       "=&v"(x[6][0]), "=&v"(x[6][1]), "=&v"(x[7][0]), "=&v"(x[7][1]), "=&v"(x[8][0]), "=&v"(x[8][1]),
                       "=&v"(x[9][0]), "=&v"(x[9][1])
                     : "v"(p[0]), "v"(p[1])
                     : "memory");
    }
};
#undef TSDPA_RD_K
#undef TSDPA_RD_V
#undef TSDPA_RD_WAIT

// PAGED: a descriptor per tile (see the forward kernel's paged variant).  HALVES: each weight multiplied as two 16-bit halves,
// see pick_halves (an instantiation of its own: the code alone costs the shortest calls 0.3 us).
template <typename T, int D, int NQ, int NW, bool PAGED, bool HALVES>
__global__ void __launch_bounds__(NW * 64, 2)
sdpa_decode_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
                   T *o, float *__restrict__ lse, int S, int heads, float c, float tau, uint32_t qsign, int causal,
                   int Skv_cap, int splits, float *ws, int rows_per_head,
                   const int *__restrict__ kv_lens, int heads_per_batch, int batches,
                   const int *__restrict__ block_table, int max_blocks, int block_shift, unsigned long long ticket)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem16<T>;
    using vec8 = typename Elem<T>::vec8;
    using vec4 = typename Elem<T>::vec4;
    using G = DecodeGeom<D>;
    constexpr int KS = D / 32, DB = D / 16, NU = G::UNITS;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = lane >> 4, l16 = lane & 15;

    // Run fastest would put the runs of one long entry next to each other; run by run, each from another head on, a CU that
    // gets several workgroups gets them from different entries.
    const int sp = blockIdx.x / heads;
    int head = blockIdx.x - sp * heads + (int)((long long)sp * heads / splits);
    if (head >= heads) head -= heads;
    int len = Skv_cap;
    int longest = len;                            // keys of the longest entry (of more than 64 entries: of this one)
    if (kv_lens != nullptr) {
        const int b = head / heads_per_batch;
        auto clamped = [&](int x) __attribute__((always_inline)) { return x < 0 ? 0 : (x < Skv_cap ? x : Skv_cap); };
        if (splits > 1 && batches > 1 && batches <= 64) {
            const int own = clamped(lane < batches ? kv_lens[lane] : 0);
            len = __builtin_amdgcn_readlane(own, b);
            // the maximum over the lanes, in the last one: within rows of 16 lanes, then across them
            longest = own;
#define TSDPA_MAX_STEP(ctrl, rows) { const int y = __builtin_amdgcn_update_dpp(0, longest, ctrl, rows, 0xf, false); longest = longest > y ? longest : y; }
            TSDPA_MAX_STEP(0x111, 0xf) TSDPA_MAX_STEP(0x112, 0xf) TSDPA_MAX_STEP(0x114, 0xf) TSDPA_MAX_STEP(0x118, 0xf)      // row_shr
            TSDPA_MAX_STEP(0x142, 0xa) TSDPA_MAX_STEP(0x143, 0xc)                                                          // row_bcast
#undef TSDPA_MAX_STEP
            longest = __builtin_amdgcn_readlane(longest, 63);
        } else {
            len = longest = clamped(kv_lens[b]);
        }
    }

    // ---- The runs' states are combined by whichever workgroup of the head is last to be done with its own, in run order
    // whoever that is.  A workgroup writes its state, waits for the writes, marks it done, and looks at all the marks of its
    // head: the last one finds them all; should two find them all, both write the same result.  Marks need no memory of
    // their own and no cleared memory: they stand in the head's part of o, which nothing else uses before the result
    // overwrites it, and a mark is the ticket of this very call, a 64-bit number that no other call has (the output of an
    // earlier replay of the same graph, or whatever else o held, equals it with probability 2^-64).
    // States and marks are written and read at agent scope, access by access: past the L2s, of which every XCD has its
    // own.  (With plain accesses and release / acquire fences every workgroup writes back and invalidates its XCD's
    // whole L2: 256 workgroups took 36 us instead of 15.)
    auto put = [](float *at, float x, float y) __attribute__((always_inline)) {
        const unsigned long long both = ((unsigned long long)__builtin_bit_cast(uint32_t, y) << 32) | __builtin_bit_cast(uint32_t, x);
        __hip_atomic_store((unsigned long long *)at, both, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    struct Pair { float x, y; };
    auto get = [](const float *at) __attribute__((always_inline)) {
        const unsigned long long both = __hip_atomic_load((unsigned long long *)at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t lo = (uint32_t)both, hi = (uint32_t)(both >> 32);
        return Pair{__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)};
    };
    auto finish = [&]() __attribute__((always_inline)) {
        unsigned long long *marks = (unsigned long long *)(o + (size_t)head * S * D);
        TSDPA_WAIT_VMCNT0();
        __syncthreads();
        typedef TSDPA_LDS float *lds_f;
        const lds_f wgt = (lds_f)lds;
        if (wave == 0) {
            if (lane == 0) (void)__hip_atomic_exchange(marks + sp, ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            TSDPA_WAIT_VMCNT0();
            bool done = true;
#pragma unroll
            for (int i = 0; i < 128; i += 64)
                if (i + lane < splits) done &= __hip_atomic_load(marks + i + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ticket;
            const bool all = __builtin_amdgcn_ballot_w64(!done) == 0;
            if (lane == 0) wgt[0] = all ? 1.f : 0.f;
        }
        __syncthreads();
        const bool last = wgt[0] != 0.f;
        __syncthreads();
        if (!last) return;
        // weights of the runs per row, then the weighted sum of their o: [splits][S] weights in the LDS
        const float *po = ws + (size_t)head * splits * S * D;
        const float *pml = ws + (size_t)heads * splits * S * D + (size_t)head * splits * S * 2;
        // one wavefront per row, a lane per run (and another 64 runs on)
        for (int row = wave; row < S; row += NW) {
            Pair st[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                st[i] = Pair{-INFINITY, 0.f};
                if (lane + i * 64 < splits) st[i] = get(pml + ((lane + i * 64) * S + row) * 2);
            }
            float M = fmaxf(st[0].x, st[1].x);
#pragma unroll
            for (int w = 1; w < 64; w <<= 1) M = fmaxf(M, __shfl_xor(M, w, 64));
            float L = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float w = st[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(st[i].x - M);
                // (a run without keys, l = 0, has left its o unwritten: marked by a negative weight; a row of NaN scores has l = NaN)
                if (lane + i * 64 < splits) wgt[(lane + i * 64) * S + row] = st[i].y == 0.f ? -1.f : w;
                L += w * st[i].y;
            }
#pragma unroll
            for (int w = 1; w < 64; w <<= 1) L += __shfl_xor(L, w, 64);
            if (lane == 0) {
                wgt[splits * S + row] = M == -INFINITY ? 0.f : 1.f / L;      // (a row that no key reaches: O = 0, LSE = -inf)
                if (lse != nullptr)
                    lse[(size_t)head * S + row] = L > 0.f ? (M + __builtin_amdgcn_logf(L)) * 0.69314718055994530942f : -INFINITY;
            }
        }
        __syncthreads();
        // Eight runs' loads in flight; the last batch, if it is not full, loads its first run again.  What bounds this part is the
        // number of round trips past the L2, so a thread has two columns where that takes all of them in one pass, and else four.
        // (The whole call in us, remainder run by run and two columns at all times -> this: 8 heads, one row of D = 64 in 7 runs 9.2 ->
        // 7.6, in 12 8.2 -> 7.4, in 8 or 16 level; 8 rows of D = 160 in 7 runs 14.7 -> 12.1; 30 heads, 4 rows of D = 128 in 7
        // 13.3 -> 12.0.  Four columns at all times cost 0.4 to 1 us at 8 and 16 runs, and several threads per four columns, which
        // share the runs, 0.3 us more up to 16.)
        auto combine = [&](auto pairs) {
            constexpr int P = pairs;
            for (int x = tid; x < S * (D / 2 / P); x += NW * 64) {
                const int row = x / (D / 2 / P);
                float sum[2 * P] = {};
                auto batch = [&](int s0, auto whole) {
                    Pair part[8][P];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float *at = po + (size_t)(whole || s0 + i < splits ? s0 + i : s0) * S * D + (size_t)x * (2 * P);
#pragma unroll
                        for (int p = 0; p < P; ++p) part[i][p] = get(at + 2 * p);
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (!whole && s0 + i >= splits) break;
                        const float w = wgt[(s0 + i) * S + row];
                        if (!(w < 0.f)) {
#pragma unroll
                            for (int p = 0; p < P; ++p) {
                                sum[2 * p] += w * part[i][p].x;
                                sum[2 * p + 1] += w * part[i][p].y;
                            }
                        }
                    }
                };
                int s0 = 0;
                for (; s0 + 8 <= splits; s0 += 8) batch(s0, std::true_type{});
                if (s0 < splits) batch(s0, std::false_type{});
                const float inv = wgt[splits * S + row];
                typedef T Out __attribute__((ext_vector_type(2 * P)));
                Out out;
#pragma unroll
                for (int c = 0; c < 2 * P; ++c) out[c] = (T)(sum[c] * inv);
                *(Out *)(o + (size_t)head * S * D + (size_t)x * (2 * P)) = out;
            }
        };
        if (S * (D / 2) <= NW * 64) combine(std::integral_constant<int, 1>{});
        else combine(std::integral_constant<int, 2>{});
    };

    // this workgroup's run of tiles: [t0, t0 + n)
    const int nT = (len + kDecodeTile - 1) / kDecodeTile;
    // (not below four tiles: one for each of four wavefronts.  Runs of a single tile, six entries of 8 heads and 12 rows with 25
    // ... 102 keys each: 14.0 us against 12.6 at D = 160, 10.5 against 9.7 at D = 64)
    int run = ((longest + kDecodeTile - 1) / kDecodeTile + splits - 1) / splits;
    if (run < 4) run = 4;
    const int t0 = sp * run;
    int n = nT - t0 < run ? nT - t0 : run;
    if (n < 0) n = 0;
    if (n == 0 && splits > 1) {                   // nothing to read: the state of no keys (the merge does not look at o then)
        if (tid < S) {
            put(ws + (size_t)heads * splits * S * D + ((size_t)(head * splits + sp) * S + tid) * 2, -INFINITY, 0.f);
        }
        if (ticket != 0) finish();
        return;
    }

    // ---- tiles: HBM -> LDS.  Wavefront w takes the tiles w, w + 4, ... of the run, the run entered at a tile that depends on
    // the workgroup: heads of a dense cache lie a power of two apart, and workgroups in step at the same distance from their
    // start would keep hitting the same memory channels.
    const lds_ptr kslot = lds + wave * 2 * G::TILE, vslot = kslot + G::TILE;
    const size_t kv_off = (size_t)head * (size_t)Skv_cap * D;
    const auto k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(k + kv_off), (short)0, len * G::ROW, 0x00020000);
    const auto v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(v + kv_off), (short)0, len * G::ROW, 0x00020000);
    const int *pages = nullptr;
    int page_head = 0;
    if constexpr (PAGED) {
        const int b = head / heads_per_batch;
        page_head = head - b * heads_per_batch;
        pages = block_table + (size_t)b * max_blocks;
    }
    int kgoff[G::KP], vgoff[G::VP];
#pragma unroll
    for (int u = 0; u < G::KP; ++u) {
        const int p = u * 64 + lane, r = p / G::CPR, cp = p % G::CPR;
        kgoff[u] = r * G::ROW + ((cp ^ G::kswz(r)) << 4);
    }
#pragma unroll
    for (int u = 0; u < G::VP; ++u) {
        const int p = u * 64 + lane, r = p / G::CPR, cp = p % G::CPR;
        vgoff[u] = r * G::ROW + ((cp ^ (G::vx(r) << 1)) << 4);
    }
    // where a tile lies: the whole head's descriptor and an offset (past the end for "no tile": nothing is fetched, zeros
    // arrive), or a descriptor of the tile's valid rows within its page
    struct Src { decltype(k_rsrc) kr, vr; int soff; };
    auto page_of = [&](int tile) __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(pages[(tile * kDecodeTile) >> block_shift]);
    };
    auto src_of = [&](int tile, bool valid, int page) __attribute__((always_inline)) {
        if constexpr (!PAGED) return Src{k_rsrc, v_rsrc, valid ? tile * G::TILE : nT * G::TILE};
        else {
            const int row0 = tile * kDecodeTile;
            int rows = valid ? len - row0 : 0;
            rows = rows < kDecodeTile ? rows : kDecodeTile;
            const size_t first = (((size_t)page * heads_per_batch + page_head) << block_shift) + (row0 & ((1 << block_shift) - 1));
            const unsigned long long byte0 = (unsigned long long)first * (unsigned long long)G::ROW;
            const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)byte0), hi = __builtin_amdgcn_readfirstlane((unsigned)(byte0 >> 32));
            const unsigned long long at = ((unsigned long long)hi << 32) | lo;
            const int bytes = __builtin_amdgcn_readfirstlane(rows * G::ROW);
            return Src{__builtin_amdgcn_make_buffer_rsrc((void *)((const char *)k + at), (short)0, bytes, 0x00020000),
                       __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)v + at), (short)0, bytes, 0x00020000), 0};
        }
    };
    auto load_k = [&](const Src &s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(s.kr, (TSDPA_LDS void *)(kslot + u * 1024), 16, kgoff[u % G::KP],
                                                     s.soff + u / G::KP * (G::KP * 1024), 0, 0);
    };
    auto load_v = [&](const Src &s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(s.vr, (TSDPA_LDS void *)(vslot + u * 1024), 16, vgoff[u % G::VP],
                                                     s.soff + u / G::VP * (G::VP * 1024), 0, 0);
    };
    const int mine = (n - wave + NW - 1) / NW;       // tiles of this wavefront (n - wave > -4)
    const int rot = n > NW ? (int)((((unsigned)blockIdx.x * 2654435761u) >> 12) % (unsigned)n) : 0;
    int cur = wave + rot;                         // within the run
    if (cur >= n) cur -= n;
    // the tile after `cur` (its index is only used while there is one)
    auto advance = [&](int x) __attribute__((always_inline)) { x += NW; return x >= n ? x - n : x; };
    // ---- Q rows as MFMA B-operands: lane holds Q[row nq*16 + l16][ks*32 + t*8 .. +7]
    vec8 qf[NQ][KS];
    int klim[NQ];                                 // key j contributes to this lane's row iff j <= klim
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        const int row = nq * 16 + l16 < S ? nq * 16 + l16 : S - 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 raw = *(const u32x4 *)(q + ((size_t)head * S + row) * D + ks * 32 + t * 8);
            raw ^= qsign;
            qf[nq][ks] = __builtin_bit_cast(vec8, raw);
        }
        klim[nq] = causal ? row % rows_per_head + len - rows_per_head : len - 1;
    }

    // the first tile's loads go out behind Q's (whose wait then leaves them on their way)
    __builtin_amdgcn_sched_barrier(0);
    int page_next = 0;                            // paged: page of this wavefront's next tile, looked up a tile ahead
    if (mine > 0) {
        if constexpr (PAGED) page_next = page_of(t0 + cur);
        const Src s = src_of(t0 + cur, true, page_next);
        load_k(s);
        load_v(s);
        if constexpr (PAGED) page_next = page_of(mine > 1 ? t0 + advance(cur) : t0);
    }

    f32x4 oacc[NQ][DB];
    float m_ref[NQ], l_run[NQ];                   // as in the forward kernel: the lazy reference, this lane's share of the normaliser
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        m_ref[nq] = klim[nq] >= t0 * kDecodeTile ? kNoWeight : -INFINITY;
        l_run[nq] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[nq][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float lazy_limit = __builtin_amdgcn_exp2f(tau);

    // ---- pointers of the operand reads
    uint32_t kptr[G::NKP], vptr[G::NVP];
#pragma unroll
    for (int i = 0; i < G::NKP; ++i)
        kptr[i] = __builtin_bit_cast(uint32_t, kslot) + l16 * G::ROW + (((4 * i + t) ^ G::kswz(l16)) << 4);
    const int v_row = 4 * t + (l16 >> 2);
#pragma unroll
    for (int i = 0; i < G::NVP; ++i)
        vptr[i] = __builtin_bit_cast(uint32_t, vslot) + v_row * G::ROW + ((i ^ G::vx(v_row)) << 5) + (lane & 3) * 8;

    // weights of one tile and their sum, this lane's share
    vec8 pb[NQ], ph[NQ];                          // (HALVES: half of each, rounded, and what that leaves of it)
    auto exponentials = [&](const f32x4 (&s)[2], int nq, int key0) __attribute__((always_inline)) {
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][e], c, -m_ref[nq]));
                if (key0 + b * 16 + e > klim[nq]) p = 0.f;
                sum += p;
                pb[nq][b * 4 + e] = (T)(HALVES ? 0.5f * p : p);
                if constexpr (HALVES) ph[nq][b * 4 + e] = (T)(p - (float)pb[nq][b * 4 + e]);
            }
        return sum;
    };

    for (int i = 0; i < mine; ++i) {
        const int next = advance(cur);
        const bool more = i + 1 < mine;
        const Src s = src_of(t0 + next, more, page_next);
        if constexpr (PAGED) page_next = page_of(i + 2 < mine ? t0 + advance(next) : t0);
        // K has landed when at most V's loads are outstanding
        u32x4 kf[2][KS];
        __builtin_amdgcn_s_waitcnt(0x0F70 | NU);
        DecodeRead<D>::keys(kf, kptr);
        load_k(s);
        f32x4 sacc[NQ][2];
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                sacc[nq][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) sacc[nq][b] = E::mfma(__builtin_bit_cast(vec8, kf[b][ks]), qf[nq][ks], sacc[nq][b]);
            }
        const int key0 = (t0 + cur) * kDecodeTile + t * 4;
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            float ps = exponentials(sacc[nq], nq, key0);
            if (__builtin_amdgcn_ballot_w64(!(ps <= lazy_limit)) != 0) {          // also inf (first score) and NaN
                // Eq. 2 for all rows of the wavefront: tile maximum, new reference, the rescale of Eqs. 3-4
                float mx = -INFINITY;
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (key0 + b * 16 + e <= klim[nq]) mx = fmaxf(mx, sacc[nq][b][e]);
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                const float m_tile = mx * c;
                const bool grow = m_tile > m_ref[nq];      // (a row without finite scores so far: -inf or NaN, left alone)
                const float alpha = grow ? __builtin_amdgcn_exp2f(m_ref[nq] - m_tile) : 1.f;
                m_ref[nq] = grow ? m_tile : m_ref[nq];
                l_run[nq] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int e = 0; e < 4; ++e) oacc[nq][db][e] *= alpha;
                ps = exponentials(sacc[nq], nq, key0);
            }
            l_run[nq] += ps;
        }
        // V has landed when at most the next K's loads are outstanding
        i16x4 vf[DB][2];
        __builtin_amdgcn_s_waitcnt(0x0F70 | NU);
        DecodeRead<D>::values(vf, vptr);
        load_v(s);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const i16x8 a = __builtin_shufflevector(vf[db][0], vf[db][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int nq = 0; nq < NQ; ++nq) {
                oacc[nq][db] = E::mfma(__builtin_bit_cast(vec8, a), pb[nq], oacc[nq][db]);
                if constexpr (HALVES) oacc[nq][db] = E::mfma(__builtin_bit_cast(vec8, a), ph[nq], oacc[nq][db]);
            }
        }
        cur = next;
    }

    // ---- the four wavefronts' states, over the LDS (no load may still be on its way into it)
    TSDPA_WAIT_VMCNT0();
    __syncthreads();
    typedef TSDPA_LDS float *lds_f;
    const lds_f mem = (lds_f)lds;
    float wgt[NQ];                                // this wavefront's weight 2^(m - M)
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        float l = l_run[nq];
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        if (t == 0) {
            mem[((wave * NQ + nq) * 16 + l16) * 2] = m_ref[nq];
            mem[((wave * NQ + nq) * 16 + l16) * 2 + 1] = l;
        }
    }
    __syncthreads();
    float M[NQ], L[NQ];
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        M[nq] = -INFINITY;
        L[nq] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) M[nq] = fmaxf(M[nq], mem[((w * NQ + nq) * 16 + l16) * 2]);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float m = mem[((w * NQ + nq) * 16 + l16) * 2];
            L[nq] += (m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M[nq])) * mem[((w * NQ + nq) * 16 + l16) * 2 + 1];
        }
        wgt[nq] = m_ref[nq] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref[nq] - M[nq]);
        // one split: the division by the normaliser on the way (no key at all: O = 0)
        if (splits == 1) wgt[nq] *= M[nq] == -INFINITY ? 0.f : 1.f / L[nq];
    }
    __syncthreads();
    // [wave][row][D] floats
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq)
        if (nq * 16 + l16 < S)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                f32x4 part;
#pragma unroll
                for (int e = 0; e < 4; ++e) part[e] = oacc[nq][db][e] * wgt[nq];
                *(TSDPA_LDS f32x4 *)(lds + ((wave * NQ * 16 + nq * 16 + l16) * D + db * 16 + t * 4) * 4) = part;
            }
    __syncthreads();
    if (wave == 0 && t == 0)
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            const int row = nq * 16 + l16;
            if (row >= S) continue;
            if (splits > 1) {
                put(ws + (size_t)heads * splits * S * D + ((size_t)(head * splits + sp) * S + row) * 2, M[nq], L[nq]);
            } else if (lse != nullptr) {
                lse[(size_t)head * S + row] = L[nq] > 0.f ? (M[nq] + __builtin_amdgcn_logf(L[nq])) * 0.69314718055994530942f : -INFINITY;
            }
        }
    for (int x = tid; x < S * (D / 4); x += NW * 64) {
        f32x4 sum = *(TSDPA_LDS f32x4 *)(lds + x * 16);
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += *(TSDPA_LDS f32x4 *)(lds + w * (NQ * 16 * D * 4) + x * 16);
        if (splits > 1) {
            float *part = ws + (size_t)(head * splits + sp) * S * D + (size_t)x * 4;
            put(part, sum[0], sum[1]);
            put(part + 2, sum[2], sum[3]);
        } else {
            vec4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (T)sum[e];
            *(vec4 *)(o + (size_t)head * S * D + (size_t)x * 4) = out;
        }
    }
    if (ticket != 0) finish();
#endif
}

template <typename T, int D, int NQ, int NW, bool PAGED, bool HALVES> int launch_decode_one(const LaunchArgs &a)
{
    auto kern = sdpa_decode_kernel<T, D, NQ, NW, PAGED, HALVES>;
    constexpr int lds_bytes = NW * 2 * DecodeGeom<D>::TILE;
    static_assert(NW * NQ * 16 * D * 4 <= lds_bytes, "the states of all wavefronts must fit");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.BH * a.splits)), dim3(NW * 64), lds_bytes, a.stream,
                       (const T *)a.q, (const T *)a.k, (const T *)a.v, (T *)a.o, a.lse, a.S, a.BH, a.c, a.tau, a.qsign, a.causal,
                       a.Skv, a.splits, a.ws, a.rows_per_head, a.kv_lens, a.heads_per_batch, a.batches, a.block_table, a.max_blocks, a.block_shift, a.ticket);
    return (int)hipGetLastError();
}

template <typename T, int D, int NQ, bool HALVES> int launch_decode_rows(const LaunchArgs &a)
{
    if (decode_waves(a.BH, a.splits, a.Skv) == 8)
        return a.block_table ? launch_decode_one<T, D, NQ, 8, true, HALVES>(a) : launch_decode_one<T, D, NQ, 8, false, HALVES>(a);
    return a.block_table ? launch_decode_one<T, D, NQ, 4, true, HALVES>(a) : launch_decode_one<T, D, NQ, 4, false, HALVES>(a);
}

template <typename T, int D> int launch_decode_dim(const LaunchArgs &a)
{
    if (a.S > 16) return launch_decode_rows<T, D, 2, false>(a);
    return a.halves ? launch_decode_rows<T, D, 1, true>(a) : launch_decode_rows<T, D, 1, false>(a);
}

template <typename T> int launch_decode(int D, const LaunchArgs &a)
{
    switch (D) {
        case 64: return launch_decode_dim<T, 64>(a);
        case 96: return launch_decode_dim<T, 96>(a);
        case 128: return launch_decode_dim<T, 128>(a);
        default: return launch_decode_dim<T, 160>(a);
    }
}

}  // namespace tsdpa
