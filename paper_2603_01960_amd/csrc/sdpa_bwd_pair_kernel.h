// dK and dV in one pass at D = 160, by pairs of wavefronts.
//
// Both accumulators and both resident operands of a 32-key block (240 registers per lane) do not fit one wavefront beside
// scores and pointers, and with a pass per gradient scores and weights are computed twice.  Here two wavefronts
// share a block: the first has K resident and computes scores, weights P and dV^T += dO^T P, the second has V resident and
// computes dP, dS = P (dP - Delta) and dK^T += Q^T dS; P goes from the one to the other through the LDS in FP32.  Four
// products instead of five, a tile of Q and dO read once for both, and the two have even work: 20 MFMAs per 32 x 32
// scores.  The second wavefront works a tile behind (P double buffered, three slots for Q), so that one barrier per tile
// serves both and the vector work of one falls into the MFMAs of the other.
// What bounds it: the matrix pipe and the clock under its power limit on large problems, the chain of tiles where a CU holds
// four wavefronts.  BF16, us per backward call, a pass each for dK and dV -> pairs: 16 heads S = 8192 2265 -> 2002, 64 heads of
// S = 2048 606 -> 538, 64 heads over 16, S = 2048, causal 399 -> 319, two heads of S = 256 24.4 -> 17.8.
#pragma once
#include "sdpa_bwd_kernel.h"

namespace tsdpa {

template <int D, int NP, int NS> struct BwdPairGeom {
    using G = BwdGeom<D>;
    static constexpr int TS = 32, TILE = G::bytes(TS), STATS = 2 * TS * 4, PBUF = 4096;
    static constexpr int DOBASE = 3 * TILE, STBASE = 5 * TILE, PBASE = STBASE + 2 * STATS;      // of a stream
    static constexpr int STREAM = PBASE + NP * 2 * PBUF;
    static constexpr int SUMS = (NS - 1) * 2 * NP * 32 * D * 4;
    static constexpr int STAGE = 2 * NP * 32 * G::OROW;
    static constexpr int LOOP = NS * STREAM;
    static constexpr int LDS_BYTES = LOOP > SUMS ? (LOOP > STAGE ? LOOP : STAGE) : (SUMS > STAGE ? SUMS : STAGE);
};

// NP pairs of wavefronts (32 * NP resident keys) in each of NS streams, 2 * NP * NS wavefronts per workgroup; the arguments
// are those of bwd_pass, `order` that of tiles of 32 * NP keys.
template <typename T, int D, int NP, int NS, bool GRP>
__device__ __forceinline__ void
bwd_pair_pass(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
              float *__restrict__ stats, T *__restrict__ dk, T *__restrict__ dv, int S, int nR, int N, float c, float scale,
              uint32_t rsign, int causal, unsigned stat_bytes, int group, const TileOrder &order, const int block)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using E = Elem<T>;
    using vec8 = typename E::vec8;
    using vec4 = typename E::vec4;
    using G = BwdGeom<D>;
    using W = BwdPairGeom<D, NP, NS>;
    constexpr int RM = NP * 32, TS = W::TS, TILE = W::TILE;
    constexpr int U = TS * G::CPR / 64;           // units per tile of one tensor
    constexpr int NL = 2 * NP, L = (2 * U + NL - 1) / NL;         // loading wavefronts of a stream, their load instructions per tile pair
    constexpr int KK = D / 16, DB = D / 32, ROW16 = G::bytes(16);

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool second = wave_id >= NP * NS;       // of the pair (eight wavefronts: both on one SIMD)
    const int idx = second ? wave_id - NP * NS : wave_id;
    const int stream = idx / NP, pair = idx % NP;
    const lds_ptr slots = lds + stream * W::STREAM;
    const int g = lane >> 5, l32 = lane & 31;

    const int Gn = GRP ? group : 1;
    int head, rt;
    if (causal && order.heads > 0) {
        const CausalTile ct = causal_tile(block, nR, order, 0);
        head = ct.head;
        rt = ct.level;
    } else {
        const int wg = remap_workgroup(block, N, false);
        head = divide(wg, order.by_tiles);
        rt = wg - head * nR;
    }
    const size_t head_off = (size_t)head * (size_t)S * D;
    const size_t shead0 = (size_t)head * Gn;
    const T *t1 = q + shead0 * (size_t)S * D, *t2 = dout + shead0 * (size_t)S * D;

    // resident rows as MFMA B-operands: K for the first wavefront of a pair, V for the second
    const int r0 = rt * RM, rrow = r0 + pair * 32 + l32;
    const int rrow_c = rrow < S ? rrow : S - 1;
    vec8 rf[KK];
    {
        const T *res = (second ? v : k) + head_off + (size_t)rrow_c * D + g * 8;
        const uint32_t sign = second ? 0u : rsign;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            u32x4 raw = *(const u32x4 *)(res + kk * 16);
            raw ^= sign;
            rf[kk] = __builtin_bit_cast(vec8, raw);
        }
    }
    const int nT = (S + TS - 1) / TS;
    const int j0 = causal ? r0 / TS : 0, j1 = nT;
    const int tlo = causal ? rrow : 0, thi = S - 1;

    const auto stat_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)stats, (short)0, (int)(2 * stat_bytes), 0x00020000);
    const int stat_goff = (lane < TS ? (int)stat_bytes : 0) + ((int)shead0 * S + lane % TS) * 4;      // LSE rows, then -Delta rows
    auto rsrc_of = [&](const T *p, int h) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)(p + (size_t)h * S * D), (short)0, S * G::GROW, 0x00020000);
    };
    auto t1_rsrc = rsrc_of(t1, 0), t2_rsrc = rsrc_of(t2, 0);
    const int lw = (second ? NP : 0) + pair;
    int goff[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int u = i * NL + lw;
        const int p = (u < U ? u : u - U) * 64 + lane;
        const int r = p / G::CPR, cp = p % G::CPR;
        goff[i] = r * G::GROW + ((cp ^ G::swz(r)) << 4);
    }
    // load instruction i of tile j (no such tile: outside the descriptor, zeros)
    auto load_part = [&](int j, bool valid, int slot1, int slot2, int i) __attribute__((always_inline)) {
        const int soff = (valid ? j : nT) * TS * G::GROW, u = i * NL + lw;
        if (2 * U % NL != 0 && u >= 2 * U) return;
        const bool first = u < U;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(first ? t1_rsrc : t2_rsrc,
                                                 (TSDPA_LDS void *)(slots + (first ? slot1 + u * G::UNIT : W::DOBASE + slot2 + (u - U) * G::UNIT)),
                                                 16, goff[i], soff, 0, 0);
    };
    auto load_stats = [&](int row0, int slot) __attribute__((always_inline)) {
        if (lw == 0)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(stat_rsrc, (TSDPA_LDS void *)(slots + W::STBASE + slot * W::STATS), 4, stat_goff,
                                                     row0 * 4, 0, 0);
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;

    // per-lane LDS read pointers, as in bwd_pass
    lds_ptr row_ptr[G::NRP], tr_lo[G::NTP], tr_hi[G::NTP];
    static_assert(D != 128, "units of D = 128 are further apart than they are long");
#pragma unroll
    for (int i = 0; i < G::NRP; ++i) {
        row_ptr[i] = slots + G::at(l32, 2 * G::rp_kk(i) + g);
        TSDPA_OPAQUE(row_ptr[i]);
    }
    const int t_row = g * 4 + ((lane & 15) >> 2), t_chunk = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
#pragma unroll
    for (int i = 0; i < G::NTP; ++i) {
        tr_lo[i] = slots + G::at(t_row, i * 4 + t_chunk) + (lane & 1) * 8;
        tr_hi[i] = slots + G::at(t_row + 8, i * 4 + t_chunk) + (lane & 1) * 8;
        TSDPA_OPAQUE(tr_lo[i]);
        TSDPA_OPAQUE(tr_hi[i]);
    }
    const lds_ptr p_ptr = slots + W::PBASE + pair * (2 * W::PBUF) + lane * 16;
    const lds_ptr st_ptr = slots + W::STBASE + g * 16;

    // acc[i] += <T_row, R_col>, row = (i/4)*8 + g*4 + i%4 of the tile in `slot`, col = this lane's row
    auto products = [&](int slot, f32x16 &acc, auto &&after_mfma) __attribute__((always_inline)) {
        lds_ptr p[G::NRP];
#pragma unroll
        for (int i = 0; i < G::NRP; ++i) p[i] = row_ptr[i] + slot;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const u32x4 raw = lds_read128(p[G::rp(kk)] + G::rp_imm(kk));
            acc = E::mfma(__builtin_bit_cast(vec8, raw), rf[kk], acc);
            after_mfma(kk);
        }
    };
    // out^T += T^T X
    auto accumulate = [&](int slot, const vec8 (&xb)[2], auto &&after_mfma) __attribute__((always_inline)) {
        lds_ptr lo_p[G::NTP], hi_p[G::NTP];
#pragma unroll
        for (int i = 0; i < G::NTP; ++i) {
            lo_p[i] = tr_lo[i] + slot;
            hi_p[i] = tr_hi[i] + slot;
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int off = ks * ROW16 + G::tp_imm(db);
                const i16x4 lo = lds_read_tr16(lo_p[G::tp(db)] + off), hi = lds_read_tr16(hi_p[G::tp(db)] + off);
                const i16x8 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                oacc[db] = E::mfma(__builtin_bit_cast(vec8, a), xb[ks], oacc[db]);
                after_mfma(ks * DB + db);
            }
    };
    auto needs_mask = [&](int j) __attribute__((always_inline)) -> bool {
        return (j + 1) * TS > S || (causal && j * TS < r0 + RM - 1);
    };

    // ---- the tiles of this stream: every NS-th of the sequence (head of the group, tile), loads a step ahead
    const int nj = j1 - j0;
    int jn = j0 + stream, hn = 0;
    auto settle = [&]() __attribute__((always_inline)) {
        bool moved = false;
        while (jn >= j1 && hn < Gn) {
            jn -= nj;
            ++hn;
            moved = true;
        }
        if (moved && hn < Gn) {
            t1_rsrc = rsrc_of(t1, hn);
            t2_rsrc = rsrc_of(t2, hn);
        }
    };
    settle();
    load_stats(hn * S + jn * TS, 0);
#pragma unroll
    for (int i = 0; i < L; ++i) load_part(jn, hn < Gn, 0, 0, i);
    int j = jn;
    bool here = hn < Gn;
    jn += NS;
    settle();
    TSDPA_WAIT_VMCNT0();
    __syncthreads();
    const int steps = (Gn * nj + NS - 1) / NS;
    auto spread = [&](int s1, int s2, int h) __attribute__((always_inline)) {
#pragma unroll
        for (int i = h * L / KK; i < (h + 1) * L / KK; ++i) load_part(jn, hn < Gn, s1, s2, i);
        __builtin_amdgcn_sched_barrier(0x786);
    };
    int q_now = 0, q_next = TILE, q_prev = 2 * TILE;              // Q slots of this tile, the next and the one before
    auto next_step = [&]() __attribute__((always_inline)) {
        TSDPA_WAIT_VMCNT0();
        __syncthreads();
        const int free_slot = q_prev;
        q_prev = q_now;
        q_now = q_next;
        q_next = free_slot;
        j = jn;
        here = hn < Gn;
        jn += NS;
        settle();
    };
    if (!second) {
        for (int step = 0; step < steps; ++step) {
            const int odd = step & 1;
            load_stats(hn * S + jn * TS, odd ^ 1);
            if (here) {
                f32x16 acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0.f;
                __builtin_amdgcn_s_setprio(1);
                products(q_now, acc, [&](int h) __attribute__((always_inline)) { spread(q_next, odd ? 0 : TILE, h); });
                __builtin_amdgcn_s_setprio(0);
                vec8 pb[2];
                const bool mask = needs_mask(j);
                const int trow0 = j * TS + g * 4;
                auto weights = [&](auto mask_tag) __attribute__((always_inline)) {
                    constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const f32x4 l2 = *(TSDPA_LDS f32x4 *)(st_ptr + odd * W::STATS + r4 * 32);
                        f32x4 p;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int i = r4 * 4 + e, trow = trow0 + r4 * 8 + e;
                            const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i], c, -l2[e]));
                            p[e] = MASK && (trow < tlo || trow > thi) ? 0.f : x;
                            pb[i >> 3][i & 7] = (T)p[e];
                        }
                        *(TSDPA_LDS f32x4 *)(p_ptr + odd * W::PBUF + r4 * 1024) = p;
                    }
                };
                if (mask) weights(std::true_type{});
                else      weights(std::false_type{});
                __builtin_amdgcn_s_setprio(2);
                accumulate(W::DOBASE + (odd ? TILE : 0), pb, [](int) __attribute__((always_inline)) {});
                __builtin_amdgcn_s_setprio(0);
            }
            next_step();
        }
    } else {
        f32x16 dp;
        int jp = 0;
        bool prev = false;
        // dS of the tile before and its share of dK; `odd`: the parity of that tile
        auto finish = [&](int odd, int slot, auto &&after_mfma) __attribute__((always_inline)) {
            vec8 xb[2];
            const int trow0 = jp * TS + g * 4;
            auto weights = [&](auto mask_tag) __attribute__((always_inline)) {
                constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 p = *(TSDPA_LDS f32x4 *)(p_ptr + odd * W::PBUF + r4 * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = r4 * 4 + e, trow = trow0 + r4 * 8 + e;
                        const float x = p[e] * dp[i];
                        xb[i >> 3][i & 7] = (T)(MASK && (trow < tlo || trow > thi) ? 0.f : x);
                    }
                }
            };
            if (needs_mask(jp)) weights(std::true_type{});
            else                weights(std::false_type{});
            __builtin_amdgcn_s_setprio(2);
            accumulate(slot, xb, after_mfma);
            __builtin_amdgcn_s_setprio(0);
        };
        for (int step = 0; step < steps; ++step) {
            const int odd = step & 1, s2 = odd ? 0 : TILE;
            load_stats(hn * S + jn * TS, odd ^ 1);
            if (prev) {
                finish(odd ^ 1, q_prev, [&](int h) __attribute__((always_inline)) { spread(q_next, s2, h); });
            } else {
#pragma unroll
                for (int i = 0; i < L; ++i) load_part(jn, hn < Gn, q_next, s2, i);
            }
            if (here) {
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4 md = *(TSDPA_LDS f32x4 *)(st_ptr + odd * W::STATS + (TS + r4 * 8) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dp[r4 * 4 + e] = md[e];
                }
                __builtin_amdgcn_s_setprio(1);
                products(W::DOBASE + (odd ? TILE : 0), dp, [](int) __attribute__((always_inline)) {});
                __builtin_amdgcn_s_setprio(0);
            }
            jp = j;
            prev = here;
            next_step();
        }
        if (prev) finish((steps - 1) & 1, q_prev, [](int) __attribute__((always_inline)) {});
    }

    // ---- the streams' sums, in the order of the streams
    if constexpr (NS > 1) {
        __syncthreads();
        const lds_ptr at = lds + ((second ? NP : 0) + pair) * (32 * D * 4) + lane * 16;
        constexpr int DIST = 2 * NP * 32 * D * 4;
        if (stream > 0) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x4 part;
#pragma unroll
                    for (int e = 0; e < 4; ++e) part[e] = oacc[db][q4 * 4 + e];
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
                        for (int e = 0; e < 4; ++e) oacc[db][q4 * 4 + e] += part[e];
                    }
        }
    }
    __syncthreads();                              // (the region's last readers are through)
    if (NS > 1 && stream != 0) return;

    // ---- store, as in bwd_pass: dV by the first wavefront of a pair, dK by the second
    constexpr int OCPR = G::OROW / 16, CMASK = OCPR - 1;
    const lds_ptr ow = lds + ((second ? NP : 0) + pair) * (32 * G::OROW);
    const float factor = second ? scale : 1.0f;
    T *dst = (second ? dk : dv) + head_off;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            vec4 val;
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = (T)(oacc[db][q4 * 4 + e] * factor);
            *(TSDPA_LDS vec4 *)(ow + l32 * G::OROW + (((db * 4 + q4) ^ (l32 & CMASK)) << 4) + g * 8) = val;
        }
    constexpr int RPI = 64 / OCPR;
    const int row0 = r0 + pair * 32;
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = i * RPI + lane / OCPR, cc = lane % OCPR;
        const u32x4 val = lds_read128(ow + r * G::OROW + ((cc ^ (r & CMASK)) << 4));
        if (row0 + r < S && cc < G::CPR) *(u32x4 *)(dst + (size_t)(row0 + r) * D + cc * 8) = val;
    }
#endif
}

template <typename T, int D, int NP, int NS, bool GRP>
__global__ void __launch_bounds__(2 * NP * NS * 64, 2)
sdpa_bwd_pair_kernel(const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, const T *__restrict__ dout,
                     float *__restrict__ stats, T *__restrict__ dk, T *__restrict__ dv, int S, int nR, int N, float c,
                     float scale, uint32_t rsign, int causal, unsigned stat_bytes, int group, TileOrder order)
{
    bwd_pair_pass<T, D, NP, NS, GRP>(q, k, v, dout, stats, dk, dv, S, nR, N, c, scale, rsign, causal, stat_bytes, group, order,
                                     blockIdx.x);
}

template <typename T, int D, int NP, int NS, bool GRP> int launch_bwd_pair(const BwdLaunchArgs &a)
{
    auto kern = sdpa_bwd_pair_kernel<T, D, NP, NS, GRP>;
    constexpr int lds_bytes = BwdPairGeom<D, NP, NS>::LDS_BYTES;
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [&] {
        attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    });
    if (attr_err != hipSuccess) return (int)attr_err;
    const int nR = (a.S + NP * 32 - 1) / (NP * 32), heads = a.BH / a.group, N = heads * nR;
    const TileOrder order = tile_order(heads, nR, a.causal != 0, (long long)a.group * a.S * D * 2 * (long long)sizeof(T));
    hipLaunchKernelGGL(kern, dim3(N), dim3(2 * NP * NS * 64), lds_bytes, a.stream, (const T *)a.q, (const T *)a.k, (const T *)a.v,
                       (const T *)a.dout, a.stats, (T *)a.dk, (T *)a.dv, a.S, nR, N, a.c, a.scale, a.rsign, a.causal, a.stat_bytes,
                       a.group, order);
    return (int)hipGetLastError();
}

}  // namespace tsdpa
