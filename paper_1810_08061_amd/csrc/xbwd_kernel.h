// xbwd_kernel.h -- the reverse loop with its exchange of dz kept inside one XCD.
//
// The counterpart of xloop_kernel.h for the backward pass: going back, a row
// needs only its own later steps, so the rows are dealt by slot to one group
// of workgroups per XCD, each group holding all of U.  Workgroup (group, role)
// owns 16 MTU hidden units, i.e. those rows of U with all 4H gate-interleaved
// columns, in registers as MFMA A-fragments (K = 4H split over eight waves).
// Per step t, from the last one back:
//   * product waves take dz_{t+1} of the rows that ran step t + 1 (16 at a
//     time), poll it until it holds no marker, form their part of
//     dh_t = dz_{t+1} U^T, and put it in LDS;
//   * one workgroup barrier (the partial sums are double buffered);
//   * cell waves (8 rows by 8 units each) add the parts to the carried term and
//     the output sequence's gradient, apply the cell's backward, keep dz in
//     fp32 over z, publish it for the group, and carry dc and the direct term
//     in registers.
// So a step is one exchange.  (The whole-loop launch of bwdblk.hip splits the
// columns over four workgroups instead, because no CU holds 4H columns of
// enough units at H = 2048, and pays a second exchange of partial sums; all of
// it through memory.)  The cell waves are four waves of their own, which load z
// and the saved state two steps ahead (and wait, as the gate waves there do, for
// all that they have in flight before the cell's backward and before publishing);
// where U leaves no registers for a third wave per SIMD (bf16 data H > 512, 128
// registers of every wave; fp32 data H > 256, 64 beside a tile's 64 columns) the
// eight waves do both.
//
// dz is exchanged in the operand type: fp32 with fp32 data; with bf16 data
// fp16, each row's 8 units by 4 gates scaled by the power of two that brings
// their largest magnitude into [2^13, 2^14), undone after that block's MFMA.
// U in fp16 is scaled by a power of two per row (bwd.hip), undone in the cell.
// The ring of four buffers, the marker and the two store policies are those of
// xloop_kernel.h; the scales (powers of two, so the upper half of a float) have
// the same marker.  The buffers start as markers for every row; a workgroup
// that has read all of dz_{t+1} marks what it published at step t + 2.
//
// Measured (MI355X): see the table at xbwd_pick.
#pragma once

#include <type_traits>

#include "loop.h"

namespace ldyn {

struct XBwdParams {
    const void* ux;          // U in A-fragment blocks (launch_xbwd_pack)
    const float* us;         // [H] inverse scales of U's rows (fp16), or null
    float* gx;               // [rows][4H] z in, dz (fp32) out
    const float* save_h;     // [rows][H] the state each step started from
    const float* save_c;
    const float* dseq;       // [B][T][H] gradient of the output sequence, or null
    const float* d_out_h;    // [B][H]
    const float* d_out_c;    // [B][H], or null
    const int32_t* perm;
    const int32_t* offsets;
    Meta* meta;
    void* dzx;               // per group four buffers of dz, [k block][k run][row] chunks of 16 bytes
    unsigned short* dzs;     // per group four buffers of scales, [row][32-column block] (fp16 only)
    float* dh0;              // [B][H] out
    float* dc0;              // [B][H] out, or null
    unsigned* amax;          // largest |dz|, float bits (atomic maximum)
    unsigned* bar;           // [64 * (1 + g)]: group g's counter, then its mask of XCC numbers
    unsigned long long timeout_ticks;
    unsigned long long* trace;  // [T + 1][4] timestamps of workgroup 0, or null (as bwdblk.hip's)
    int B, H, T;
    int ng_shift, gsize, rg;    // as in XLoopParams
};

typedef void (*xbwd_fn)(XBwdParams);

constexpr int XB_KW = 8;     // product waves
constexpr int XB_PAUSE = 6;  // their pause after a step's barrier, in units of 64 clocks

template <typename E, int MTU, int KSW>
struct XBLayout {
    static constexpr int KPAD = XB_KW * KSW * E::KSTEP;      // padded 4H
    static constexpr int PART = XB_KW * MTU * 1024;          // one buffer of partial sums
    // more than half of a CU's LDS, so that each workgroup has a CU of its own
    static constexpr int BYTES = 84 * 1024;
    static_assert(2 * PART <= BYTES, "LDS");
    // U and a tile's columns leave the register file of three waves per SIMD:
    // eight waves, each both product and cell wave
    static constexpr bool BOTH = MTU > 1 || KSW >= 64;
    static constexpr int THREADS = BOTH ? XB_KW * 64 : (XB_KW + 4) * 64;
};

template <typename E, int MTU, int KSW, int NT, int CELL>
__global__ void __launch_bounds__((XBLayout<E, MTU, KSW>::THREADS), 1)
xbwd_kernel(XBwdParams p) {
    constexpr bool F32 = E::KPL == 1;
    constexpr bool BOTH = XBLayout<E, MTU, KSW>::BOTH;
    constexpr int CW = BOTH ? XB_KW : 4;               // cell waves
    constexpr int UB = 16 * MTU;                       // units per workgroup
    constexpr int PPT = 4 * MTU;                       // 8 x 8 pieces per row tile
    constexpr int PAIRS = (NT * PPT + CW - 1) / CW;    // pieces per cell wave
    using S = typename E::store_t;
    using LY = XBLayout<E, MTU, KSW>;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int KPAD = LY::KPAD;
    constexpr int CK = 16 / (int)sizeof(S);      // columns per 16-byte chunk
    constexpr int KB = 4 * CK;                   // columns per block
    constexpr int NB = KSW * E::KSTEP / KB;      // blocks of a wave's columns
    constexpr int NBLK = KPAD / KB;
    // A tile's blocks are loaded NBC at a time into NBUF register sets (MTU > 1:
    // all sixteen at once would spill beside the U block).
    constexpr int NBC = MTU > 1 && NB > 4 ? 4 : NB, NCH = NB / NBC, NBUF = NCH < 2 ? NCH : 2;
    static_assert(NB % NBC == 0, "whole chunks");
    static_assert(F32 || NB == KSW, "fp16: one block per K-step");
    static_assert(F32 || KSW % 2 == 0, "scales are loaded two at a time");

    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ int lds_ok, lds_local, lds_abort;

    const int tid = threadIdx.x;
    int l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng = 1 << p.ng_shift;
    const int g = blockIdx.x & (ng - 1), role = blockIdx.x >> p.ng_shift;
    const int B = p.B, H = p.H, H4 = 4 * H, RG = p.rg;
    if (g >= B) return;  // a group without rows
    const unsigned long long t_begin = wall_clock64();  // the bound of the start barrier counts from here
    const int Bg = (B - g + ng - 1) >> p.ng_shift;
    const int u0 = role * UB;
    const bool is_mma = w < XB_KW;
    const int ci = BOTH ? w : w - XB_KW;         // cell wave number (negative: none)
    const int kb0 = (w % XB_KW) * NB;            // the wave's first block
    const unsigned blk_bytes = 64u * (unsigned)RG;
    const unsigned ring = (unsigned)NBLK * blk_bytes;
    const unsigned sring = (unsigned)(RG * NBLK) * 2u;
    const __amdgpu_buffer_rsrc_t R = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<char*>(p.dzx) + (size_t)g * 4 * ring, (short)0, (int)(4u * ring), 0x00020000);
    const __amdgpu_buffer_rsrc_t Rs = __builtin_amdgcn_make_buffer_rsrc(
        F32 ? (void*)p.dzx : (void*)(reinterpret_cast<char*>(p.dzs) + (size_t)g * 4 * sring), (short)0,
        (int)(4u * sring), 0x00020000);
    if (tid == 0) lds_abort = 0x7fffffff;

    // ---- this wave's columns of the U block -> registers
    typename E::frag_t afrag[MTU][KSW];
    {
        const u32x4* const ux = static_cast<const u32x4*>(p.ux);
#pragma unroll
        for (int mt = 0; mt < MTU; ++mt)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const u32x4 v = ux[((size_t)(role * MTU + mt) * NBLK + kb0 + b) * 64 + l];
                if constexpr (F32) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) afrag[mt][4 * b + e] = __uint_as_float(v[e]);
                } else {
                    afrag[mt][b] = __builtin_bit_cast(typename E::frag_t, v);
                }
            }
    }

    // ---- cell waves: piece i is number ci + i CW: row tile, half of it (8
    // rows), 8 of the workgroup's units.  Lane l: row l >> 3, unit l & 7.
    const int npieces = ((Bg + 15) >> 4) * PPT;
    auto piece = [&](int i) __attribute__((always_inline)) { return ci + i * CW; };
    auto piece_ok = [&](int i) __attribute__((always_inline)) { return ci >= 0 && piece(i) < npieces; };
    auto piece_tile = [&](int i) __attribute__((always_inline)) { return piece(i) / PPT; };
    auto piece_row = [&](int i) __attribute__((always_inline)) {  // local row of this lane
        return piece_tile(i) * 16 + (piece(i) & 1) * 8 + (l >> 3);
    };
    auto piece_ub = [&](int i) __attribute__((always_inline)) { return (piece(i) % PPT) >> 1; };
    auto piece_unit = [&](int i) __attribute__((always_inline)) { return u0 + 8 * piece_ub(i) + (l & 7); };
    float dhc[PAIRS], dcc[PAIRS], inv_u[PAIRS];
    unsigned eoff[PAIRS], soff[PAIRS];  // this lane's dz (16 or 8 bytes) and its row block's scale
    int brow[PAIRS];
    using dev_t = std::integral_constant<int, P_SC1>;
    using loc_t = std::integral_constant<int, 0>;
    // Publishes a lane's dz (all ones: the marker) and, lane 0 of a row, its scale.
    auto put = [&](auto policy, int i, unsigned slot, u32x4 v, unsigned short sc) __attribute__((always_inline)) {
        constexpr int POL = decltype(policy)::value;
        if constexpr (F32) {
            __builtin_amdgcn_raw_buffer_store_b128(v, R, slot * ring + eoff[i], 0, POL);
        } else {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, R, slot * ring + eoff[i], 0, POL);
            if ((l & 7) == 0) __builtin_amdgcn_raw_buffer_store_b16(sc, Rs, slot * sring + soff[i], 0, POL);
        }
    };
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) {
        dhc[i] = dcc[i] = 0.f;
        inv_u[i] = 1.f;
        eoff[i] = soff[i] = 0;
        brow[i] = 0;
        if (!piece_ok(i)) continue;
        const int r = piece_row(i), u = piece_unit(i);
        if (r < Bg) {
            const int col = 4 * u;
            eoff[i] = (unsigned)(col / KB) * blk_bytes + (unsigned)(((col % KB) / CK) * RG + r) * 16u +
                      (unsigned)(col % CK) * (unsigned)sizeof(S);
            soff[i] = (unsigned)(r * NBLK + col / KB) * 2u;
            brow[i] = p.perm[(r << p.ng_shift) + g];
            if (u < H) {
                const size_t ib = (size_t)brow[i] * H + u;
                dhc[i] = p.d_out_h[ib];
                if (p.d_out_c) dcc[i] = p.d_out_c[ib];
                if (!F32) inv_u[i] = p.us[u];
            }
            for (unsigned slot = 0; slot < 4; ++slot) put(dev_t{}, i, slot, u32x4{~0u, ~0u, ~0u, ~0u}, 0xffffu);
        }
    }
    // Columns that no workgroup owns: zero in all four buffers, scale 1.
    if (role == 0) {
        const int b0 = p.gsize * UB * 4 / KB;
        for (int e = tid; e < (NBLK - b0) * 4 * RG * 4; e += LY::THREADS) {
            const unsigned slot = (unsigned)e & 3u, at = (unsigned)e >> 2;  // chunk of the buffer's tail
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, R,
                                                   slot * ring + (unsigned)b0 * blk_bytes + at * 16u, 0, P_SC1);
        }
        if constexpr (!F32) {
            for (int e = tid; e < (NBLK - b0) * RG * 4; e += LY::THREADS) {
                const unsigned slot = (unsigned)e & 3u;
                const int r = (e >> 2) % RG, b = b0 + (e >> 2) / RG;
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)0x3f80, Rs,
                                                      slot * sring + (unsigned)(r * NBLK + b) * 2u, 0, P_SC1);
            }
        }
    }

    // ---- the group's steps: its last is the last step of slot g
    const int max_len = p.meta->max_len;
    const_i32* const offs = (const_i32*)p.offsets;
    auto off_at = [&](int i) __attribute__((always_inline)) { return offs[max(min(i, max_len), 0)]; };
    int tg;  // steps of this group: active(t) > g for t < tg
    {
        int lo = 0, hi = max_len;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (offs[mid + 1] - offs[mid] > g) lo = mid + 1;
            else hi = mid;
        }
        tg = lo;
    }
    auto rows_of = [&](int act) __attribute__((always_inline)) { return max((act - g + ng - 1) >> p.ng_shift, 0); };

    // ---- start barrier of the group (as in xloop_kernel.h)
    drain_stores();
    __syncthreads();
    if (tid == 0) {
        int ok = 1, local = 1;
        if (p.gsize > 1) {
            unsigned* const cnt = p.bar + 64 * (1 + g);
            unsigned xcc;
            asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
            const unsigned seen = __hip_atomic_fetch_or(cnt + 1, 1u << (xcc & 15u), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::"v"(seen) : "memory");  // the mask before the count
            __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (unsigned)p.gsize) {
                if (wall_clock64() - t_begin > p.timeout_ticks) {
                    ok = 0;
                    __hip_atomic_fetch_or(&p.meta->status, STATUS_TIMEOUT, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            const unsigned mask = __hip_atomic_load(cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            local = (mask & (mask - 1)) == 0;
#ifdef LDYN_STRESS
            if (g & 1) local = 0;  // the diagnostic build runs both store policies
#endif
        }
        lds_ok = ok;
        lds_local = local;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(lds_ok) == 0) return;  // (no wave is past this barrier alone)
    const bool local = __builtin_amdgcn_readfirstlane(lds_local) != 0;

    // step offsets off[t - 2] .. off[t + 3], t the step; the next loaded a step ahead
    int t = tg - 1, cnt = 0;
    unsigned turn = 0;  // steps done: input slot turn mod 4, output slot one further
    int q_m2 = off_at(t - 2), q_m1 = off_at(t - 1), q_0 = off_at(t), q_1 = off_at(t + 1), q_2 = off_at(t + 2),
        q_3 = off_at(t + 3);
    const bool tr0 = p.trace && blockIdx.x == 0 && tid == 0;
    const bool tr1 = p.trace && blockIdx.x == 0 && tid == (BOTH ? 0 : XB_KW * 64);

    // ---- product waves
    u32x4 f[NBUF][NBC];
    constexpr int NSW = F32 ? 1 : KSW / 2;  // words of scales: two each
    unsigned fs[NSW];
    int seen_abort = 0x7fffffff;
    auto leaves = [&](int at) __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(seen_abort) <= at;
    };
    const bool few = F32 && RG <= 4;  // products of four rows (loop.h), by the batch as in xloop_kernel.h
    // Row tile j: the wave's part of dh_t into LDS; false where the loop ended
    // at the last barrier.
    auto product_tile = [&](int j, int rows) __attribute__((always_inline)) -> bool {
        // (lanes without a row take the tile's first: its products are not used,
        // and no row of another tile may stand in, whose slot may be marked
        // again while this tile is still read)
        const int r = j * 16 + (l & (few ? 3 : 15)), rr = r < rows ? r : j * 16;
        const unsigned slot = turn & 3u;
        const unsigned lane = slot * ring + (unsigned)kb0 * blk_bytes + (unsigned)((l >> 4) * RG + rr) * 16u;
        const unsigned slane = slot * sring + (unsigned)(rr * NBLK + kb0) * 2u;
        auto load_scales = [&]() __attribute__((always_inline)) {
            if constexpr (!F32) {
                if constexpr (KSW % 8 == 0) {
#pragma unroll
                    for (int q = 0; q < NSW; q += 4) {
                        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(Rs, slane, 4u * q, P_SC1);
#pragma unroll
                        for (int e = 0; e < 4; ++e) fs[q + e] = v[e];
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < NSW; ++q) fs[q] = __builtin_amdgcn_raw_buffer_load_b32(Rs, slane, 4u * q, P_SC1);
                }
            }
        };
        auto load_chunk = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < NBC; ++b)
                f[c % NBUF][b] = __builtin_amdgcn_raw_buffer_load_b128(R, lane, (unsigned)(c * NBC + b) * blk_bytes, P_SC1);
        };
        // whether a lane's part of chunk c (chunk 0: or a scale) still holds the marker
        auto incomplete = [&](int c) __attribute__((always_inline)) -> bool {
            bool m;
            if constexpr (F32) {
                unsigned x = 0;
#pragma unroll
                for (int b = 0; b < NBC; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) x = max(x, f[c % NBUF][b][e]);
                m = x == 0xffffffffu;
            } else {
                typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
                u16x2 x = {0, 0};
#pragma unroll
                for (int b = 0; b < NBC; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned d = f[c % NBUF][b][e];
                        x = __builtin_elementwise_max(x, __builtin_bit_cast(u16x2, d));
                    }
                if (c == 0) {
#pragma unroll
                    for (int q = 0; q < NSW; ++q) x = __builtin_elementwise_max(x, __builtin_bit_cast(u16x2, fs[q]));
                }
                m = x[0] == 0xffffu || x[1] == 0xffffu;
            }
            return __builtin_amdgcn_ballot_w64(m) != 0;
        };
        stress_delay(t, 1 + j);
        if constexpr (!BOTH) {  // the cell waves are still at work (see xloop_kernel.h)
            if (j == 0) __builtin_amdgcn_s_sleep(XB_PAUSE);
        }
        load_scales();
#pragma unroll
        for (int c = 0; c < NBUF; ++c) load_chunk(c);
        if (leaves(cnt - 1)) return false;
        constexpr int NACC = F32 ? 4 : MTU;  // fp32: four chains, so that an MFMA does not wait for the last
        static_assert(!F32 || MTU == 1, "fp32: one unit tile");
        f32x4_t acc[NACC];
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[a] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (incomplete(c)) {
                const unsigned long long t0 = wall_clock64();
                int tries = 0;
                do {
                    __builtin_amdgcn_s_sleep(1);
                    if (c == 0) load_scales();
                    load_chunk(c);
                    if ((++tries & 3) == 0 && wall_clock64() - t0 > p.timeout_ticks) {
                        if (l == 0) {  // past the deadline: every wave leaves after the next barrier
                            lds_abort = cnt;
                            __hip_atomic_fetch_or(&p.meta->status, STATUS_TIMEOUT, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                        }
                        break;
                    }
                } while (incomplete(c));
            }
            if constexpr (F32) {
                if (few) {
#pragma unroll
                    for (int k = 0; k < 4 * NBC; ++k)
                        acc[k & 3] = mfma_few(afrag[0][c * 4 * NBC + k], __uint_as_float(f[c % NBUF][k >> 2][k & 3]), acc[k & 3]);
                } else {
#pragma unroll
                    for (int k = 0; k < 4 * NBC; ++k)
                        acc[k & 3] = E::mfma(afrag[0][c * 4 * NBC + k], __uint_as_float(f[c % NBUF][k >> 2][k & 3]), acc[k & 3]);
                }
            } else {
#pragma unroll
                for (int b = 0; b < NBC; ++b) {
                    const int ks = c * NBC + b;
                    const unsigned sw = fs[ks / 2];
                    const float inv = __builtin_amdgcn_rcpf(
                        __uint_as_float((ks & 1) ? sw & 0xffff0000u : sw << 16));  // a power of two: exact
#pragma unroll
                    for (int mt = 0; mt < MTU; ++mt)
                        acc[mt] += E::mfma(afrag[mt][ks], __builtin_bit_cast(typename E::frag_t, f[c % NBUF][b]),
                                           f32x4_t{0.f, 0.f, 0.f, 0.f}) *
                                   inv;
                    if constexpr (MTU > 1) __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (c + NBUF < NCH) load_chunk(c + NBUF);
        }
        float* const part = lds + (cnt & 1) * (LY::PART / 4);
        if constexpr (F32) {
            acc[0] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            if (few) {  // lane l: row l & 3, units 4 (l >> 2) ..; to their place below
                acc[0] = sum_runs(acc[0]);
                if (l < 16) *reinterpret_cast<f32x4_t*>(part + ((w * 64 + (l >> 2) * 16 + (l & 3)) << 2)) = acc[0];
                return true;
            }
        }
#pragma unroll
        for (int mt = 0; mt < MTU; ++mt)
            *reinterpret_cast<f32x4_t*>(part + (((w * MTU + mt) * 64 + l) << 2)) = acc[mt];
        return true;
    };

    // ---- cell waves
    struct In {
        f32x4_t z;
        float s, ds;  // the saved state the cell needs (c, GRU: h), the sequence's gradient
    };
    In in[2][PAIRS];  // by parity of the steps done
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) in[0][i] = in[1][i] = In{f32x4_t{0.f, 0.f, 0.f, 0.f}, 0.f, 0.f};
    // The inputs of step tt (first compact row off, act rows); lanes without a
    // row or unit load another's.
    auto load_in = [&](In* dst, int tt, int off, int act) __attribute__((always_inline)) {
        const int rows = rows_of(act);
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            const int r = piece_row(i), u = piece_unit(i);
            const bool ok = piece_ok(i) && r < rows && u < H;
            const size_t row = (size_t)off + (ok ? (r << p.ng_shift) : 0) + g;
            const int uu = ok ? u : 0;
            dst[i].z = *reinterpret_cast<const f32x4_t*>(p.gx + row * H4 + 4 * uu);
            if constexpr (CELL == CELL_LSTM) dst[i].s = p.save_c[row * H + uu];
            if constexpr (CELL == CELL_GRU) dst[i].s = p.save_h[row * H + uu];
            const float* const ds = p.dseq ? p.dseq + ((size_t)brow[i] * p.T + tt) * H + uu : p.d_out_h;
            dst[i].ds = *ds;
        }
    };
    unsigned am = 0;
    // Pieces of tile j at step t (last: only dh entering step 0); have: the
    // tile has a product, for local rows below rows_p.
    auto cell_tile = [&](const In* x, int j, int rows_p, int rows_c, int rows_m, bool last) __attribute__((always_inline)) {
        const float* const part = lds + (cnt & 1) * (LY::PART / 4);
        bool drained = false;
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            if (!piece_ok(i) || piece_tile(i) != j) continue;
            const int r = piece_row(i), u = piece_unit(i);
            float dh = 0.f;
            if (j * 16 < rows_p) {
                const int uu = 8 * piece_ub(i) + (l & 7), mt = uu >> 4;
                const int at = (((uu & 15) >> 2) * 16 + (r & 15)) * 4 + (uu & 3);
                float pv[XB_KW];
#pragma unroll
                for (int ww = 0; ww < XB_KW; ++ww) pv[ww] = part[(ww * MTU + mt) * 256 + at];
#pragma unroll
                for (int span = 1; span < XB_KW; span *= 2)
#pragma unroll
                    for (int b = 0; b + span < XB_KW; b += 2 * span) pv[b] += pv[b + span];
                dh = r < rows_p ? pv[0] * inv_u[i] : 0.f;
            }
            dh += dhc[i];
            if (last) {
                if (r < Bg && u < H) {
                    p.dh0[(size_t)brow[i] * H + u] = dh;
                    if (p.dc0) p.dc0[(size_t)brow[i] * H + u] = dcc[i];
                }
                continue;
            }
            const bool live = r < rows_c;
            if (p.dseq) dh += x[i].ds;
            float dcp, dhd;
            f32x4_t dz = cell_backward<CELL>(x[i].z, x[i].s, x[i].s, dh, dcc[i], dcp, dhd);
            if (u >= H) dz = f32x4_t{0.f, 0.f, 0.f, 0.f};
            unsigned m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) m = max(m, __float_as_uint(dz[e]) & 0x7fffffffu);
            u32x4 v;
            unsigned short sc16 = 0;
            if constexpr (F32) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {  // an all-ones word (the marker) as the canonical quiet NaN
                    const unsigned d = __float_as_uint(dz[e]);
                    v[e] = d == 0xffffffffu ? 0x7fc00000u : d;
                }
                if (live) am = max(am, m);
            } else {
                // the row block's scale: its largest magnitude into [2^13, 2^14)
                m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xf, 0xf, true));   // lanes 1 0 3 2
                m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xf, 0xf, true));   // lanes 2 3 0 1
                m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xf, 0xf, true));  // mirrored in 8
                if (live) am = max(am, m);
                float sc = 1.0f;
                if (m > 0u && __uint_as_float(m) < 3.0e38f)
                    sc = __uint_as_float((unsigned)(127 + min(140 - (int)(m >> 23), 126)) << 23);
                sc16 = (unsigned short)(__float_as_uint(sc) >> 16);
                unsigned short hb[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned short b16 = __builtin_bit_cast(unsigned short, (_Float16)(dz[e] * sc));
                    hb[e] = b16 == 0xffffu ? (unsigned short)0x7e00u : b16;
                }
                v = u32x4{hb[0] | (unsigned)hb[1] << 16, hb[2] | (unsigned)hb[3] << 16, 0u, 0u};
            }
            if (!drained) {
                // the marks of the last step complete before anything is
                // published (waves that poll have waited for loads issued after them)
                if constexpr (!BOTH) drain_stores();
                drained = true;
            }
            stress_delay(t, 300 + i);
            const unsigned out = (turn + 1) & 3u, far = (turn + 3) & 3u;
            const u32x4 ones = u32x4{~0u, ~0u, ~0u, ~0u};
            // Slot far holds dz_{t+2}: this workgroup has read the tile of
            // dz_{t+1} from every workgroup of the group, so every one has
            // finished reading that tile of dz_{t+2}.
            if (local) {
                if (live) put(loc_t{}, i, out, v, sc16);
                if (r < rows_m) put(loc_t{}, i, far, ones, 0xffffu);
            } else {
                if (live) put(dev_t{}, i, out, v, sc16);
                if (r < rows_m) put(dev_t{}, i, far, ones, 0xffffu);
            }
            if (live) {
                dcc[i] = dcp;
                dhc[i] = dhd;
                if (u < H)
                    *reinterpret_cast<f32x4_t*>(p.gx + ((size_t)q_0 + (r << p.ng_shift) + g) * H4 + 4 * u) = dz;
            }
        }
    };

    // One step; false where the loop ends.  PAR: parity of the steps done; MMA:
    // a product wave (see xloop_kernel.h).
    auto step = [&](auto par, auto mma) __attribute__((always_inline)) -> bool {
        constexpr int PAR = decltype(par)::value;
        constexpr bool MMA = decltype(mma)::value;
        if (t < -1) return false;
        // values derived from the lane number (addresses) are formed again in
        // each step rather than kept live across it
        if constexpr (BOTH) asm volatile("" : "+v"(l));
        const int q_m3 = off_at(t - 3);
        const bool last = t < 0;
        const int rows_p = rows_of(q_2 - q_1);                // rows with dz_{t+1}
        const int rows_c = last ? Bg : rows_of(q_1 - q_0);    // rows that run step t
        const int rows_m = rows_of(q_3 - q_2);                // rows with dz_{t+2}
        const int tiles_p = (rows_p + 15) >> 4, tiles_c = (rows_c + 15) >> 4;
        const int ti = last ? max_len : t;
        if (tr0) p.trace[4 * ti] = wall_clock64();
        if constexpr (BOTH) {
            for (int j = 0; j < tiles_c; ++j) {
                if (j < tiles_p) {
                    if (!product_tile(j, rows_p)) return false;
                }
                if (j == 0 && t >= 1) load_in(in[PAR ^ 1], t - 1, q_m1, q_0 - q_m1);
                if (j < tiles_p) {
                    x_barrier();
                    seen_abort = lds_abort;
                }
                if (tr0 && j == 0) p.trace[4 * ti + 1] = wall_clock64();
                cell_tile(in[PAR], j, rows_p, rows_c, rows_m, last);
                if (j < tiles_p) ++cnt;
            }
            if (tr0) p.trace[4 * ti + 2] = wall_clock64();
        } else if constexpr (MMA) {
            for (int j = 0; j < tiles_p; ++j) {
                if (!product_tile(j, rows_p)) return false;
                x_barrier();
                seen_abort = lds_abort;
                if (tr0 && j == 0) p.trace[4 * ti + 1] = wall_clock64();
                ++cnt;
            }
        } else {
            for (int j = 0; NT == 1 ? j < 1 : j < tiles_c; ++j) {
                if (j < tiles_p) {
                    x_barrier();
                    seen_abort = lds_abort;
                }
                cell_tile(in[PAR], j, rows_p, rows_c, rows_m, last);
                if (j < tiles_p) {
                    if (leaves(cnt)) return false;
                    ++cnt;
                }
            }
            if (tr1) p.trace[4 * ti + 2] = wall_clock64();
            asm volatile("" ::: "memory");  // the loads stay behind the stores
            if (t >= 2) load_in(in[PAR], t - 2, q_m2, q_m1 - q_m2);
            asm volatile("" ::: "memory");
        }
        if (tr1) p.trace[4 * ti + 3] = wall_clock64();
        q_3 = q_2;
        q_2 = q_1;
        q_1 = q_0;
        q_0 = q_m1;
        q_m1 = q_m2;
        q_m2 = q_m3;
        --t;
        ++turn;
        return true;
    };
    // The cell waves' memory instructions go first: eight waves that poll fill
    // the CU's address unit, and being older they would otherwise keep the
    // stores that the other workgroups wait for out of it (for milliseconds, at
    // H = 256).
    if constexpr (!BOTH) {
        if (!is_mma) __builtin_amdgcn_s_setprio(3);
    }
    if (!is_mma || BOTH) {
        if (t >= 0) load_in(in[0], t, q_0, q_1 - q_0);
        if constexpr (!BOTH) {
            if (t >= 1) load_in(in[1], t - 1, q_m1, q_0 - q_m1);
        }
    }
    using even_t = std::integral_constant<int, 0>;
    using odd_t = std::integral_constant<int, 1>;
    if (is_mma) {
        while (step(even_t{}, std::true_type{}) && step(odd_t{}, std::true_type{})) {
        }
    } else if constexpr (!BOTH) {
        while (step(even_t{}, std::false_type{}) && step(odd_t{}, std::false_type{})) {
        }
    }
    drain_stores();
    if (ci >= 0) {
        for (int o = 32; o > 0; o >>= 1) am = max(am, (unsigned)__shfl_xor((int)am, o));
        if (l == 0 && am) atomicMax(p.amax, am);
    }
}

// A compiled variant: f[cell].
struct XBVariant {
    int bf16, mtu, ksw, nt, kpad, lds_bytes, threads;
    xbwd_fn f[3];
};
#define XBV(BF, ET, MTU, KS, NT)                                                                  \
    {BF, MTU, KS, NT, XBLayout<ET, MTU, KS>::KPAD, XBLayout<ET, MTU, KS>::BYTES,                    \
     XBLayout<ET, MTU, KS>::THREADS,                                                              \
     {xbwd_kernel<ET, MTU, KS, NT, CELL_LSTM>, xbwd_kernel<ET, MTU, KS, NT, CELL_GRU>,              \
      xbwd_kernel<ET, MTU, KS, NT, CELL_RNN>}}
#define XBV_NT(BF, ET, MTU, KS) XBV(BF, ET, MTU, KS, 1), XBV(BF, ET, MTU, KS, 2)

}  // namespace ldyn
