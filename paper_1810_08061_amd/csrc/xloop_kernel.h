// xloop_kernel.h -- the time loop with its exchange of h kept inside one XCD.
//
// The rows of a batch are independent: only the hidden units of one row have
// to see each other between steps.  Where the U of a layer fits the registers
// of 32 CUs (bf16 data: H <= 1024; fp32 data: H <= 512), the grid is cut into
// one group of up to 32 workgroups per XCD, each group holds all of U, and the
// rows are dealt to the groups by slot (the slots are sorted by length, so
// every group gets long and short rows).  Then
//   * what a step waits for, the store of h by one workgroup and its load by
//     the others, goes through the XCD's own L2 and not through memory: a
//     16-row exchange of H = 512 among 32 workgroups measured 0.71 us a step
//     against 1.38 us at device scope (H = 1024: 0.75 against 1.63 us);
//   * a batch of up to 128 rows is one 16-row tile per group and step, where
//     the device-wide loop (persistent.hip) runs ceil(B / 16) tiles in turn.
// The device-wide loop remains for wider layers.
//
// Workgroup (group g, role) owns 4 MT hidden units (MT gate tiles of 16
// gate-interleaved columns of U, in registers as MFMA A-fragments, K split
// over KW waves).  Per step and 16-row tile of the group's rows:
//   * product waves load their K range of the tile of h_t, poll it until it
//     holds no marker, multiply, and put their partial sums in LDS;
//   * one workgroup barrier (the partial sums are double buffered);
//   * gate waves, one gate tile each, add the partial sums and Gx, apply the
//     cell, store their elements of h_{t+1}, and mark the buffer that will
//     take h_{t+3}.
// With KW = 4 four further waves are the gate waves: the product waves never
// store, so their polls wait for nothing but h, and the gate waves never poll.
// Those wait for all that they have in flight before the gates (Gx, loaded two
// steps ahead, in a branch, so that the compiler's wait covers the load of the
// next step too) and again before the stores of h (the marks of the last step).
// With KW = 8 (H > 512: the U slice takes 72 registers of every wave up to H = 768
// and 128 beyond) each wave is both.
//
// The exchange is the device-wide loop's: a ring of four buffers, the marker
// (all ones, never a value) in every element not yet written, loads at device
// scope (they pass by the CU's own cache).  Only the stores differ: where all
// workgroups of a group run on one XCD (each reads its XCC number at the
// start), they are plain stores, which the XCD's L2 holds; otherwise they are
// written through to memory, and the loop is correct wherever the workgroups
// run.  h lies in the buffer as [k block][k run][row of the group] chunks of 16
// bytes, so a group's ring takes no room for rows that it does not have.
//
// Measured (MI355X, whole forward, the device-wide loop and this one):
//   fp32 H 256, 32 rows, 100 steps         292 and 160 us
//   fp32 H 256, 128 full rows, 128 steps   814 and 242 us (with the sequence)
//   bf16 H 512, 64 rows, 200 steps         506 and 303 us
//   bf16 H 1024, 128 rows, 500 steps      1201 and 1034 us (most steps a few rows)
//   bf16 H 1024, 64 rows, 256 steps, stop  858 and 632 us
// What bounds a step now (H = 512, 1.3 us): the store's and the load's way
// through L2 (about 0.55 us with the wait's granularity), then 16 MFMAs, the
// partial sums through LDS and the barrier (0.4), then the gates (0.3).
#pragma once

#include <type_traits>

#include "loop.h"

namespace ldyn {

struct XLoopParams {
    const void* U;
    const void* ux;         // U in A-fragment blocks (prep.hip), or null: staged here from U
    const float* h0;
    const float* c0;
    float* out_h;
    float* out_c;
    const float* gx;
    void* hx;
    unsigned* bar;          // [64 * (1 + g)]: group g's counter, then its mask of XCC numbers
    Meta* meta;
    const int32_t* perm;
    const int32_t* offsets;
    int B, H;
    int ng_shift;           // the grid has 1 << ng_shift groups; group = blockIdx mod that
    int gsize;              // workgroups per group
    int rg;                 // rows per group, at most: ceil(B / groups)
    unsigned long long timeout_ticks;
    unsigned long long* trace;  // [T + 1][4] timestamps from workgroup 0, or null
    float* seq;                 // output sequence [B][T][H] (fp32), or null
    const float* stop_v;        // termination from the state, as in persistent.hip
    float stop_c;
    int32_t* steps;
    const int32_t* lengths;
    int T;
    float* save_h;              // forward for training, as in persistent.hip
    float* save_c;
};

typedef void (*xloop_fn)(XLoopParams);

constexpr int X_WAVES = 8;
constexpr int X_PAUSE = 6;  // product waves' pause after a step's barrier, in units of 64 clocks

// Compile-time shape of a variant.
template <typename E, int MT, int KSW, int KW>
struct XLayout {
    using S = typename E::store_t;
    static constexpr int HPAD = KW * KSW * E::KSTEP;
    static constexpr int STRIDE = HPAD + 16 / (int)sizeof(S);  // staged row of the U slice
    static constexpr int PART = KW * MT * 1024;                // one buffer of partial sums
    static constexpr int TILE = 16 * STRIDE * (int)sizeof(S);  // staged bytes of one gate tile
    static constexpr int ROOM = 140 * 1024;
    static constexpr int TP = ROOM / TILE < MT ? ROOM / TILE : MT;  // gate tiles staged at a time
    static constexpr int NEED = 2 * PART > TP * TILE ? 2 * PART : TP * TILE;
    // more than half of a CU's LDS, so that each workgroup has a CU of its own
    static constexpr int BYTES = NEED > 84 * 1024 ? NEED : 84 * 1024;
    static_assert(TP >= 1 && 2 * PART <= ROOM, "LDS");
};

template <typename E, int MT, int KSW, int KW, int NT, int CELL, int LMODE>
__global__ void __launch_bounds__(X_WAVES * 64, 1)
xloop_kernel(XLoopParams p) {
    constexpr bool STOP = LMODE == LM_STOP;
    constexpr bool SAVE = LMODE == LM_SAVE;
    constexpr bool BOTH = KW == X_WAVES;          // every wave multiplies and computes gates
    constexpr int GW = BOTH ? KW : X_WAVES - KW;  // gate waves
    constexpr int PAIRS = (NT * MT + GW - 1) / GW;  // (row tile, gate tile) pairs per gate wave
    using S = typename E::store_t;
    using IO = HxIO<E>;
    using LY = XLayout<E, MT, KSW, KW>;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int HPAD = LY::HPAD;
    constexpr int CK = 16 / (int)sizeof(S);     // k per 16-byte chunk
    constexpr int KB = 4 * CK;                  // k per block (four chunks of each row)
    constexpr int NB = KSW * E::KSTEP / KB;     // blocks of a wave's K range
    static_assert(NB * KB == KSW * E::KSTEP && NB >= 1, "a wave's K range is whole blocks");

    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ int lds_ok, lds_local, lds_abort, lds_run[4];
    constexpr int VST = STOP ? HPAD : 1;
    __shared__ __attribute__((aligned(16))) S vst[VST];
    __shared__ float s_part[2][STOP ? KW : 1][16];

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng = 1 << p.ng_shift;
    const int g = blockIdx.x & (ng - 1), role = blockIdx.x >> p.ng_shift;
    const int B = p.B, H = p.H, H4 = 4 * H, RG = p.rg;
    if (g >= B) return;  // a group without rows
    const unsigned long long t_begin = wall_clock64();  // the bound of the start barrier counts from here
    const int Bg = (B - g + ng - 1) >> p.ng_shift;  // rows of this group: slots g, g + ng, ...
    const int u0 = role * 4 * MT;
    const bool is_mma = w < KW;
    const int gwi = BOTH ? w : w - KW;              // gate wave number (negative: none)
    const int kw0 = (w % KW) * KSW * E::KSTEP;
    const unsigned blk_bytes = 64u * (unsigned)RG;
    const unsigned ring = (unsigned)(HPAD / KB) * blk_bytes;  // one of the four buffers
    const __amdgpu_buffer_rsrc_t R = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<char*>(p.hx) + (size_t)g * 4 * ring, (short)0, (int)(4u * ring), 0x00020000);
    // Byte offset of h[local row r][k] within one buffer.
    auto hoff = [&](int r, int k) __attribute__((always_inline)) {
        return (unsigned)(k / KB) * blk_bytes + (unsigned)(((k % KB) / CK) * RG + r) * 16u +
               (unsigned)(k % CK) * (unsigned)sizeof(S);
    };
    if (tid == 0) {
        lds_abort = 0x7fffffff;
        for (int i = 0; i < 4; ++i) lds_run[i] = 0;
    }
    if constexpr (STOP) {
        for (int k = tid; k < VST; k += X_WAVES * 64) vst[k] = E::from_f32(k < H ? p.stop_v[k] : 0.0f);
    }

    // ---- U slice -> registers: one 16-byte load per fragment (fp32: per four)
    // from the packed copy.  Without one (a caller's scratch without room for
    // it): TP gate tiles at a time through LDS, turned: ust[c'][k]; a thread
    // takes four units of one gate at one k (one 8- or 16-byte load where H is
    // a multiple of 4), lanes along k.
    typename E::frag_t afrag[MT][KSW];
    if (p.ux) {
        const u32x4* const ux = static_cast<const u32x4*>(p.ux);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const u32x4 v = ux[((size_t)(role * MT + mt) * (HPAD / KB) + kw0 / KB + b) * 64 + l];
                if constexpr (E::KPL == 1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) afrag[mt][4 * b + e] = __uint_as_float(v[e]);
                } else {
                    afrag[mt][b] = __builtin_bit_cast(typename E::frag_t, v);
                }
            }
    } else {
        using Src = typename E::src_t;
        typedef Src src4_t __attribute__((ext_vector_type(4)));
        const Src* U = static_cast<const Src*>(p.U);
        S* ust = reinterpret_cast<S*>(lds);
        const bool vec = (H & 3) == 0;
        constexpr int STRIDE = LY::STRIDE;
#pragma unroll
        for (int mt0 = 0; mt0 < MT; mt0 += LY::TP) {
            constexpr int UN = 8;
            const int tp = MT - mt0 < LY::TP ? MT - mt0 : LY::TP;
            const int items = HPAD * 4 * tp;  // a multiple of the 512 threads (HPAD is one of 128, or 64)
            for (int e0 = 0; e0 < items; e0 += X_WAVES * 64 * UN) {
                src4_t v[UN];
#pragma unroll
                for (int r = 0; r < UN; ++r) {
                    const int e = e0 + r * X_WAVES * 64 + tid;
                    const int k = e % HPAD, rest = e / HPAD, gate = rest & 3;
                    const int u = u0 + 4 * (mt0 + (rest >> 2));
                    const bool in = e < items && k < H;
                    if (vec) {
                        const size_t at = in && u < H ? (size_t)k * H4 + (size_t)gate * H + u : 0;
                        v[r] = *reinterpret_cast<const src4_t*>(U + at);
                        if (!(in && u < H)) v[r] = src4_t{(Src)0.0f, (Src)0.0f, (Src)0.0f, (Src)0.0f};
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const bool ok = in && u + q < H;
                            const Src s = U[ok ? (size_t)k * H4 + (size_t)gate * H + u + q : 0];
                            v[r][q] = ok ? s : (Src)0.0f;
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < UN; ++r) {
                    const int e = e0 + r * X_WAVES * 64 + tid;
                    const int k = e % HPAD, rest = e / HPAD, gate = rest & 3, uu = 4 * (rest >> 2);
                    if (e < items)
#pragma unroll
                        for (int q = 0; q < 4; ++q) ust[(4 * (uu + q) + gate) * STRIDE + k] = E::from_src(v[r][q]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (mt < mt0 || mt >= mt0 + LY::TP) continue;
#pragma unroll
                for (int ks = 0; ks < KSW; ++ks)
                    afrag[mt][ks] = E::load(ust + ((mt - mt0) * 16 + (l & 15)) * STRIDE + kw0 + kslot<E, KSW>(ks, l));
            }
            __syncthreads();  // the LDS is written again
        }
    }

    // ---- Owned state of the gate waves: pair i is (row tile, gate tile) number
    // gwi + i GW; lane l holds row l & 15 of the tile and unit l >> 4 of the
    // gate tile.  c and h stay in registers until the end.
    const int npairs = ((Bg + 15) >> 4) * MT;
    float cst[PAIRS], hst[PAIRS];
    unsigned eoff[PAIRS];  // the element's offset in a buffer
    int brow[PAIRS];       // batch row
    auto pair_tile = [&](int i) __attribute__((always_inline)) { return (gwi + i * GW) / MT; };
    auto pair_unit = [&](int i) __attribute__((always_inline)) { return u0 + 4 * ((gwi + i * GW) % MT) + (l >> 4); };
    auto pair_ok = [&](int i) __attribute__((always_inline)) { return gwi >= 0 && gwi + i * GW < npairs; };
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) {
        cst[i] = 0.f;
        hst[i] = 0.f;
        eoff[i] = 0;
        brow[i] = 0;
        if (!pair_ok(i)) continue;
        const int r = pair_tile(i) * 16 + (l & 15), u = pair_unit(i);
        if (r < Bg) {
            eoff[i] = hoff(r, u);
            brow[i] = p.perm[(r << p.ng_shift) + g];
            if (u < H) {
                const size_t ib = (size_t)brow[i] * H + u;
                hst[i] = p.h0[ib];  // read before the final write: exact aliasing out_h == h0 is allowed
                if constexpr (CELL == CELL_LSTM) cst[i] = p.c0[ib];
            }
            IO::template store<P_SC1>(R, eoff[i], hst[i]);  // (padding units: zero)
            if constexpr (STOP) {
                // a row that never ends early runs to its cap
                if (role == 0 && (gwi + i * GW) % MT == 0 && l < 16)
                    p.steps[brow[i]] = min(max(p.lengths[brow[i]], 0), p.T);
            }
        }
    }
    // Columns that no workgroup owns (the K range is padded further than the
    // group's units): zero in all four buffers, for good.
    if (role == 0) {
        const int kpad = HPAD - p.gsize * 4 * MT;
        for (int e = tid; e < kpad * RG * 4; e += X_WAVES * 64) {
            const int b = e & 3, r = (e >> 2) % RG, k = p.gsize * 4 * MT + (e >> 2) / RG;
            IO::template store<P_SC1>(R, (unsigned)b * ring + hoff(r, k), 0.0f);
        }
    }

    // Offsets of steps t .. t + 3 travel in scalar registers.
    const int max_len = p.meta->max_len;
    const_i32* const offs = (const_i32*)p.offsets;
    auto offset_at = [&](int t) __attribute__((always_inline)) { return offs[min(t, max_len)]; };
    int o0 = offset_at(0), o1 = offset_at(1), o2 = offset_at(2), o3 = offset_at(3);
    auto rows_of = [&](int act) __attribute__((always_inline)) { return max((act - g + ng - 1) >> p.ng_shift, 0); };  // of this group

    // The elements of this wave's pairs in one buffer, rows [0, rows): not yet written.
    auto mark = [&](auto policy, int i, unsigned part, int rows) __attribute__((always_inline)) {
        const int r = pair_tile(i) * 16 + (l & 15);
        if (r < rows) IO::template mark<decltype(policy)::value>(R, part + eoff[i]);
    };
    using dev_t = std::integral_constant<int, P_SC1>;
    using loc_t = std::integral_constant<int, 0>;
#pragma unroll
    for (int i = 0; i < PAIRS; ++i)
        if (pair_ok(i)) {
            mark(dev_t{}, i, ring, rows_of(o2 - o1));
            mark(dev_t{}, i, 2u * ring, rows_of(o3 - o2));
        }

    // Gx[tt] of this wave's pairs (tt a step this group runs); lanes without a
    // row or unit load another's, which is not used.
    auto load_gx = [&](f32x4_t* dst, int off, int act) __attribute__((always_inline)) {
        const int rows = rows_of(act);
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            const int r = pair_tile(i) * 16 + (l & 15), u = pair_unit(i);
            const bool ok = pair_ok(i) && r < rows && u < H;
            const size_t row = (size_t)off + (ok ? (r << p.ng_shift) : 0) + g;
            dst[i] = *reinterpret_cast<const f32x4_t*>(p.gx + row * H4 + (ok ? 4 * u : 0));
        }
    };
    f32x4_t gxr[2][PAIRS];  // by step parity
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) gxr[0][i] = gxr[1][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // ---- Start: h_0 and the first marks visible to the group.  One counter
    // barrier per group; on the way each workgroup adds its XCC number to the
    // group's mask, which tells whether the group sits on one XCD.
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
    const bool alive = __builtin_amdgcn_readfirstlane(lds_ok) != 0;
    const bool local = __builtin_amdgcn_readfirstlane(lds_local) != 0;

    // ---- one row tile's product: this wave's partial sums into LDS
    // (cnt counts the tiles; it numbers the barriers and picks the LDS buffer)
    int t = 0, cnt = 0, iters = 0;
    unsigned stopped = 0;  // STOP: bit i set once the lane's row of pair i has ended
    const bool tr0 = p.trace && blockIdx.x == 0 && tid == 0;
    const bool tr1 = p.trace && blockIdx.x == 0 && tid == (BOTH ? 0 : KW * 64);
    u32x4 f[NB];
    // whether a lane's part of the tile still holds the marker: the largest of
    // its elements as integers
    auto incomplete = [&]() __attribute__((always_inline)) -> bool {
        bool m;
        if constexpr (E::KPL == 1) {
            unsigned x = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) x = max(x, f[b][e]);
            m = x == 0xffffffffu;
        } else {
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            u16x2 x = {0, 0};
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned d = f[b][e];
                    x = __builtin_elementwise_max(x, __builtin_bit_cast(u16x2, d));
                }
            m = x[0] == 0xffffu || x[1] == 0xffffu;
        }
        return __builtin_amdgcn_ballot_w64(m) != 0;
    };
    // The flags as they stood after barrier cnt; every wave reads them there,
    // and so all leave the loop after the same barrier (a flag set for a later
    // one holds a later number).
    int seen_abort = 0x7fffffff, seen_run = 1;
    auto read_flags = [&](int j) __attribute__((always_inline)) {
        seen_abort = lds_abort;
        if constexpr (STOP) {
            seen_run = 1;
            if (j == 0 && t > 0) {
                // some row ran at step t - 1, or none ever runs again
                seen_run = lds_run[(t - 1) & 3];
                iters = t;
            }
            if (j == 0 && tid == 0) lds_run[(t + 2) & 3] = 0;
        }
    };
    auto leaves = [&](int at) __attribute__((always_inline)) -> bool {
        bool out = __builtin_amdgcn_readfirstlane(seen_abort) <= at;
        if constexpr (STOP) out |= __builtin_amdgcn_readfirstlane(seen_run) == 0;
        return out;
    };
    // fp32, at most four rows per group: products of four rows (loop.h).  By the
    // batch, not by the rows that still run, so that every row of a batch goes
    // the same way whatever its slot.  (32 rows, H 256, 100 steps: a forward 172 ->
    // 164 us; with the reverse loop's a training step 497 -> 398, RNN H 333 364 ->
    // 295.)
    const bool few = E::KPL == 1 && RG <= 4;
    // Loads the wave's part of tile j and polls it; false where the loop ended
    // at the last barrier (known only here, so that the loads travel while the
    // flags are read).
    auto fetch_tile = [&](int j, int rows) __attribute__((always_inline)) -> bool {
        // lanes without an active row read the tile's first row instead, whose
        // products they then repeat (no row of another tile may stand in, whose
        // slot other workgroups may mark again while this tile is still read)
        const int r = j * 16 + (l & (few ? 3 : 15));
        const unsigned lane = (unsigned)(t & 3) * ring + (unsigned)(kw0 / KB) * blk_bytes +
                              (unsigned)((l >> 4) * RG + (r < rows ? r : j * 16)) * 16u;
        stress_delay(t, 1 + j);
        auto load_all = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
                f[b] = __builtin_amdgcn_raw_buffer_load_b128(R, lane, (unsigned)b * blk_bytes, P_SC1);
        };
        // Right after the barrier the others' gate waves are still at work: a
        // load now finds markers, and 32 workgroups reloading delay their
        // stores.  (H = 512, 64 rows: 1.52 us a step without the pause, 1.44
        // with 4, 1.40 with 6, 1.38 with 8, 1.46 with 12; H = 256 in fp32, 32
        // rows: 1.60, 1.52, 1.49, 1.56, 1.61.)  Waves that compute gates
        // themselves come late enough.
        if constexpr (!BOTH) {
            if (j == 0) __builtin_amdgcn_s_sleep(X_PAUSE);
        }
        load_all();
        if (leaves(cnt - 1)) return false;
        if (incomplete()) {
            const unsigned long long t0 = wall_clock64();
            int tries = 0;
            do {
                __builtin_amdgcn_s_sleep(1);
                load_all();
                // (the clock costs more than a try: read at every fourth)
                if ((++tries & 3) == 0 && wall_clock64() - t0 > p.timeout_ticks) {
                    // past the deadline: every wave leaves after the next barrier
                    if (l == 0) {
                        lds_abort = cnt;
                        __hip_atomic_fetch_or(&p.meta->status, STATUS_TIMEOUT, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                    }
                    break;
                }
            } while (incomplete());
        }
        if (tr0 && j == 0) p.trace[4 * t + 3] = wall_clock64();
        return true;
    };
    auto mma_tile = [&]() __attribute__((always_inline)) {
        float* const part = lds + (cnt & 1) * (LY::PART / 4);
        if constexpr (E::KPL == 1) {
            if (few) {
                constexpr int NC = MT == 1 ? 4 : 2;  // chains per gate tile: an MFMA does not wait for the last
                f32x4_t acc[MT][NC];
                f32x4_t sacc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc[mt][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KSW; ++ks) {
                    const float b = __uint_as_float(f[ks >> 2][ks & 3]);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[mt][ks % NC] = mfma_few(afrag[mt][ks], b, acc[mt][ks % NC]);
                    if constexpr (STOP) sacc = E::mfma(E::load(vst + kw0 + kslot<E, KSW>(ks, l)), b, sacc);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    f32x4_t v = acc[mt][0] + acc[mt][1];
                    if constexpr (NC == 4) v += acc[mt][2] + acc[mt][3];
                    v = sum_runs(v);  // lane l: row l & 3, unit l >> 2; to the place of (row, unit) below
                    if (l < 16) *reinterpret_cast<f32x4_t*>(part + (((w * MT + mt) * 64 + (l >> 2) * 16 + (l & 3)) << 2)) = v;
                }
                if constexpr (STOP) {
                    if (l < 16) s_part[cnt & 1][w][l] = sacc[0];
                }
                return;
            }
        }
        f32x4_t acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        f32x4_t sacc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) {
            typename E::frag_t b;
            if constexpr (E::KPL == 1) b = __uint_as_float(f[ks >> 2][ks & 3]);
            else b = __builtin_bit_cast(typename E::frag_t, f[ks]);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = E::mfma(afrag[mt][ks], b, acc[mt]);
            // halting score: every row of the A operand is v, so lane l gets
            // this wave's partial v . h of row (l & 15) of the tile
            if constexpr (STOP) sacc = E::mfma(E::load(vst + kw0 + kslot<E, KSW>(ks, l)), b, sacc);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            *reinterpret_cast<f32x4_t*>(part + (((w * MT + mt) * 64 + l) << 2)) = acc[mt];
        if constexpr (STOP) {
            if (l < 16) s_part[cnt & 1][w][l] = sacc[0];
        }
    };
    // ---- one row tile's gates: this wave's pairs of tile j, after the barrier
    auto gate_tile = [&](const f32x4_t* gx, int j, int rows, int rows3) __attribute__((always_inline)) {
        const float* const part = lds + (cnt & 1) * (LY::PART / 4);
        bool drained = false;
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) {
            if (!pair_ok(i) || pair_tile(i) != j) continue;
            const int mt = (gwi + i * GW) % MT;
            f32x4_t pv[KW + 1];
#pragma unroll
            for (int ww = 0; ww < KW; ++ww)
                pv[ww] = *reinterpret_cast<const f32x4_t*>(part + (((ww * MT + mt) * 64 + l) << 2));
            pv[KW] = gx[i];
#pragma unroll
            for (int span = 1; span <= KW; span *= 2)
#pragma unroll
                for (int b = 0; b + span <= KW; b += 2 * span) pv[b] += pv[b + span];
            const f32x4_t z = pv[0];
            const int r = j * 16 + (l & 15), u = pair_unit(i);
            const bool live = r < rows;
            bool runs = true;
            if constexpr (STOP) {
                float sum = 0.f;
#pragma unroll
                for (int ww = 0; ww < KW; ++ww) sum += s_part[cnt & 1][ww][l & 15];
                if (live && t > 0 && sum + p.stop_c > 0.f && !((stopped >> i) & 1)) {  // ended after step t - 1
                    stopped |= 1u << i;
                    if (role == 0 && mt == 0 && l < 16) p.steps[brow[i]] = t;
                }
                runs = !((stopped >> i) & 1);
                if (runs && live) lds_run[t & 3] = 1;
            }
            const float h_in = hst[i], c_in = cst[i];
            float c = c_in, h = h_in;
            apply_cell(CELL, z, c, h);
            if (live && u < H && runs) {
                cst[i] = c;
                hst[i] = h;
            }
            if (!drained) {
                // the marks of the last step complete before h_{t+1} is stored
                // (waves that poll have waited for loads issued after them)
                if constexpr (!BOTH) drain_stores();
                drained = true;
            }
            stress_delay(t, 64 + i);
            const unsigned nxt = (unsigned)((t + 1) & 3) * ring, far = (unsigned)((t + 3) & 3) * ring;
            // Buffer (t + 3) mod 4 still holds h_{t-1}: this workgroup has seen
            // the tile of h_t from every workgroup of the group, so every one
            // has finished reading that tile of h_{t-1}.
            if (local) {
                if (live) IO::template store<0>(R, nxt + eoff[i], hst[i]);
                mark(loc_t{}, i, far, rows3);
            } else {
                if (live) IO::template store<P_SC1>(R, nxt + eoff[i], hst[i]);
                mark(dev_t{}, i, far, rows3);
            }
            if constexpr (SAVE) {
                if (live && u < H) {  // z in place of Gx, and the state the step started from
                    const size_t row = (size_t)o0 + (r << p.ng_shift) + g;
                    *reinterpret_cast<f32x4_t*>(const_cast<float*>(p.gx) + row * H4 + 4 * u) = z;
                    p.save_h[row * H + u] = h_in;
                    p.save_c[row * H + u] = c_in;
                }
            }
            if (p.seq && live && u < H) p.seq[((size_t)brow[i] * p.T + t) * H + u] = hst[i];
        }
    };
    auto next_step = [&](int o4) __attribute__((always_inline)) {
        o0 = o1;
        o1 = o2;
        o2 = o3;
        o3 = o4;
        ++t;
    };

    // One step; false where the loop ends.  PAR: parity of t.
    auto step = [&](auto par) __attribute__((always_inline)) -> bool {
        constexpr int PAR = decltype(par)::value;
        if (t >= max_len) return false;
        const int rows = rows_of(o1 - o0);
        if (rows == 0) return false;
        const int o4 = offset_at(t + 4);
        const int tiles = (rows + 15) >> 4, rows3 = rows_of(o4 - o3);
        if (tr0) p.trace[4 * t] = wall_clock64();
        if constexpr (BOTH) {
            for (int j = 0; j < tiles; ++j) {
                if (!fetch_tile(j, rows)) return false;
                if (j == 0 && o2 - o1 > g) load_gx(gxr[PAR ^ 1], o1, o2 - o1);
                mma_tile();
                x_barrier();
                read_flags(j);
                if (tr0 && j == 0) p.trace[4 * t + 1] = wall_clock64();
                gate_tile(gxr[PAR], j, rows, rows3);
                ++cnt;
            }
            if (tr1) p.trace[4 * t + 2] = wall_clock64();
        } else if (is_mma) {
            for (int j = 0; j < tiles; ++j) {
                if (!fetch_tile(j, rows)) return false;
                mma_tile();
                x_barrier();
                read_flags(j);
                if (tr0 && j == 0) p.trace[4 * t + 1] = wall_clock64();
                ++cnt;
            }
        } else {
            // (one row tile: no loop, or the compiler waits for every Gx load at its head)
            for (int j = 0; NT == 1 ? j < 1 : j < tiles; ++j) {
                x_barrier();
                read_flags(j);
                gate_tile(gxr[PAR], j, rows, rows3);
                if (leaves(cnt)) return false;
                ++cnt;
            }
            if (tr1) p.trace[4 * t + 2] = wall_clock64();
            asm volatile("" ::: "memory");  // the loads stay behind the stores
            if (o3 - o2 > g) load_gx(gxr[PAR], o2, o3 - o2);
            asm volatile("" ::: "memory");
        }
        next_step(o4);
        return true;
    };
    // The gate waves' memory instructions go before those of the (older) waves
    // that poll, which would otherwise hold up the stores that are polled for.
    if constexpr (!BOTH) {
        if (!is_mma) __builtin_amdgcn_s_setprio(3);
    }
    if (alive && max_len > 0) {
        if (!is_mma || BOTH) {
            if (o1 - o0 > g) load_gx(gxr[0], o0, o1 - o0);
            if constexpr (!BOTH) {
                if (o2 - o1 > g) load_gx(gxr[1], o1, o2 - o1);
            }
        }
        using even_t = std::integral_constant<int, 0>;
        using odd_t = std::integral_constant<int, 1>;
        while (step(even_t{}) && step(odd_t{})) {
        }
    }

    drain_stores();
    if constexpr (STOP) {
        __syncthreads();
        // a loop that ran to its end: did some row run in its last step?
        if (seen_run == 0) --iters;  // (counted before the flag had arrived)
        if (alive && t > 0 && lds_run[(t - 1) & 3] != 0) iters = t;
        if (role == 0 && tid == 0) atomicMax(&p.meta->iters, iters);
    }
    if (tr0) p.trace[4 * max_len] = wall_clock64();
    // ---- final state, batch order
#pragma unroll
    for (int i = 0; i < PAIRS; ++i) {
        if (!pair_ok(i)) continue;
        const int r = pair_tile(i) * 16 + (l & 15), u = pair_unit(i);
        if (r < Bg && u < H) {
            p.out_c[(size_t)brow[i] * H + u] = cst[i];
            p.out_h[(size_t)brow[i] * H + u] = hst[i];
        }
    }
}

// A compiled variant: f[cell][mode].
struct XVariant {
    int bf16, mt, ksw, kw, nt, hpad, lds_bytes;
    xloop_fn f[3][3];
};
#define XV_CELL(ET, MT, KS, KW, NT, C)                                                             \
    {xloop_kernel<ET, MT, KS, KW, NT, C, LM_PLAIN>, xloop_kernel<ET, MT, KS, KW, NT, C, LM_STOP>, \
     xloop_kernel<ET, MT, KS, KW, NT, C, LM_SAVE>}
#define XV(BF, ET, MT, KS, KW, NT)                                                                 \
    {BF, MT, KS, KW, NT, XLayout<ET, MT, KS, KW>::HPAD, XLayout<ET, MT, KS, KW>::BYTES,             \
     {XV_CELL(ET, MT, KS, KW, NT, CELL_LSTM), XV_CELL(ET, MT, KS, KW, NT, CELL_GRU),                \
      XV_CELL(ET, MT, KS, KW, NT, CELL_RNN)}}
#define XV_NT(BF, ET, MT, KS, KW) XV(BF, ET, MT, KS, KW, 1), XV(BF, ET, MT, KS, KW, 2)

}  // namespace ldyn
