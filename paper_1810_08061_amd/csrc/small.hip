// small.hip -- the whole forward in one workgroup, one launch (H <= 32).
//
// When the 4H gate columns fit the 8 gate tiles of one workgroup, nothing
// needs a grid: the loop bound is reduced in LDS, each step forms
// z = x_t W + h U + b with MFMA (W and U slices held in registers, each wave
// owning one gate tile over the full K = D + H, so no cross-wave reduction),
// applies the gates to the rows with t < L[b] (the per-row select of the
// paper's loop, Section 9 "RNN cells"), and passes h to the next step through
// LDS.  Rows stay in batch order; finished rows are simply not updated.  With
// bf16 data, x W takes bf16 operands and h U fp16 operands (U widened from
// bf16), as in the persistent loop.
//
// A step is one chain: h from LDS, the products of h (fp32: 16 of 32 cycles each
// per SIMD), the gates, h to LDS, a barrier.  The products of x need no h: those
// of step t + 1 are issued right after step t's products of h and run in the
// matrix unit while the gates are computed, on x loaded ahead.  Eight waves of
// one gate tile, h U in two chains, instead of four waves of two tiles with both
// products in the chain.
//
// Every wave needs all of x_t, whose fragments are gathers of single elements (D
// is any number).  The workgroup gathers each 16-byte chunk of them once, by one
// of its waves, and shares it through LDS.  Taken by each wave for itself, these
// loads are what a step waits for; 64 rows, 60 steps, with four waves of two
// tiles, with eight waves that each take all of x, and shared:
//   fp32 D 16    340, 357 and 188 us
//   fp32 D 64    727, 1027 and 332
//   bf16 D 128  1020, 1704 and 313
// (16 rows, fp32 D 12, 200 steps with the sequence: 336, 369 and 231; 4 rows, D 16,
// 20 steps: 50.7, 44.5 and 39.4.)
#include "launch.h"

namespace ldyn {

constexpr int SM_WAVES = 8;  // each one gate tile: 8 x 16 columns = 4H <= 128
constexpr int SM_THREADS = 64 * SM_WAVES;

struct SmallParams {
    const void* x;
    const int32_t* lengths;
    const void* W;
    const void* U;
    const float* b;
    const float* h0;
    const float* c0;
    float* out_h;
    float* out_c;
    float* seq;  // [B][T][H] output sequence (valid steps only), or null
    Meta* meta;
    int B, D, H, T;
    int cell;  // CellKind (only the LSTM has a cell state)
    // termination from the state (stop_v null: none): a row ends after a step
    // that leaves v . h + c > 0; steps[b] receives the steps it ran
    const float* stop_v;
    float stop_c;
    int32_t* steps;
};

// E: element type of x and W; EH: of the recurrent operands (U, h).
template <typename E, typename EH, int KD, int KH, int NT>
__global__ void __launch_bounds__(SM_THREADS, 1)
small_kernel(SmallParams p) {
    using S = typename E::store_t;
    using F = typename E::frag_t;
    using SH = typename EH::store_t;
    using FH = typename EH::frag_t;
    static_assert(E::KSTEP == EH::KSTEP && E::KPL == EH::KPL, "one fragment shape");
    constexpr int HP = KH * EH::KSTEP;      // padded hidden width of the LDS h rows
    constexpr int HS = HP + 16 / sizeof(SH);  // row stride (16-byte pad)
    __shared__ __attribute__((aligned(16))) SH hs[2][NT * 16 * HS];
    __shared__ int len[NT * 16];
    __shared__ int maxlen, bad;
    // x of a step as chunks of 16 bytes per lane: CPU K-steps of one row tile each
    constexpr int CPU = 16 / (int)sizeof(F), CHUNKS = NT * KD / CPU;
    static_assert(KD % CPU == 0, "whole chunks");
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    __shared__ u32x4 xs[2][CHUNKS * 64];  // by step parity
    __shared__ int ended[NT * 16];  // termination from the state: 1 once the row ended
    __shared__ int ran[2];          // some row ran at step t (slot t & 1)

    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int B = p.B, D = p.D, H = p.H, T = p.T, H4 = 4 * H;
    const S* X = static_cast<const S*>(p.x);
    const S* W = static_cast<const S*>(p.W);
    const typename EH::src_t* U = static_cast<const typename EH::src_t*>(p.U);

    if (tid == 0) {
        maxlen = 0;
        bad = 0;
        ran[0] = 0;
        ran[1] = 0;
    }
    __syncthreads();
    for (int i = tid; i < NT * 16; i += SM_THREADS) {
        int v = 0;
        if (i < B) {
            v = p.lengths[i];
            if (v < 0 || v > T) {
                atomicOr(&bad, 1);
                v = v < 0 ? 0 : T;
            }
            atomicMax(&maxlen, v);
        }
        len[i] = v;
        ended[i] = 0;
        if (p.stop_v && i < B) p.steps[i] = v;  // a row that never ends runs to its cap
    }
    // h0 -> LDS (operand type); padding rows and columns are zero in both buffers
    for (int i = tid; i < NT * 16 * HS; i += SM_THREADS) {
        const int n = i / HS, k = i - n * HS;
        hs[0][i] = EH::from_f32((n < B && k < H) ? p.h0[(size_t)n * H + k] : 0.0f);
        hs[1][i] = EH::from_f32(0.0f);
    }

    // A-fragments of W^T and U^T for this wave's gate tile (clamped loads).
    F wf[KD];
    FH uf[KH];
    f32x4_t bias;
    {
        const int cp = w * 16 + (l & 15);
        const bool uok = (cp >> 2) < H;
        const int col = uok ? gate_col(cp, H) : 0;
#pragma unroll
        for (int ks = 0; ks < KD; ++ks) {
            F f = E::zero();
#pragma unroll
            for (int e = 0; e < E::KPL; ++e) {
                const int k = ks * E::KSTEP + (l >> 4) * E::KPL + e;
                const S v = W[(size_t)min(k, D - 1) * H4 + col];
                if constexpr (E::KPL == 1) f = (uok && k < D) ? v : 0.0f;
                else f[e] = (uok && k < D) ? v : E::from_f32(0.0f);
            }
            wf[ks] = f;
        }
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) {
            FH f = EH::zero();
#pragma unroll
            for (int e = 0; e < EH::KPL; ++e) {
                const int k = ks * EH::KSTEP + (l >> 4) * EH::KPL + e;
                const SH v = EH::from_src(U[(size_t)min(k, H - 1) * H4 + col]);
                if constexpr (EH::KPL == 1) f = (uok && k < H) ? v : 0.0f;
                else f[e] = (uok && k < H) ? v : EH::from_f32(0.0f);
            }
            uf[ks] = f;
        }
    }
    // this lane's four gates belong to one unit
    const int u = (w * 16 + 4 * (l >> 4)) >> 2;
#pragma unroll
    for (int g = 0; g < 4; ++g) bias[g] = u < H ? p.b[g * H + u] : 0.0f;

    // Owned state: lane holds (row nt*16 + (l & 15), unit u).
    float cst[NT], hst[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = nt * 16 + (l & 15);
        const bool ok = n < B && u < H;
        cst[nt] = ok && p.cell == CELL_LSTM ? p.c0[(size_t)n * H + u] : 0.0f;
        hst[nt] = ok ? p.h0[(size_t)n * H + u] : 0.0f;
    }
    __syncthreads();
    const int ml = maxlen;

    // One K-step's x fragment of a row tile: lane holds row nt*16 + (l & 15), K slice of D.
    auto load_frag = [&](int nt, int ks, int t) __attribute__((always_inline)) -> F {
        const int n = nt * 16 + (l & 15);
        const size_t row = (size_t)min(n, B - 1) * T + min(t, T - 1);
        F f = E::zero();
#pragma unroll
        for (int e = 0; e < E::KPL; ++e) {
            const int k = ks * E::KSTEP + (l >> 4) * E::KPL + e;
            const S v = X[row * D + min(k, D - 1)];
            if constexpr (E::KPL == 1) f = k < D ? v : 0.0f;
            else f[e] = k < D ? v : E::from_f32(0.0f);
        }
        return f;
    };
    // The wave's chunks of a step: OWN of them.  Dealt from the last wave on where
    // that one owns no unit (1 row, H = 8, 60 steps: 72 us from the first wave, 67
    // from the last), else from the first, which the SIMD issues first (bf16, 1
    // row, H = 32, 60 steps: 51.3 us from the first, 54.4 from the last).
    constexpr int OWN = (CHUNKS + SM_WAVES - 1) / SM_WAVES;
    F xo[OWN][CPU];
    const int w_own = H > 4 * (SM_WAVES - 1) ? w : SM_WAVES - 1 - w;
    auto own = [&](int i) __attribute__((always_inline)) { return w_own + i * SM_WAVES; };
    auto load_x = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int c = own(i);
            if (c < CHUNKS)
#pragma unroll
                for (int e = 0; e < CPU; ++e) xo[i][e] = load_frag(c / (KD / CPU), c % (KD / CPU) * CPU + e, t);
        }
    };
    auto share_x = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int c = own(i);
            if (c < CHUNKS) xs[t & 1][c * 64 + l] = __builtin_bit_cast(u32x4, xo[i]);
        }
    };
    int lenr[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) lenr[nt] = len[nt * 16 + (l & 15)];  // 0 for padding rows

    // x_t W + b of the step to come: its products run while the step before
    // computes its gates
    f32x4_t accx[NT];
    auto project = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) accx[nt] = bias;
#pragma unroll
        for (int kc = 0; kc < KD / CPU; ++kc)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const u32x4 v = xs[t & 1][(nt * (KD / CPU) + kc) * 64 + l];
                F f[CPU];
                __builtin_memcpy(f, &v, sizeof(v));
#pragma unroll
                for (int e = 0; e < CPU; ++e) accx[nt] = E::mfma(wf[kc * CPU + e], f[e], accx[nt]);
            }
    };
    if (ml > 0) {
        load_x(0);
        share_x(0);
        load_x(1);
        share_x(1);
        load_x(2);
        __syncthreads();
        project(0);
        __syncthreads();  // x_0 has been read: step 0 puts x_2 in its place
    }

    int iters = 0;  // termination from the state: steps in which some row ran
    int t = 0;
    // Step t: x_{t+1} is in LDS, the wave holds its chunks of x_{t+2}.  False
    // where the loop ends.
    auto step = [&]() __attribute__((always_inline)) -> bool {
        const SH* hcur = hs[t & 1];
        SH* hnext = hs[(t + 1) & 1];
        if (p.stop_v) {
            // Halting scores of h_t (the operand in LDS, k in order): a row
            // that ran step t-1 and scores > 0 has ended.  Wave nt forms those
            // of row tile nt; only its lanes read ended[] of these rows before
            // lane (row, unit 0) changes it.
            if (t > 0) {
                if (ran[(t - 1) & 1] == 0) return false;  // no row ran at step t-1: none runs again
                iters = t;
                if (w < NT) {
                    const int n = w * 16 + (l & 15);
                    float sc = 0.f;
                    for (int k = 0; k < H; ++k) sc += p.stop_v[k] * EH::to_f32(hcur[n * HS + k]);
                    const bool ends = n < B && t - 1 < len[n] && !ended[n] && sc + p.stop_c > 0.f;
                    if (ends && (l >> 4) == 0) {
                        ended[n] = 1;
                        p.steps[n] = t;
                    }
                }
            }
            if (tid == 0) ran[t & 1] = 0;
            __syncthreads();
        }
        // h U in two chains of products per row tile, one from x_t W + b
        f32x4_t acc[2][NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            acc[0][nt] = accx[nt];
            acc[1][nt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int ks = 0; ks < KH; ++ks)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const FH hf = EH::load(hcur + (nt * 16 + (l & 15)) * HS + ks * EH::KSTEP + (l >> 4) * EH::KPL);
                acc[ks & 1][nt] = EH::mfma(uf[ks], hf, acc[ks & 1][nt]);
            }
        __builtin_amdgcn_sched_barrier(0);
        project(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int n = nt * 16 + (l & 15);
            if (u >= H) continue;
            if (t < lenr[nt] && !(p.stop_v && ended[n])) {
                if (p.stop_v) ran[t & 1] = 1;
                const f32x4_t z = acc[0][nt] + acc[1][nt];
                float c = cst[nt], h = hst[nt];
                apply_cell(p.cell, z, c, h);
                cst[nt] = c;
                hst[nt] = h;
                if (p.seq) p.seq[((size_t)n * T + t) * H + u] = h;  // output at step t
            }
            hnext[n * HS + u] = EH::from_f32(hst[nt]);
        }
        share_x(t + 2);  // over x_t, read in step t - 1
        if (t + 3 < ml) load_x(t + 3);
        __syncthreads();
        ++t;
        return t < ml;
    };
    if (ml > 0) {
        while (step()) {
        }
    }

#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = nt * 16 + (l & 15);
        if (n < B && u < H) {
            p.out_h[(size_t)n * H + u] = hst[nt];
            p.out_c[(size_t)n * H + u] = cst[nt];
        }
    }
    if (tid == 0) {
        int total = 0;
        for (int i = 0; i < B; ++i) total += len[i];
        p.meta->max_len = ml;
        p.meta->total_rows = total;
        p.meta->status = bad ? STATUS_BAD_LENGTHS : 0;
        // a loop that ran to ml: did some row run in its last step?
        if (p.stop_v && t == ml && ml > 0 && ran[(ml - 1) & 1] != 0) iters = ml;
        p.meta->iters = p.stop_v ? iters : ml;
    }
}

typedef void (*small_fn)(SmallParams);
struct SmallVariant { int bf16, kd, kh, nt; small_fn f; };
#define SV(BF, ET, EH, KD, KH, NT) {BF, KD, KH, NT, small_kernel<ET, EH, KD, KH, NT>}
static const SmallVariant kSmall[] = {
    // fp32: K-step 4; D <= 64, H <= 32; B <= 16 or 64
    SV(0, EltF32, EltF32, 4, 8, 1), SV(0, EltF32, EltF32, 16, 8, 1), SV(0, EltF32, EltF32, 4, 8, 4),
    SV(0, EltF32, EltF32, 16, 8, 4),
    // bf16 data (fp16 recurrent operands): K-step 32; D <= 128, H <= 32
    SV(1, EltBF16, EltH16, 1, 1, 1), SV(1, EltBF16, EltH16, 4, 1, 1), SV(1, EltBF16, EltH16, 1, 1, 4),
    SV(1, EltBF16, EltH16, 4, 1, 4),
};
#undef SV

// Smallest variant covering (D, H, B); fills *kd, *nt.  Returns false if none.
bool small_pick(int bf16, int B, int D, int H, int* kd, int* nt) {
    const int kstep = bf16 ? 32 : 4;
    const int kdn = (D + kstep - 1) / kstep, khn = (H + kstep - 1) / kstep;
    const int ntn = (B + 15) / 16;
    int best = -1;
    for (int i = 0; i < (int)(sizeof(kSmall) / sizeof(kSmall[0])); ++i) {
        const SmallVariant& v = kSmall[i];
        if (v.bf16 != bf16 || v.kd < kdn || v.kh < khn || v.nt < ntn) continue;
        if (best < 0 || v.kd * v.nt < kSmall[best].kd * kSmall[best].nt) best = i;
    }
    if (best < 0) return false;
    *kd = kSmall[best].kd;
    *nt = kSmall[best].nt;
    return true;
}

hipError_t launch_small(const Dims& d, int kd, int nt, const void* x, const int32_t* lengths,
                        const void* W, const void* U, const float* b, const float* h0,
                        const float* c0, float* out_h, float* out_c, float* seq,
                        const StopArgs* stop, const Workspace& ws, hipStream_t s) {
    small_fn f = nullptr;
    for (const SmallVariant& v : kSmall)
        if (v.bf16 == d.bf16 && v.kd == kd && v.nt == nt) f = v.f;
    if (!f) return hipErrorInvalidValue;
    SmallParams p{x, lengths, W, U, b, h0, c0, out_h, out_c, seq, ws.meta, d.B, d.D, d.H, d.T, d.cell,
                  stop ? stop->v : nullptr, stop ? stop->c : 0.0f, stop ? stop->steps : nullptr};
    hipLaunchKernelGGL(f, dim3(1), dim3(SM_THREADS), 0, s, p);
    return hipGetLastError();
}

}  // namespace ldyn
