// gemm.hip -- MFMA GEMM with gathered rows and gate-interleaved columns.
//
// Two uses:
//   * the input projection hoisted out of the time loop: x does not depend on
//     the state, so x[b, t] W + b for every valid (b, t) is one GEMM over all
//     time steps, M = sum of lengths (compact rows), N = 4H, K = D;
//   * the per-step comparison path's recurrent product h U + Gx[t] for the
//     rows active at step t, M = active(t), N = 4H, K = H (with bf16 data in
//     fp16 operands, as in the persistent loop: U is widened from bf16 on its
//     way into LDS, h is kept in fp16).
//
// C^T is formed as (W^T)(A^T): MFMA rows are gate-interleaved columns c', MFMA
// columns are data rows, so each lane's four fp32 results are the four gates
// (i, f, g, o) of one (row, unit) and leave as one 16-byte store.
#include "launch.h"

namespace ldyn {

constexpr int G_THREADS = 256;
constexpr int G_CM = 128;  // c' per tile (MFMA M)
constexpr int G_RN = 128;  // rows per tile (MFMA N)
constexpr int G_SMALL = 64;  // c' and rows per small tile

enum GemmMode { MODE_INPROJ = 0, MODE_STEP = 1 };

struct GemmParams {
    const void* A;         // INPROJ: x [B*T][D]; STEP: operand buffer [bpad][hpad]
    const void* Bw;        // W [D][4H] or U [H][4H]
    const float* bias;     // INPROJ: b [4H]
    const float* gx;       // STEP: addend rows gx[offsets[t] + r]
    float* out;            // INPROJ: gx; STEP: z  (row stride 4H)
    const Meta* meta;
    const int32_t* rowsrc;
    const int32_t* offsets;
    int K, lda, H, t;
    int a_vec, b_vec;      // the A rows / the gates' runs of a B row are whole, aligned 16-byte vectors
    int small_upto;        // small tiles where there are at most this many large ones
};

// T: c' and rows per tile, BKB: bytes of K per block.
template <typename E, int T, int BKB>
struct GemmTile {
    using S = typename E::store_t;
    static constexpr int VE = 16 / sizeof(S);      // elements per 16-byte vector
    static constexpr int BK = BKB / sizeof(S);     // K per block
    static constexpr int LDK = BK + VE;            // padded LDS row
    static constexpr int KS = BK / E::KSTEP;       // MFMA K-steps per block
    static constexpr int UV = (T / 4) / VE;        // vectors per (k, gate) row segment
    static constexpr int SEG = BK / VE;            // vectors per row
    static constexpr int AV = T * SEG / G_THREADS;     // vectors per thread of either tile
    static constexpr int FT = T / 32;              // 16 x 16 result tiles per wave and side
    static constexpr int LDS = 2 * T * LDK;        // elements
    static_assert(AV * G_THREADS == T * SEG && BK * 4 * UV == T * SEG, "whole vectors per thread");
};

// The tiles of one workgroup (grid-strided), row_base: first compact row.
template <typename E, int MODE, int T, int BKB>
__device__ __forceinline__ void gemm_tiles(const GemmParams& p, int nrows, int row_base,
                                           typename E::store_t* lds) {
    using S = typename E::store_t;
    using Src = typename E::src_t;  // element type of Bw (the caller's W or U)
    static_assert(sizeof(Src) == sizeof(S), "operand and source elements have one size");
    using F = typename E::frag_t;
    using TL = GemmTile<E, T, BKB>;
    constexpr int VE = TL::VE, BK = TL::BK, LDK = TL::LDK, KS = TL::KS, UV = TL::UV, AV = TL::AV, FT = TL::FT;
    S* const As = lds;
    S* const Bs = lds + T * LDK;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int H = p.H, N4 = 4 * H, K = p.K;
    const int ntc = (N4 + T - 1) / T;
    const int ntr = (nrows + T - 1) / T;
    const int ntiles = ntc * ntr;
    const S* __restrict__ A = static_cast<const S*>(p.A);
    const Src* __restrict__ Bw = static_cast<const Src*>(p.Bw);
    const int nkb = (K + BK - 1) / BK;

    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int tr = tile / ntc, tc = tile - tr * ntc;
        const int r0 = tr * T, c0 = tc * T, ubase = c0 >> 2;

        // Per-thread source rows of the A tile (AV 16-byte vectors per thread).
        const S* arow[AV];
        bool arow_ok[AV];
        int aseg[AV], ar[AV];
#pragma unroll
        for (int j = 0; j < AV; ++j) {
            const int v = tid + G_THREADS * j;
            ar[j] = v / TL::SEG;
            aseg[j] = v % TL::SEG;
            const int r = r0 + ar[j];
            arow_ok[j] = r < nrows;
            long src = 0;
            if (arow_ok[j]) src = (MODE == MODE_INPROJ) ? (long)p.rowsrc[r] : (long)r;
            arow[j] = A + src * p.lda;
        }
        // B tile vectors: (kk, gate, seg) per thread.
        int bkk[AV], bg[AV], bseg[AV];
#pragma unroll
        for (int j = 0; j < AV; ++j) {
            const int v = tid + G_THREADS * j;
            bseg[j] = v % UV;
            bg[j] = (v / UV) & 3;
            bkk[j] = v / (UV * 4);
        }

        S areg[AV][VE];
        Src breg[AV][VE];
        auto load_tiles = [&](int k0) {
#pragma unroll
            for (int j = 0; j < AV; ++j) {
                const int k = k0 + aseg[j] * VE;
                // Rows of whole 16-byte vectors: past the end another is taken and not
                // used, so that no load waits behind a branch.  Else the same loads at
                // the elements' alignment, and one by one at a row's end (one by one
                // throughout, 2115 tiles at H 257, D 400 took 404 us, and 362 so).
                if (p.a_vec) {
                    const bool ok = arow_ok[j] && k < K;
                    const uint4 v = *reinterpret_cast<const uint4*>(arow[j] + (k < K ? k : 0));
                    const S* vs = reinterpret_cast<const S*>(&v);
#pragma unroll
                    for (int e = 0; e < VE; ++e) areg[j][e] = ok ? vs[e] : E::from_f32(0.0f);
                } else if (arow_ok[j] && k + VE <= K) {
                    __builtin_memcpy(areg[j], arow[j] + k, 16);
                } else {
#pragma unroll
                    for (int e = 0; e < VE; ++e)
                        areg[j][e] = (arow_ok[j] && k + e < K) ? arow[j][k + e] : E::from_f32(0.0f);
                }
                const int kb = k0 + bkk[j];
                const int u = ubase + bseg[j] * VE;
                const Src* src = Bw + (long)min(kb, K - 1) * N4 + bg[j] * H;
                if (p.b_vec) {
                    const bool ok = kb < K && u < H;
                    const uint4 v = *reinterpret_cast<const uint4*>(src + (u < H ? u : 0));
                    const Src* vs = reinterpret_cast<const Src*>(&v);
#pragma unroll
                    for (int e = 0; e < VE; ++e) breg[j][e] = ok ? vs[e] : (Src)0.0f;
                } else if (kb < K && u + VE <= H) {
                    __builtin_memcpy(breg[j], src + u, 16);
                } else {
#pragma unroll
                    for (int e = 0; e < VE; ++e) breg[j][e] = (kb < K && u + e < H) ? src[u + e] : (Src)0.0f;
                }
            }
        };
        auto store_tiles = [&]() {
#pragma unroll
            for (int j = 0; j < AV; ++j) {
                S* dst = As + ar[j] * LDK + aseg[j] * VE;
#pragma unroll
                for (int e = 0; e < VE; ++e) dst[e] = areg[j][e];
#pragma unroll
                for (int e = 0; e < VE; ++e)
                    Bs[(4 * (bseg[j] * VE + e) + bg[j]) * LDK + bkk[j]] = E::from_src(breg[j][e]);
            }
        };

        f32x4_t acc[FT][FT];
#pragma unroll
        for (int i = 0; i < FT; ++i)
#pragma unroll
            for (int j = 0; j < FT; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        load_tiles(0);
        __syncthreads();  // previous tile's readers are done with LDS
        store_tiles();
        __syncthreads();
        for (int kb = 0; kb < nkb; ++kb) {
            if (kb + 1 < nkb) load_tiles((kb + 1) * BK);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int koff = ks * E::KSTEP + (lane >> 4) * E::KPL;
                F af[FT], bf[FT];
#pragma unroll
                for (int i = 0; i < FT; ++i)
                    af[i] = E::load(Bs + (wm * (T / 2) + i * 16 + (lane & 15)) * LDK + koff);
#pragma unroll
                for (int j = 0; j < FT; ++j)
                    bf[j] = E::load(As + (wn * (T / 2) + j * 16 + (lane & 15)) * LDK + koff);
#pragma unroll
                for (int i = 0; i < FT; ++i)
#pragma unroll
                    for (int j = 0; j < FT; ++j) acc[i][j] = E::mfma(af[i], bf[j], acc[i][j]);
            }
            __syncthreads();
            if (kb + 1 < nkb) {
                store_tiles();
                __syncthreads();
            }
        }

        // Epilogue: lane holds gates 0..3 of unit u for one row.
#pragma unroll
        for (int i = 0; i < FT; ++i) {
            const int cp = c0 + wm * (T / 2) + i * 16 + 4 * (lane >> 4);
            const int u = cp >> 2;
            if (u >= H) continue;
#pragma unroll
            for (int j = 0; j < FT; ++j) {
                const int r = r0 + wn * (T / 2) + j * 16 + (lane & 15);
                if (r >= nrows) continue;
                f32x4_t v = acc[i][j];
                if (MODE == MODE_INPROJ) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) v[g] += p.bias[g * H + u];
                } else {
                    const f32x4_t a =
                        *reinterpret_cast<const f32x4_t*>(p.gx + (long)(row_base + r) * N4 + cp);
                    v += a;
                }
                *reinterpret_cast<f32x4_t*>(p.out + (long)r * N4 + cp) = v;
            }
        }
    }
}

// Input projection: tiles of 128 x 128, or where those are too few to occupy the
// CUs (the number of rows is known here only) of 64 x 64, four times as many.
// BKL, BKS: bytes of K per block of either; see launch_inproj.
template <typename E, int MODE, int BKL, int BKS>
__global__ void __launch_bounds__(G_THREADS)
gemm_kernel(GemmParams p) {
    using S = typename E::store_t;
    using Large = GemmTile<E, G_CM, BKL>;
    using Small = GemmTile<E, G_SMALL, BKS>;
    constexpr int LDS = MODE == MODE_INPROJ && Small::LDS > Large::LDS ? Small::LDS : Large::LDS;
    __shared__ __attribute__((aligned(16))) S lds[LDS];
    if constexpr (MODE == MODE_INPROJ) {
        const int nrows = p.meta->total_rows;
        const int large = ((4 * p.H + G_CM - 1) / G_CM) * ((nrows + G_RN - 1) / G_RN);
        if (large <= p.small_upto) gemm_tiles<E, MODE, G_SMALL, BKS>(p, nrows, 0, lds);
        else gemm_tiles<E, MODE, G_CM, BKL>(p, nrows, 0, lds);
    } else {
        const int row_base = p.offsets[p.t];
        gemm_tiles<E, MODE, G_CM, BKL>(p, p.offsets[p.t + 1] - row_base, row_base, lds);
    }
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

hipError_t launch_inproj(const Dims& d, const void* x, const void* W, const float* b,
                         const Workspace& ws, int num_cus, hipStream_t s) {
    GemmParams p{};
    p.A = x;
    p.Bw = W;
    p.bias = b;
    p.out = ws.gx;
    p.meta = ws.meta;
    p.rowsrc = ws.rowsrc;
    p.K = d.D;
    p.lda = d.D;
    p.H = d.H;
    p.a_vec = (d.D % 4 == 0) && aligned16(x);
    p.b_vec = (d.H % 4 == 0) && aligned16(W);
    // Small tiles while there is at most one large tile per CU (D 128: 96 large ones
    // take 23 us, their four times as many small ones 15; 190 25 and 22; 256 27 and
    // 24; 400 34 and 35), but only up to three quarters of that where D is five runs
    // of 16, which the small tiles' blocks pad to eight (D 65: 190 large ones 22 and
    // 21, 247 23 and 26).
    const int n16 = (d.D + 15) / 16;
    p.small_upto = n16 == 5 ? num_cus * 3 / 4 : num_cus;
    // Bytes of K per block.  Small tiles: 256, or what D fills (D 16, 190 tiles: 22.9
    // us with 256, 16.6 and now 13.9 with 64).  Large tiles: 64, and 128 where D fills those and H
    // the tiles' columns (a memory latency per block is in the way; 752 tiles at D
    // 256: 104 and 89 us; 1775 at D 48, in part zeros: 63 and 74; at H 40, the
    // second tile of columns nearly empty, D 512: 205 and 212).
    const int ntc = (4 * d.H + G_CM - 1) / G_CM;
    const bool wide = n16 > 2 && n16 % 2 == 0 && 8LL * ntc * G_CM <= 9 * 4LL * d.H;
    const long long tiles = (((long long)d.B * d.T + G_SMALL - 1) / G_SMALL) * ((4LL * d.H + G_SMALL - 1) / G_SMALL);
    const int grid = (int)(tiles < 4LL * num_cus ? tiles : 4LL * num_cus);
    auto k = n16 <= 1   ? gemm_kernel<EltF32, MODE_INPROJ, 64, 64>
             : n16 <= 2 ? gemm_kernel<EltF32, MODE_INPROJ, 64, 128>
             : wide     ? gemm_kernel<EltF32, MODE_INPROJ, 128, 256>
                        : gemm_kernel<EltF32, MODE_INPROJ, 64, 256>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(G_THREADS), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_step_gemm(const Dims& d, int t, const void* U, const Workspace& ws, hipStream_t s) {
    GemmParams p{};
    p.A = ws.hx;
    p.Bw = U;
    p.gx = ws.gx;
    p.out = ws.z;
    p.offsets = ws.offsets;
    p.K = d.H;
    p.lda = d.hpad;
    p.H = d.H;
    p.t = t;
    const int ve = d.bf16 ? 8 : 4;
    p.a_vec = (d.hpad % ve == 0);
    p.b_vec = (d.H % ve == 0) && aligned16(U);
    const int grid = ((4 * d.H + G_CM - 1) / G_CM) * ((d.B + G_RN - 1) / G_RN);
    if (d.bf16)
        hipLaunchKernelGGL((gemm_kernel<EltH16, MODE_STEP, 64, 64>), dim3(grid), dim3(G_THREADS), 0, s, p);
    else
        hipLaunchKernelGGL((gemm_kernel<EltF32, MODE_STEP, 64, 64>), dim3(grid), dim3(G_THREADS), 0, s, p);
    return hipGetLastError();
}

}  // namespace ldyn
