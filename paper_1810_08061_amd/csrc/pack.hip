// pack.hip -- GRU and tanh-RNN weights in the LSTM's four-gate-block layout.
//
// The paper's loop takes the cell as a parameter (Section 9 "RNN cells").
// Every kernel of this library reads W [D][4H], U [H][4H] and b [4H] as four
// gate blocks of H columns and hands each hidden unit its four
// pre-activations; the gate step then applies the cell's update to them.
//
// GRU: a unit has three gate blocks (r, u, n), and its n block needs the
// input and recurrent parts separately (the reset gate scales only the
// recurrent part), so the four blocks carry r, u, the recurrent part of n and
// the input part of n, with zero weights where a part has no term:
//   W4 = (W_r, W_u, 0, W_n),  U4 = (U_r, U_u, U_n, 0),
//   b4 = (b_ir + b_hr, b_iu + b_hu, b_hn, b_in).
// RNN: one pre-activation per unit in block 0, zeros elsewhere:
//   W4 = (W, 0, 0, 0),  U4 = (U, 0, 0, 0),  b4 = (b, 0, 0, 0).
// One pass per forward; the three zero blocks of the RNN cost MFMA work (the
// loop is bound by the exchange of h, not by the products, at the sizes it is
// built for).
#include "launch.h"

namespace ldyn {

// One wave per row of W4, then of U4, then b4 (no division: with one element
// per thread, three 64-bit ones each, the GRU's 200 + 750 rows of 3000 took
// 10 us; 6.8 so).
template <typename S, int CELL>
__global__ void __launch_bounds__(256)
cell_pack_kernel(const S* __restrict__ W, const S* __restrict__ U, const float* __restrict__ b,
                 S* __restrict__ W4, S* __restrict__ U4, float* __restrict__ b4, int D, int H) {
    constexpr int N = CELL == CELL_RNN ? 1 : 3;  // blocks of the cell's own layout
    const S zero = (S)0.0f;
    const int lane = threadIdx.x & 63;
    for (long r = blockIdx.x * 4L + (threadIdx.x >> 6); r <= (long)D + H; r += gridDim.x * 4L) {
        if (r == (long)D + H) {
            for (int u = lane; u < H; u += 64) {
                if constexpr (CELL == CELL_RNN) {
                    b4[u] = b[u];
#pragma unroll
                    for (int g = 1; g < 4; ++g) b4[(size_t)g * H + u] = 0.0f;
                } else {
                    const float* bih = b;
                    const float* bhh = b + 3 * (size_t)H;
#pragma unroll
                    for (int g = 0; g < 2; ++g) b4[(size_t)g * H + u] = bih[(size_t)g * H + u] + bhh[(size_t)g * H + u];
                    b4[2 * (size_t)H + u] = bhh[2 * (size_t)H + u];
                    b4[3 * (size_t)H + u] = bih[2 * (size_t)H + u];
                }
            }
            continue;
        }
        const bool is_u = r >= D;
        const long k = is_u ? r - D : r;
        const S* src = (is_u ? U : W) + k * N * H;
        S* dst = (is_u ? U4 : W4) + k * 4 * H;
#pragma unroll 4
        for (int u = lane; u < H; u += 64) {
            S v[N];
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = src[(size_t)j * H + u];
            dst[u] = v[0];
            if constexpr (N == 1) {
#pragma unroll
                for (int g = 1; g < 4; ++g) dst[(size_t)g * H + u] = zero;
            } else {  // GRU: W4 (r, u, 0, n), U4 (r, u, n, 0)
                dst[(size_t)H + u] = v[1];
                dst[2 * (size_t)H + u] = is_u ? v[2] : zero;
                dst[3 * (size_t)H + u] = is_u ? zero : v[2];
            }
        }
    }
}

template <typename S>
static void launch_pack(const Dims& d, const void* W, const void* U, const float* b, void* W4, void* U4,
                        float* b4, hipStream_t s) {
    const long g4 = ((long)d.D + d.H + 4) / 4;
    auto k = d.cell == CELL_GRU ? cell_pack_kernel<S, CELL_GRU> : cell_pack_kernel<S, CELL_RNN>;
    hipLaunchKernelGGL(k, dim3((unsigned)(g4 > 4096 ? 4096 : g4)), dim3(256), 0, s, static_cast<const S*>(W),
                       static_cast<const S*>(U), b, static_cast<S*>(W4), static_cast<S*>(U4), b4, d.D, d.H);
}

hipError_t launch_cell_pack(const Dims& d, const void* W, const void* U, const float* b, void* W4,
                            void* U4, float* b4, hipStream_t s) {
    if (d.cell != CELL_GRU && d.cell != CELL_RNN) return hipErrorInvalidValue;
    if (d.bf16) launch_pack<__bf16>(d, W, U, b, W4, U4, b4, s);
    else launch_pack<float>(d, W, U, b, W4, U4, b4, s);
    return hipGetLastError();
}

}  // namespace ldyn
