// seq.hip -- the output sequence of the loop.
//
// The loop of the paper (Section 9 "RNN cells", Appendix A) appends the
// cell's output at every step.  out_seq[b][t] is the hidden state of row b
// after step t for t < L[b]; past a sequence's length (or past the step at
// which a row ended, with termination from the state) the output is zero (no
// value is defined there; zero is the padding convention chosen).
//
// Every loop writes the valid outputs itself; this kernel writes the zeros
// past each row's last step.
#include "launch.h"

namespace ldyn {

struct SeqParams {
    float* seq;              // [B][T][H]
    const int32_t* lengths;  // [B] last step + 1 of each row: its length as passed, or the
                             // step it ended at (clamped here to [0, T])
    int B, T, H;
};

// One wave per output row; float4 stores when H is a multiple of 4 and
// out_seq is 16-byte aligned.
template <bool VEC>
__global__ void __launch_bounds__(256)
seq_finish_kernel(SeqParams p) {
    const int lane = threadIdx.x & 63;
    const long wave = ((long)blockIdx.x * 256 + threadIdx.x) >> 6;
    const long nwaves = (long)gridDim.x * 4;
    const int H = p.H, T = p.T;
    const long nrows = (long)p.B * T;
    for (long row = wave; row < nrows; row += nwaves) {
        const int b = (int)(row / T), t = (int)(row - (long)b * T);
        const int L = min(max(p.lengths[b], 0), T);
        if (t < L) continue;
        float* dst = p.seq + (size_t)row * H;
        if constexpr (VEC) {
            for (int u = 4 * lane; u < H; u += 256) *reinterpret_cast<f32x4_t*>(dst + u) = f32x4_t{0.f, 0.f, 0.f, 0.f};
        } else {
            for (int u = lane; u < H; u += 64) dst[u] = 0.0f;
        }
    }
}

// Output sequence of the forward for training: the state after step t of a
// row is the state step t + 1 started from (kept per compact row), or its
// final state after its last step.  Zeros past each length.  One wave per
// output row, bound by its writes (26 MB at 128 rows, 100 steps, H = 512: 20 us
// with one element per thread and three divisions for it, 9 us so); VEC: four
// elements per access (H a multiple of 4, out_h and seq 16-byte aligned).
template <bool VEC>
__global__ void __launch_bounds__(256)
seq_from_saved_kernel(float* seq, const float* __restrict__ save_h, const float* __restrict__ out_h,
                      const int32_t* __restrict__ perm, const int32_t* __restrict__ offsets,
                      const int32_t* __restrict__ lengths, int B, int T, int H) {
    constexpr int V = VEC ? 4 : 1;
    typedef float v_t __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63;
    const long n = (long)B * T;
    // rows in slot order, which is the length order: neighbours read neighbours
    for (long q = blockIdx.x * 4L + (threadIdx.x >> 6); q < n; q += gridDim.x * 4L) {
        const int s = (int)(q / T), t = (int)(q - (long)s * T);
        const int b = perm[s];
        const int L = min(max(lengths[b], 0), T);
        v_t* dst = reinterpret_cast<v_t*>(seq + ((long)b * T + t) * H);
        if (t < L) {
            const v_t* src = reinterpret_cast<const v_t*>(t + 1 < L ? save_h + (long)(offsets[t + 1] + s) * H
                                                                    : out_h + (long)b * H);
#pragma unroll 4
            for (int u = lane; u < H / V; u += 64) dst[u] = src[u];
        } else {
            for (int u = lane; u < H / V; u += 64) dst[u] = v_t{};
        }
    }
}

hipError_t launch_seq_from_saved(const Dims& d, float* seq, const float* save_h, const float* out_h,
                                 const int32_t* lengths, const Workspace& ws, int num_cus,
                                 hipStream_t s) {
    long grid = ((long)d.B * d.T + 3) / 4;
    if (grid > 16L * num_cus) grid = 16L * num_cus;
    const bool vec =
        d.H % 4 == 0 && ((reinterpret_cast<uintptr_t>(seq) | reinterpret_cast<uintptr_t>(out_h)) & 15) == 0;
    auto k = vec ? seq_from_saved_kernel<true> : seq_from_saved_kernel<false>;
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(256), 0, s, seq, save_h, out_h, ws.perm, ws.offsets,
                       lengths, d.B, d.T, d.H);
    return hipGetLastError();
}

hipError_t launch_seq_finish(const Dims& d, float* seq, const int32_t* lengths, int num_cus,
                             hipStream_t s) {
    SeqParams p{seq, lengths, d.B, d.T, d.H};
    const long rows = (long)d.B * d.T;
    long grid = (rows + 3) / 4;
    if (grid > 8L * num_cus) grid = 8L * num_cus;
    if (grid < 1) grid = 1;
    const bool vec = d.H % 4 == 0 && (reinterpret_cast<uintptr_t>(seq) & 15) == 0;
    if (vec)
        hipLaunchKernelGGL(seq_finish_kernel<true>, dim3((unsigned)grid), dim3(256), 0, s, p);
    else
        hipLaunchKernelGGL(seq_finish_kernel<false>, dim3((unsigned)grid), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace ldyn
