// xbwd.hip -- host side of the XCD-grouped reverse loop (xbwd_kernel.h): which
// sizes take it, the packing of U, and its launch.
#include "xbwd_kernel.h"

namespace ldyn {

extern const XBVariant kXBH16[], kXBF32[];

constexpr int XB_GROUP = 32;  // CUs of one XCD: workgroups per group, at most

static const XBVariant* find_xbvariant(int bf16, int H, int rg) {
    const XBVariant* best = nullptr;
    for (const XBVariant* v = bf16 ? kXBH16 : kXBF32; v->mtu; ++v) {
        if (v->kpad < 4 * H || 16 * v->mtu * XB_GROUP < H || 16 * v->nt < rg) continue;
        if (!best || v->kpad < best->kpad || (v->kpad == best->kpad && v->nt < best->nt)) best = v;
    }
    return best;
}

// Whole training steps (MI355X, the path before and this one; the forward, which
// gained 50 to 250 us of it, included; lengths uniform but where full):
//   fp32 H 256, D 256, 32 rows, 100 steps        1201 and 407 us (two launches per step)
//   fp32 H 512, D 512, 64 rows, 100 full steps   2616 and 1294 us
//   bf16 H 512, D 512, 64 rows, 200 steps        1710 and 854 us (the whole-loop launch)
//   bf16 H 768, D 512, 128 rows, 100 full steps  3206 and 1488 us (two launches per step)
//   GRU bf16 H 750, D 200, 37 rows, 61 steps     1228 and 637 us
// In bf16 beyond H = 512 the 64 KB of dz per row tile that every CU reads, and
// spills of the U block (55 to 64 registers with one row tile, 115 to 135 with
// two), cost more than the whole-loop launch's second exchange (H 1024, D 512,
// 200 steps, that launch and this one: 8 rows 1413 and 1729 us, 64 rows 1836 and
// 2178, 256 rows 4106 and 5549), so that launch keeps the one size there that
// both take (H 1024; of the multiples of 256 below it is compiled for 256 and 512).
bool xbwd_pick(const Dims& d, int num_cus, XBwdConfig* xb) {
    *xb = XBwdConfig{};
    int shift = 3;
    while (shift >= 0 && (XB_GROUP << shift) > num_cus) --shift;
    if (shift < 0) return false;
    if (d.bf16 && d.H > 512 && bwd_block_fits(d, num_cus)) return false;
    const int rg = (d.B + (1 << shift) - 1) >> shift;
    const XBVariant* v = find_xbvariant(d.bf16, d.H, rg);
    if (!v) return false;
    xb->ng_shift = shift;
    xb->gsize = (d.H + 16 * v->mtu - 1) / (16 * v->mtu);
    xb->rg = rg;
    xb->kpad = v->kpad;
    xb->urows = xb->gsize * 16 * v->mtu;
    const long long e = d.bf16 ? 2 : 4;
    xb->ux_bytes = e * xb->urows * v->kpad;
    xb->dzx_bytes = 4 * e * v->kpad * (rg << shift);
    xb->dzs_bytes = d.bf16 ? 4LL * 2 * (v->kpad / 32) * (rg << shift) : 0;
    xbwd_fn f = d.cell >= CELL_LSTM && d.cell <= CELL_RNN ? v->f[d.cell] : nullptr;
    int n = 0;
    if (!f ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                            v->lds_bytes) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(f), v->threads,
                                                     v->lds_bytes) != hipSuccess ||
        (xb->gsize << shift) > n * num_cus) {
        (void)hipGetLastError();  // not an error of a later call: another path serves
        *xb = XBwdConfig{};
        return false;
    }
    xb->variant = v;
    return true;
}

// U [H][4H] (gate blocks) -> 1 KB A-fragment blocks, block (rt, kb): rows
// 16 rt .. + 15 of U and one run of gate-interleaved columns (32 in fp16, 16 in
// fp32); chunk q * 16 + r of a block holds row r and the q-th 16 bytes of the
// run.  One wave per row; fp16 rows are scaled by the power of two that brings
// their largest magnitude into [2^13, 2^14), us gets its inverse.  Zero past H
// and past 4H.  The first workgroup also clears the loop's counters and maxima
// and hands the forward's sum of lengths to the host.  Loads are issued eight
// at a time: one by one a row's 4H scalars were 32 memory latencies at H = 512
// (20 us, now 7.5).
template <typename E>
__global__ void __launch_bounds__(256)
xbwd_pack_kernel(const typename E::src_t* __restrict__ U, void* ux, float* us, int H, int urows, int kpad,
                 unsigned* bar, unsigned* amax, const Meta* meta, int32_t* host_rows) {
    using S = typename E::store_t;
    constexpr int CK = 16 / (int)sizeof(S);  // columns per chunk: CK / 4 units
    typedef S chunk_t __attribute__((ext_vector_type(CK)));
    const int tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x == 0) {
        if (tid < BAR_WORDS / 64) {
            bar[64 * tid] = 0u;
            bar[64 * tid + 1] = 0u;
        }
        if (tid < 5) amax[tid] = 0u;
        if (tid == 64)  // (for the host, which waits for an event and not for the stream)
            __hip_atomic_store(host_rows, meta->total_rows, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    const int k = blockIdx.x * 4 + (tid >> 6);
    if (k >= urows) return;
    const typename E::src_t* const row = U + (size_t)(k < H ? k : 0) * 4 * H;
    float sc = 1.0f;
    if constexpr (CK == 8) {
        unsigned m = 0;
        if (k < H) {
#pragma unroll 8
            for (int c = lane; c < 4 * H; c += 64) m = max(m, __float_as_uint((float)row[c]) & 0x7fffffffu);
        }
        for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
        if (m > 0u && __uint_as_float(m) < 3.0e38f)
            sc = __uint_as_float((unsigned)(127 + min(140 - (int)(m >> 23), 126)) << 23);
        if (lane == 0 && k < H) us[k] = __builtin_amdgcn_rcpf(sc);  // a power of two: exact
    }
#pragma unroll 2
    for (int c = lane; c < kpad / CK; c += 64) {
        chunk_t v;
#pragma unroll
        for (int e = 0; e < CK; ++e) {
            const int u = c * (CK / 4) + (e >> 2);
            const float x = k < H && u < H ? (float)row[(size_t)(e & 3) * H + u] : 0.0f;
            v[e] = (S)(x * sc);
        }
        static_cast<chunk_t*>(ux)[((size_t)(k >> 4) * (kpad / (4 * CK)) + (c >> 2)) * 64 + (c & 3) * 16 + (k & 15)] = v;
    }
}

hipError_t launch_xbwd_pack(const Dims& d, const XBwdConfig& xb, const void* U, void* ux, float* us,
                            unsigned* bar, unsigned* amax, const Meta* meta, int32_t* host_rows,
                            hipStream_t s) {
    const dim3 grid((unsigned)((xb.urows + 3) / 4));
    if (d.bf16)
        hipLaunchKernelGGL(xbwd_pack_kernel<EltH16>, grid, dim3(256), 0, s, static_cast<const __bf16*>(U), ux, us,
                           d.H, xb.urows, xb.kpad, bar, amax, meta, host_rows);
    else
        hipLaunchKernelGGL(xbwd_pack_kernel<EltF32>, grid, dim3(256), 0, s, static_cast<const float*>(U), ux, us,
                           d.H, xb.urows, xb.kpad, bar, amax, meta, host_rows);
    return hipGetLastError();
}

hipError_t launch_xbwd(const Dims& d, const XBwdConfig& xb, const void* ux, const float* us,
                       const float* save_h, const float* save_c, const float* dseq, const float* d_out_h,
                       const float* d_out_c, float* dh0, float* dc0, void* dzx, void* dzs, unsigned* amax_dz,
                       unsigned* bar, unsigned long long timeout_ticks, unsigned long long* trace,
                       const Workspace& ws, hipStream_t s) {
    const XBVariant* v = static_cast<const XBVariant*>(xb.variant);
    if (!v || d.cell < CELL_LSTM || d.cell > CELL_RNN) return hipErrorInvalidValue;
    XBwdParams p{};
    p.ux = ux;
    p.us = us;
    p.gx = ws.gx;
    p.save_h = save_h;
    p.save_c = save_c;
    p.dseq = dseq;
    p.d_out_h = d_out_h;
    p.d_out_c = d_out_c;
    p.perm = ws.perm;
    p.offsets = ws.offsets;
    p.meta = ws.meta;
    p.dzx = dzx;
    p.dzs = static_cast<unsigned short*>(dzs);
    p.dh0 = dh0;
    p.dc0 = dc0;
    p.amax = amax_dz;
    p.bar = bar;
    p.timeout_ticks = timeout_ticks;
    p.trace = trace;
    p.B = d.B;
    p.H = d.H;
    p.T = d.T;
    p.ng_shift = xb.ng_shift;
    p.gsize = xb.gsize;
    p.rg = xb.rg;
    void* args[] = {&p};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(v->f[d.cell]), dim3(xb.gsize << xb.ng_shift),
                                      dim3(v->threads), args, (unsigned)v->lds_bytes, s);
}

}  // namespace ldyn
