// xloop.hip -- host side of the XCD-grouped loop (xloop_kernel.h): which sizes
// take it, and its launch.
#include "xloop_kernel.h"

namespace ldyn {

extern const XVariant kXH16[], kXH16W[], kXF32[];

constexpr int X_GROUP = 32;     // CUs of one XCD: workgroups per group, at most

static const XVariant* find_xvariant(int bf16, int H, int rg) {
    // the narrowest that covers H with 32 workgroups, with room for the rows
    const XVariant* const tables[] = {kXH16, kXH16W, kXF32};
    const XVariant* best = nullptr;
    for (const XVariant* v : tables)
        for (; v->mt; ++v) {
            if (v->bf16 != bf16 || v->hpad < H || 4 * v->mt * X_GROUP < H || 16 * v->nt < rg) continue;
            if (!best || v->hpad < best->hpad || (v->hpad == best->hpad && v->nt < best->nt)) best = v;
        }
    return best;
}

static xloop_fn xloop_of(const XLoopConfig& xc, int cell, int mode) {
    if (!xc.variant || cell < CELL_LSTM || cell > CELL_RNN || mode < LM_PLAIN || mode > LM_SAVE) return nullptr;
    return static_cast<const XVariant*>(xc.variant)->f[cell][mode];
}

// The grouped loop serves whatever a variant covers: bf16 data up to H = 1024
// and fp32 data up to H = 512 (the U of 32 workgroups is 128 registers of each
// product wave there), 32 rows per group (beyond, the device-wide loop's chunks
// are full; with two row tiles the widest variants already spill: 8 to 20
// registers at fp32 H = 512 and 2 to 25 at bf16 H = 1024, with termination or for
// training).  Against the device-wide loop, whole forwards of 100 full steps:
// fp32 H 512, 1 row 314 and 248 us, 8 rows 315 and 269, 16 rows 321 and 268, 64
// rows 527 and 374; H 385, 8 rows 304 and 259; bf16 H 513, 8 rows 259 and 225,
// 24 rows 320 and 231.  The one place where it is not faster is bf16 beyond H =
// 768 with up to 16 rows, where the two are within 4% of each other (H 1024, 8
// rows: 260 and 269 us; with termination 303 and 297, GRU 258 and 247, a training
// step 979 and 882).
bool xloop_pick(const Dims& d, int num_cus, XLoopConfig* xc) {
    *xc = XLoopConfig{};
    int shift = 3;
    while (shift >= 0 && (X_GROUP << shift) > num_cus) --shift;
    if (shift < 0) return false;
    const int rg = (d.B + (1 << shift) - 1) >> shift;
    const XVariant* v = find_xvariant(d.bf16, d.H, rg);
    if (!v) return false;
    xc->variant = v;
    xc->ng_shift = shift;
    xc->gsize = (d.H + 4 * v->mt - 1) / (4 * v->mt);
    xc->rg = rg;
    xc->hpad = v->hpad;
    xc->ugroups = xc->gsize * v->mt;
    xc->ux_bytes = 16LL * xc->ugroups * v->hpad * (d.bf16 ? 2 : 4);
    // the rings of all groups, within the operand buffer of the device-wide loop
    const long long need = 4LL * (rg << shift) * v->hpad, room = 4LL * d.bpad * d.hpad;
    if (need <= room) return true;
    *xc = XLoopConfig{};
    return false;
}

bool xloop_fits(const Dims& d, const XLoopConfig& xc, int mode, int num_cus) {
    xloop_fn f = xloop_of(xc, d.cell, mode);
    if (!f) return false;
    const XVariant* v = static_cast<const XVariant*>(xc.variant);
    int n = 0;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                            v->lds_bytes) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(f), X_WAVES * 64,
                                                     v->lds_bytes) != hipSuccess) {
        (void)hipGetLastError();  // not an error of a later call: the device-wide loop serves
        return false;
    }
    return n >= 1 && (xc.gsize << xc.ng_shift) <= n * num_cus;
}

hipError_t launch_xloop(const Dims& d, const XLoopConfig& xc, const PersistentConfig& pc, const void* U,
                        const float* h0, const float* c0, float* out_h, float* out_c,
                        const Workspace& ws, hipStream_t s) {
    xloop_fn f = xloop_of(xc, d.cell, pc.stop ? LM_STOP : pc.save_h ? LM_SAVE : LM_PLAIN);
    if (!f) return hipErrorInvalidValue;
    XLoopParams p{};
    p.U = U;
    p.ux = ws.ux;
    p.h0 = h0;
    p.c0 = c0;
    p.out_h = out_h;
    p.out_c = out_c;
    p.gx = ws.gx;
    p.hx = ws.hx;
    p.bar = ws.bar;
    p.meta = ws.meta;
    p.perm = ws.perm;
    p.offsets = ws.offsets;
    p.B = d.B;
    p.H = d.H;
    p.ng_shift = xc.ng_shift;
    p.gsize = xc.gsize;
    p.rg = xc.rg;
    p.timeout_ticks = pc.timeout_ticks;
    p.trace = pc.trace;
    p.seq = pc.seq;
    p.T = d.T;
    p.save_h = pc.save_h;
    p.save_c = pc.save_c;
    if (pc.stop) {
        p.stop_v = pc.stop->v;
        p.stop_c = pc.stop->c;
        p.steps = pc.stop->steps;
        p.lengths = pc.stop->lengths;
    }
    void* args[] = {&p};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(f), dim3(xc.gsize << xc.ng_shift),
                                      dim3(X_WAVES * 64), args,
                                      (unsigned)static_cast<const XVariant*>(xc.variant)->lds_bytes, s);
}

}  // namespace ldyn
