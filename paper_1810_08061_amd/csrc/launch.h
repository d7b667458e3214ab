// launch.h -- host-side launchers of the kernels (one translation unit per
// kernel family) and the device workspace they share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace ldyn {

// Device workspace of one handle (all pointers into one hipMalloc block).
struct Workspace {
    Meta* meta;         // loop bound, row count, status
    int32_t* perm;      // [B] slot -> batch index; slots sorted by length, descending (stable)
    int32_t* offsets;   // [T_max + 1] first compact row of step t; offsets[t+1]-offsets[t] = active rows
    int32_t* rowsrc;    // [B * T_max] compact row -> b * T_max + t
    float* gx;          // [B * T_max][4H] x W + b for valid (b, t), gate-interleaved columns
    void* hx;           // [4][bpad][hpad] recurrent operand (dtype), slot order; row-major in two
                        // buffers for the per-step path, MFMA fragment order in four for the persistent loop
    unsigned* bar;      // grid-barrier counters: [0] global, [64 * (1 + x)] group x, and a word of flags
                        // after each (zeroed by prep)
    float* z;           // [bpad][4H] per-step pre-activations (per-step mode only)
    void* wt;           // bf16: W transposed to [np][dp] (gate-interleaved rows, zero padded)
    void* ux;           // U in A-fragment blocks for the XCD-grouped loop, or null
    int32_t* stopped;   // [B] per-step path, termination from the state: 1 once row b ended
    int32_t* running;   // [T_max] per-step path: rows still running after step t
};

struct Dims {
    int B, D, H, T;     // batch, input width, hidden width, padded time extent
    int bf16;           // 1: x, W, U are bf16; 0: fp32
    int hpad, bpad;     // padded hidden width / batch rows of the operand buffer
    int cell;           // CellKind; GRU and RNN weights are packed into the LSTM's four gate blocks
};

// GRU and RNN: the caller's weights packed into the four gate blocks of the
// LSTM path (d.cell selects the packing).  GRU: W [D][3H], U [H][3H] (gate
// blocks r, u, n), b [6H] = b_ih ++ b_hh -> W4 [D][4H] = (W_r, W_u, 0, W_n),
// U4 [H][4H] = (U_r, U_u, U_n, 0), b4 [4H] = (b_ir + b_hr, b_iu + b_hu, b_hn,
// b_in).  RNN: W [D][H], U [H][H], b [H] -> (W, 0, 0, 0), (U, 0, 0, 0),
// (b, 0, 0, 0).
hipError_t launch_cell_pack(const Dims& d, const void* W, const void* U, const float* b, void* W4,
                            void* U4, float* b4, hipStream_t s);

// Preparation: clamp and validate lengths, stable descending length sort,
// per-step active counts and compact row offsets, compact row sources.
// stop: rows may end before their lengths, so the steps that some row ran
// (meta->iters) start at zero for the loop to count.
// With U and ws.ux, further workgroups of the launch write U for the
// XCD-grouped loop: 1 KB blocks, block (ug, kb) the MFMA A-fragment of units
// 4 ug .. 4 ug + 3 (16 gate-interleaved columns) and one run of k (32 in fp16,
// 16 in fp32), zero past H; xc gives the padded sizes.
struct XLoopConfig;
hipError_t launch_prep(const Dims& d, const int32_t* lengths, const Workspace& ws, hipStream_t s,
                       bool stop = false, const void* U = nullptr, const XLoopConfig* xc = nullptr);

// The workspace of a persistent-mode LSTM forward carved from caller memory
// (api.hip): returns its bytes; fills ws when base is not null.
// ux_bytes: room for the packed U, or 0 for none.
long long carve_forward_workspace(const Dims& d, char* base, Workspace* ws, long long* hx_off,
                                  long long* hx_bytes, long long ux_bytes);

// Input projection over all valid (b, t): gx[r][c'] = x[rowsrc[r]] . W[:, col(c')] + b[col(c')].
// (fp32 data)
hipError_t launch_inproj(const Dims& d, const void* x, const void* W, const float* b,
                         const Workspace& ws, int num_cus, hipStream_t s);

// bf16 input projection: W -> Wt, then the tiled GEMM (inproj.hip).
void inproj_bf16_wt_shape(const Dims& d, int* np, int* dp);
int inproj_bf16_tiles_max(const Dims& d);
hipError_t inproj_bf16_setup();
hipError_t launch_transpose_w(const Dims& d, const void* W, const Workspace& ws, hipStream_t s);
hipError_t launch_inproj_bf16(const Dims& d, const void* x, const float* b, const Workspace& ws,
                              int grid, hipStream_t s);

// Persistent on-device time loop.
// Termination computed from the state: a row ends after a step that leaves
// its halting score v . h + c positive.
struct StopArgs {
    const float* v;          // [H]
    float c;
    int32_t* steps;          // [B] (batch order), written: the steps each row ran
    const int32_t* lengths;  // [B] caps
};

struct PersistentConfig {
    int mt, groups, ksw, kw, nst, lds_bytes;
    unsigned long long timeout_ticks;  // barrier wait bound in wall-clock ticks
    unsigned long long* trace;         // per-step timestamps (diagnostics) or null
    float* seq;                        // output sequence [B][T][H]: each step's h of the rows that
                                       // ran it (zeros past them written afterwards), or null
    const StopArgs* stop;              // termination from the state, or null
    float* save_h;                     // forward for training: the state each step starts from,
    float* save_c;                     // [compact rows][H] (z is kept in place of Gx); else null
};
constexpr int BAR_WORDS = 64 * 9;  // global + 8 group counters, 256 bytes apart
hipError_t launch_persistent(const Dims& d, const PersistentConfig& pc, const void* U,
                             const float* h0, const float* c0, float* out_h, float* out_c,
                             const Workspace& ws, hipStream_t s);
// Occupancy check for the co-resident grid; returns blocks per CU (0 if none).
// mode: 0 plain, 1 termination from the state, 2 forward for training
int persistent_blocks_per_cu(int bf16, int mt, int ksw, int kw, int nst, int lds_bytes, int cell,
                             int mode);
// Compiled variant with exactly (mt, kw, ksw) and the smallest state capacity >= nstate.
bool persistent_pick_variant(int bf16, int mt, int kw, int ksw, int nstate, int* nst);
int persistent_lds_bytes(int bf16, int mt, int kw, int nst, int hpad);

// The loop in one group of workgroups per XCD (xloop.hip), where all of U fits
// the CUs of one XCD and the batch its row tiles.
struct XLoopConfig {
    const void* variant;  // the compiled variant, or null: the device-wide loop
    int ng_shift;         // 1 << ng_shift groups; rows are dealt to them by slot
    int gsize;            // workgroups per group
    int rg;               // rows per group, at most
    int hpad, ugroups;    // the packed U: padded K, groups of four units; its bytes
    long long ux_bytes;
};
// Whether the sizes take the grouped loop on a device of num_cus CUs; fills xc.
bool xloop_pick(const Dims& d, int num_cus, XLoopConfig* xc);
// Whether its grid is resident at once (mode: LoopMode).
bool xloop_fits(const Dims& d, const XLoopConfig& xc, int mode, int num_cus);
hipError_t launch_xloop(const Dims& d, const XLoopConfig& xc, const PersistentConfig& pc, const void* U,
                        const float* h0, const float* c0, float* out_h, float* out_c,
                        const Workspace& ws, hipStream_t s);

// xloop_pick and xloop_fits; and either loop's launch, by xc.variant.
bool xloop_for(const Dims& d, int mode, int num_cus, XLoopConfig* xc);
hipError_t launch_loop(const Dims& d, const XLoopConfig& xc, const PersistentConfig& pc, const void* U,
                       const float* h0, const float* c0, float* out_h, float* out_c,
                       const Workspace& ws, hipStream_t s);

// Whole forward in one single-workgroup launch (H <= 32).
bool small_pick(int bf16, int B, int D, int H, int* kd, int* nt);
hipError_t launch_small(const Dims& d, int kd, int nt, const void* x, const int32_t* lengths,
                        const void* W, const void* U, const float* b, const float* h0,
                        const float* c0, float* out_h, float* out_c, float* seq,
                        const StopArgs* stop, const Workspace& ws, hipStream_t s);

// Per-step comparison path.
hipError_t launch_step_init(const Dims& d, const float* h0, const float* c0, float* out_h,
                            float* out_c, const Workspace& ws, hipStream_t s);
hipError_t launch_step_gemm(const Dims& d, int t, const void* U, const Workspace& ws, hipStream_t s);
hipError_t launch_step_gates(const Dims& d, int t, float* out_h, float* out_c, float* seq,
                             bool stop, const Workspace& ws, hipStream_t s,
                             float* save_h = nullptr, float* save_c = nullptr);
// Termination from the state on the per-step path: init (steps = caps, no row
// ended, counters zero), then after the gates of each step the halting scores
// of the rows that ran; running[t] counts the rows that run at step t + 1.
hipError_t launch_step_stop_init(const Dims& d, const StopArgs& stop, const Workspace& ws,
                                 hipStream_t s);
hipError_t launch_step_stop(const Dims& d, int t, const StopArgs& stop, const Workspace& ws,
                            hipStream_t s);

// Backward pass (bwd.hip).
hipError_t launch_bwd_weights(const Dims& d, const void* W, int rows, float* Wil, hipStream_t s);
hipError_t launch_bwd_init(const Dims& d, const float* dh_out, const float* dc_out, float* dH,
                           float* dC, const Workspace& ws, hipStream_t s);
// off, act: the step's first compact row and its number of rows (known to the
// host from the forward's step offsets).
hipError_t launch_bwd_cell(const Dims& d, int t, int off, int act, const float* save_h,
                           const float* save_c,
                           const float* dseq, float* dH, float* dC, const Workspace& ws,
                           hipStream_t s);
hipError_t launch_bwd_state_out(const Dims& d, const float* dH, const float* dC, const float* srow,
                                float* dh0, float* dc0, const Workspace& ws, hipStream_t s);
// bf16 data: the cell's backward with one workgroup per row, also writing the
// row's dz in fp16 scaled by a power of two (srow) for dz U^T.
hipError_t launch_bwd_cell16(const Dims& d, int t, int off, int act, const float* save_h,
                             const float* save_c, const float* dseq, float* dH, float* dC,
                             float* srow, _Float16* dz16, const Workspace& ws, hipStream_t s);
hipError_t launch_bwd_ones(float* a, int n, hipStream_t s);
// bf16 data: the reverse loop over steps max_len - 1 .. t_end in one
// cooperative launch (one workgroup of 8 units per CU, those units' rows of U
// in LDS, each step's dz published in fp16 with a power-of-two scale per row
// and 32-column block, one grid barrier per step), leaving in dH the
// gradient entering step t_end - 1.  bwd_loop_fits: its workgroup count, or
// 0 where it does not apply (H odd, below 16 or above 2048, more than 512
// rows, not all resident).
// dzx [2][bpad][kp] fp16, dzs [2][bpad][nblk] and bar [9 * 64] must be zero
// at the launch; dH, dC hold the upstream gradients (slot order) and receive
// dh0, dc0.
int bwd_loop_fits(const Dims& d, int num_cus);
void bwd_loop_shape(int H, int* kp, int* nblk);
hipError_t launch_bwd_loop(const Dims& d, const _Float16* u16, float alpha_u, const float* save_h,
                           const float* save_c, const float* dseq, float* dH, float* dC,
                           _Float16* dzx, float* dzs, unsigned* bar, unsigned long long timeout_ticks,
                           int t_end, const Workspace& ws, hipStream_t s);
// bf16 data, H 256, 512, 1024 or 2048: the whole reverse loop in one
// cooperative launch (H / 8 workgroups, each with a 32-unit x H-column block
// of U in registers; per step the blocks' shares of dh = dz U^T, then the
// cell's backward of 8 units, each exchange polled for, no grid barrier),
// leaving dh0 and dc0 in dH and dC.  bwd_block_fits: its workgroup count, or
// 0 where it does not apply.  dzx [4][bpad][4H] fp16, dzs [4][bpad][H / 8]
// and pdh [4][4][bpad][H] must be all ones (the marker) at the launch; trace
// [T + 1][4] or null.  amax_dz receives the largest |dz| over all compact
// rows (float bits, atomic maximum: it must hold 0 or a lower bound).
int bwd_block_fits(const Dims& d, int num_cus);
hipError_t launch_bwd_block(const Dims& d, const _Float16* u16, float alpha_u, const float* save_h,
                            const float* save_c, const float* dseq, float* dH, float* dC, _Float16* dzx,
                            float* dzs, float* pdh, unsigned* amax_dz, unsigned long long timeout_ticks,
                            unsigned long long* trace, const Workspace& ws, hipStream_t s);
// The reverse loop in one group of workgroups per XCD (xbwd.hip), for persistent
// handles where all of U fits the CUs of one XCD: one cooperative launch for
// every step, dh0 and dc0 written to the caller's buffers.  xbwd_pick: false
// where it does not apply.  launch_xbwd_pack fills ux (ux_bytes) and us [H]
// (bf16 data) from U [H][4H] in gate blocks, clears bar and amax [5] and puts
// the forward's sum of lengths into host_rows (pinned); dzx and dzs need no
// contents.
struct XBwdConfig {
    const void* variant;  // the compiled variant, or null
    int ng_shift, gsize, rg;  // as in XLoopConfig
    int kpad, urows;          // padded 4H; rows of U that the groups hold
    long long ux_bytes, dzx_bytes, dzs_bytes;
};
bool xbwd_pick(const Dims& d, int num_cus, XBwdConfig* xb);
hipError_t launch_xbwd_pack(const Dims& d, const XBwdConfig& xb, const void* U, void* ux, float* us,
                            unsigned* bar, unsigned* amax, const Meta* meta, int32_t* host_rows,
                            hipStream_t s);
hipError_t launch_xbwd(const Dims& d, const XBwdConfig& xb, const void* ux, const float* us,
                       const float* save_h, const float* save_c, const float* dseq, const float* d_out_h,
                       const float* d_out_c, float* dh0, float* dc0, void* dzx, void* dzs, unsigned* amax_dz,
                       unsigned* bar, unsigned long long timeout_ticks, unsigned long long* trace,
                       const Workspace& ws, hipStream_t s);
// Operands of the GEMMs over all compact rows: xh [rows][D + H] (x, then the h
// each step started from) and w [D][4H] (gate-interleaved), fp32, or fp16 with
// bf16 data: scaled from amax[1..3] (|x|, |h|, |W| as float bits), which this
// fills (two launches).  amax has BWD_MAX_WORDS words, those from BWD_MAX_AT on
// for its use.  max_rows: B * T (grid sizes only).
constexpr int BWD_MAX_PARTS = 512, BWD_MAX_AT = 64, BWD_MAX_WORDS = BWD_MAX_AT + 3 * BWD_MAX_PARTS;
hipError_t launch_bwd_operands(const Dims& d, const void* x, const void* W, const float* save_h,
                               long max_rows, void* xh, void* w, unsigned* amax, const Workspace& ws,
                               hipStream_t s);
// Largest magnitude (as float bits, atomic and order free), a scaled conversion.
hipError_t launch_bwd_absmax(const float* a, long n, unsigned* out, hipStream_t s);
hipError_t launch_bwd_to_f16(const float* src, _Float16* dst, long n, float scale, hipStream_t s);
// part [BWD_CS_CHUNKS][ncols]: partial column sums of dz [rows][ncols] (ncols a
// multiple of 4); with dz16, also dz16 = fp16(dz scaled from *amax).
constexpr int BWD_CS_CHUNKS = 64;
hipError_t launch_bwd_colsum(const float* dz, long rows, int ncols, float* part, _Float16* dz16,
                             const unsigned* amax, hipStream_t s);
// dW, dU, db in the cell's own layout from il [(D + H)][4H] (gate-interleaved;
// null: no compact row) and part; amax: the fp16 operands' maxima, or null.
hipError_t launch_bwd_grads(const Dims& d, const float* il, const float* part, const unsigned* amax,
                            float* dW, float* dU, float* db, hipStream_t s);
// dx [B][T][D] from its compact rows (amax as above).
hipError_t launch_bwd_dx(const Dims& d, const float* dxc, const int32_t* lengths, const unsigned* amax,
                         float* dx, const Workspace& ws, hipStream_t s);
// Forward for training from the saved state: out_seq[b][t] for t < L[b]
// (the state after step t is the one step t + 1 started from, or out_h).
hipError_t launch_seq_from_saved(const Dims& d, float* seq, const float* save_h, const float* out_h,
                                 const int32_t* lengths, const Workspace& ws, int num_cus,
                                 hipStream_t s);

// Output sequence: zeros past each row's last step (lengths: that step + 1;
// the loops write the valid steps themselves).
hipError_t launch_seq_finish(const Dims& d, float* seq, const int32_t* lengths, int num_cus,
                             hipStream_t s);

}  // namespace ldyn
