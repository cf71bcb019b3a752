// Internal declarations shared by the translation units of libssd_magc (not part of the ABI).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ssd_magc.h"

namespace ssdk {

// bf16 storage as raw bits; conversion is round-to-nearest-even.
struct bf16_t {
    uint16_t v;
};

__host__ __device__ inline float bf16_to_float(bf16_t b) {
    union {
        uint32_t u;
        float f;
    } c;
    c.u = (uint32_t)b.v << 16;
    return c.f;
}

__host__ __device__ inline bf16_t float_to_bf16(float f) {
    union {
        uint32_t u;
        float f;
    } c;
    c.f = f;
    bf16_t o;
    if ((c.u & 0x7fffffffu) > 0x7f800000u) {  // NaN stays NaN
        o.v = (uint16_t)((c.u >> 16) | 0x40u);
    } else {
        o.v = (uint16_t)((c.u + 0x7fffu + ((c.u >> 16) & 1u)) >> 16);
    }
    return o;
}

// The step sizes as a block's input projection leaves them: dt = softplus(dt + bias), rounded to the storage type; rows rs
// elements apart, one batch.  dt NULL: none.
struct RawDt {
    const void* dt;
    int64_t rs;
    const float* bias;
};
// max(v, 0) + log(1 + e^-|v|): no overflow
static __device__ __forceinline__ float softplus(float v) { return fmaxf(v, 0.f) + log1pf(__expf(-fabsf(v))); }

// Sums over a wave by lane exchanges of the vector ALUs: rows of 16 lanes, then across the rows.  Every lane ends with
// the sum of the lanes up to its own (lane 63: of all).
template <int CTRL, int ROWS>
static __device__ __forceinline__ float dpp_add(float v) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, true));
}
static __device__ __forceinline__ float wave_prefix(float v) {
    v = dpp_add<0x111, 0xF>(v);  // row_shr:1
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}
// The sum over the wave, in every lane.
static __device__ __forceinline__ float wave_total(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_prefix(v)), 63));
}

// One span of one layer, as the kernels see it: one or several consecutive checkpoint segments that share their
// launches.  Tensor pointers are already offset to the first token of the span; batch strides are those of the
// full tensors (elements).
struct SegParams {
    int Bt, H, P, G, N, Q, nc, hpg;    // nc: chunks of the span (the last one possibly ragged)
    int ntok;                          // tokens of the span, <= nc Q: rows beyond them do not exist in memory
    int seg_chunks;                    // chunks per checkpoint segment (== nc when the span is one segment)
    int64_t xs_b, ys_b, dys_b, dxs_b;  // batch strides of x, y, dy, dx
    int64_t dts_b, bcs_b;              // of dt/ddt and of B/C/dB/dC
    const uint8_t* reset;              // optional [Bt][tokens of the segment]: non-zero = a packed sequence starts here
    int64_t reset_bs;                  // its batch stride
    uint32_t flags;
    int accumulate;                    // bwd: 1 = add the call's dA / dD to what is there
    // inputs / outputs
    const void* x;
    const void* dt;
    const void* Bm;
    const void* Cm;
    const void* dy;
    const float* A;
    const float* D;
    void* y;
    void* dx;
    void* ddt;
    void* dB;
    void* dC;
    // per-segment workspace (fp32)
    float* cum;        // [Bt][H][nc][Q]  chunk-local inclusive cumsum of dt*A
    float* dtf;        // [Bt][H][nc][Q]  dt as fp32, head-major
    float* states;     // generic path only: [Bt][nc+1][H][P][N]  slot c: state entering chunk c; slot nc: state leaving the segment
    float* dstates;    // generic path only: [Bt][nc][H][P][N]    slot c: adjoint of the state leaving chunk c
    float* Gm;         // [Bt][nc][G][Q][Q]    C_i . B_j   (generic path: fp32)
    float* dG;         // generic path: [Bt][nc][G][dg_split][Q][Q] fp32 per-slice sums of masked dY X^T; MFMA path: [Bt][nc][G][dg_split][Q/32][Q/32][32][32] per-slice sums, tile by tile, bf16 or (dg_f32) fp32
    // Per-token scalars; on the generic path gterm, sterm, erow, ecol, fterm and dDrow are partial sums over pieces of 32
    // columns (or rows) of a tile, piece k at k tok_stride.
    int64_t tok_stride;
    float* gterm;      // [Bt][H][nc][Q]  gradient of cum, per token: the part through the entering state
    float* sterm;      // [Bt][H][nc][Q]  dt_j x_j . (part of u_j through the leaving adjoint); subtracted
    float* gintra;     // [Bt][H][nc][Q]  MFMA path: chunk-local part (row sums minus column sums of E); added
    float* erow;       // generic path: row sums of E, piece k = columns 32 k ..
    float* ecol;       // generic path: column sums of E, piece k = rows 32 k ..
    float* fterm;      // [Bt][H][nc][Q]
    float* dDrow;      // [Bt][H][nc][Q]
    float* tail_part;  // [Bt][H][nc][nslice]
    float* dA_part;    // [Bt][nc_total][H]
    float* dD_part;    // [Bt][nc_total][H]
    float* dcarry;     // [Bt][H][P][N] adjoint of the state entering the span to the right of the current one
    const float* dcarry_in;  // where the reverse scan starts from: dcarry, the caller's dfinal_state, or NULL for zeros
    int nslice;
    int param_stride;  // see param_count
    // extra scratch of the MFMA path
    float* ein;        // [Bt][H][nc][Q] exp(cum_i - cum at the start of i's 64-token block)
    float* eout;       // [Bt][H][nc][Q] exp(cum at the end of j's 64-token block - cum_j)
    bf16_t* states_bf;   // [Bt][nc][H][P][N] chunk states, replaced in place by the states entering the chunks (bf16 only)
    bf16_t* dstates_bf;  // [Bt][nc][H][P][N] local state adjoints, replaced in place by the adjoints of the leaving states
    int dg_split;        // number of head slices whose dG / dB / dC partial sums are kept apart
    int dg_f32;          // MFMA path: the partial sums of dG are kept in fp32 (see fit_splits)
    int dual_split;      // number of head slices per (batch, chunk, group) in the dual-form kernels (backward, 0: chosen at the launch)
    int part_split;      // number of head slices of the dB / dC head sums
    int outer_split;     // number of head slices of the chunk-state / local-adjoint kernel
    int part_alternate;  // the head-sum pass alternates between the halves of its slice (see part_body)
    int wg_target;       // least number of workgroups a persistent-over-heads launch should have
    int first_span;      // bwd: 1 = the first span of a call that the reverse scan walks
    float* dbc_part;     // [Bt][nc][G][part_split][2][Q][N] per-slice head terms of dC (0) and dB (1)
    // state plumbing for the scans (all fp32, element strides between batches)
    const float* state_in;   // state entering the span, or NULL for zeros
    int64_t state_in_bs;
    float* bnd_write;        // where to store that entering state (checkpoint slot), or NULL
    int64_t bnd_write_bs;
    // checkpoints between the segments of a span: slot of segment q >= 1 of the span at q H P N elements, batches
    // ckpt_bs apart; written by the forward pass (ckpt / ckpt16 where the caller keeps them), read by the backward
    // pass, which restarts every segment from its slot
    float* ckpt;
    bf16_t* ckpt16;
    int64_t ckpt_bs;
    float* state_out;        // where to store the state leaving the span, or NULL
    int64_t state_out_bs;
    float* state_out2;       // second copy (final_state when the last segment also has no slot), or NULL
    int64_t state_out2_bs;
    // bf16 checkpoints: the entering state comes from (state_in16, used when state_in is NULL) or goes to
    // (bnd_write16, state_out16) a bf16 slot; strides as for their fp32 counterparts
    const bf16_t* state_in16;
    bf16_t* bnd_write16;
    bf16_t* state_out16;
    int64_t state_out16_bs;
    float* dinit_out;        // bwd: where the adjoint of the entering state goes at segment 0, or NULL
    float* dA;
    float* dD;
    // dA / dD partial sums: slot (b, chunk0 + c, h) of an array with nc_total chunks per batch, by default (0 and nc) one
    // span's; where one array serves all spans of a call, they may run concurrently.  param_count[h param_stride]: chunks of
    // head h that have left theirs, a cache line apart where they fit so (24 heads in one line took 7 us of a launch of 15).
    // The reverse scan of a call's first span, which every finalisation follows, sets it to zero (first_span); the chunk that
    // makes it full sums them (ddt_finalize.h).
    int chunk0, nc_total;
    int* param_count;
    // optional cross-stream ordering of the state scans (consecutive segments run on different streams):
    // the scan waits for ev_wait and records ev_record when it has been enqueued
    hipEvent_t ev_wait, ev_record;
    // dt as it leaves a projection (raw.dt set: dt is not read).  Last: in the middle it moved what the small kernels load first
    // off its cache lines (512 fp32 tokens of 4 heads, eight launches: 64.2 -> 64.7 us)
    RawDt raw;
#ifdef SSDK_STAMPS
    unsigned long long* stamps;  // diagnostics build: cycle stamps of the head loops (see SSDK_STAMP)
#endif
};

// Diagnostics build (-DSSDK_STAMPS): wave 0 of the first eight workgroups of a head-walking kernel writes the
// shader cycle counter at six points of every head iteration, slot (body, workgroup, head, point).
#ifdef SSDK_STAMPS
extern unsigned long long* g_stamps;
#define SSDK_STAMP(body, id)                                                                              \
    do {                                                                                                  \
        if (sp.stamps && lane == 0 && w == 0 && zlog < 8 && hh < 64)                                      \
            sp.stamps[((((body)) * 8 + zlog) * 64 + hh) * 16 + (id)] = __builtin_readcyclecounter();      \
    } while (0)
#else
#define SSDK_STAMP(body, id) \
    do {                     \
    } while (0)
#endif

// Tokens of chunk c that exist (the last chunk of a sequence may be ragged): its further rows read as zeros
// under dt = 0, i.e. they are identity steps of the recurrence, and are never stored.
__host__ __device__ inline int chunk_rows(const SegParams& sp, int c, int Q) {
    const int left = sp.ntok - c * Q;
    return left < Q ? left : Q;
}

// Validated dimensions of one call.
struct Dims {
    int64_t Bt, L, s;
    int H, P, G, N, Q, nc, hpg;
    int64_t nseg;       // segments, the last one possibly short
    // the launch plan (plan_dims): span k = segments [k F, (k + 1) F), on lane k % nl
    int nc_seg;         // chunks per segment
    int F, nl;          // segments per span, spans in flight
    bool dg_f32;        // workspace for partial sums of dG in fp32 on the matrix-core path
    int64_t nspan;
    int64_t nct;        // chunks of the sequence; nc above: chunks of the largest span
    size_t esz;
    bool bf16;
    int64_t xs_b, dts_b, bcs_b;
    const uint8_t* reset;  // optional packed-sequence flags [Bt][L]
};

// What a packed-sequence start adds to the token's log-decay dt*A: exp(-100) < 4e-44 cuts the state off
// (and with it every gradient path through it) while every decay factor stays a product of factors <= 1.
constexpr float RESET_LOG_DECAY = -100.f;

// Byte offsets of the per-segment scratch arrays inside the caller's workspace (WS_NONE: the array
// does not exist on the chosen kernel path and its pointer stays null).
constexpr size_t WS_NONE = ~(size_t)0;
constexpr int GENERIC_SLICES = 4;  // head slices of the shape-generic kernels' partial sums, at most
struct WsLayout {
    size_t cum, dtf, states, Gm, dstates, dG, gterm, fterm, dDrow, tail_part, dA_part, dD_part, dcarry, total;
    size_t ein, eout, states_bf, dstates_bf, dbc_part, sterm, gintra, erow, ecol, tok;
    int nslice;
};

int check_shape(const ssd_shape_t* sh, Dims* d);
// Chooses segments per launch and launches in flight (fills nc and the launch plan).
void plan_dims(Dims* d, bool mfma, bool one_stream);
// mfma: the layout for the matrix-core kernels, which keep the chunk states and their adjoints in
// bf16 only (the fp32 arrays of the shape-generic kernels are left out).
// fp32cs: the matrix-core layout keeps fp32 chunk states / local adjoints beside the bf16 operand copies.
WsLayout ws_layout(const Dims& d, bool bwd, bool mfma, int wg_target = 256, bool fp32cs = false);
void bind_workspace(SegParams& sp, const WsLayout& w, void* workspace, bool bwd);
// Head slices of the backward passes for a span of sp.nc chunks.
void fit_splits(SegParams& sp, const Dims& d, bool mfma, int wg_target);
void base_params(SegParams& sp, const Dims& d, uint32_t flags);
bool use_mfma(const ssd_shape_t& sh, uint32_t flags);

// Kernel ids for the optional event timing (see prof.hip).
enum KernelId {
    K_CHUNK_STATE, K_SCAN_FWD, K_CHUNK_OUT, K_SCAN_BWD, K_BWD_MAIN, K_DBC, K_FILL, K_COPY,
    K_MFMA_CHUNK_STATE, K_MFMA_CHUNK_OUT, K_MFMA_DSTATE, K_MFMA_BWD_MAIN, K_MFMA_DG, K_MFMA_DBC, K_MFMA_BWD_TRIO,
    K_MFMA_FINAL_DDT, K_COUNT
};
// When timing of kernel `kid` is enabled: a pair of events for the launch to fill in (kernel start
// and end, as the command processor stamps them -- the time the launch waits behind other work is
// not part of it); otherwise false.
bool prof_events(int kid, hipEvent_t* start, hipEvent_t* stop);

// Launch on `st`, timed when enabled; returns the launch error from the enclosing function.
#define SSDK_LAUNCH_LDS(kid, st, kernel, grid, block, lds, ...)                               \
    do {                                                                                      \
        hipEvent_t ea_ = nullptr, eb_ = nullptr;                                              \
        if (::ssdk::prof_events(kid, &ea_, &eb_))                                             \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, st, ea_, eb_, 0, __VA_ARGS__);    \
        else                                                                                  \
            hipLaunchKernelGGL(kernel, grid, block, lds, st, __VA_ARGS__);                    \
        hipError_t e_ = hipGetLastError();                                                    \
        if (e_ != hipSuccess) return e_;                                                      \
    } while (0)
#define SSDK_LAUNCH(kid, st, kernel, grid, block, ...) SSDK_LAUNCH_LDS(kid, st, kernel, grid, block, 0, __VA_ARGS__)

// Launchers.  Each returns hipSuccess or the launch error.  is_bf16 selects the storage type.
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t st);
hipError_t launch_copy_f32(float* dst, const float* src, size_t n, hipStream_t st);
hipError_t generic_forward_segment(const SegParams& sp, bool is_bf16, bool need_y, hipStream_t st);
hipError_t generic_backward_segment(const SegParams& sp, bool is_bf16, hipStream_t st);

// MFMA path (bf16, P = 64, N = 128, Q in {64, 128, 256}).
bool mfma_path_supported(const ssd_shape_t& s);
hipError_t mfma_forward_segment(const SegParams& sp, bool need_y, hipStream_t st);
hipError_t mfma_backward_segment(const SegParams& sp, hipStream_t st);
// One dual-form pass over a segment: epi 0 = forward output, 2 = the backward pass (chunks of 64).
hipError_t mfma_launch_dual(const SegParams& sp, int epi, hipStream_t st);
// dG, the head sums and the final contraction that give dB and dC of one segment.
hipError_t mfma_launch_grad_bc(const SegParams& sp, hipStream_t st);
// Smallest divisor ns of heads_per_group with base * ns >= target workgroups (else heads_per_group).
int pick_split(int heads_per_group, int64_t base, int target);
// The heads of slice i of ns: slices of equal length, or of two lengths one apart, the longer first.
struct Slice {
    int first, n;
};
__host__ __device__ inline Slice slice_of(int heads, int ns, int i) {
    const int q = heads / ns, r = heads - q * ns;
    return {q * i + (i < r ? i : r), q + (i < r ? 1 : 0)};
}
// Slices for a launch that has the machine to itself (see api.hip).
int pick_rounds(int heads_per_group, int64_t base, int per_unit, int prologue);

// The block's convolution with its output (forward) or the gradient of its output (backward) given as three
// dense tensors side by side -- channels [0, c1), [c1, c2), [c2, C) with rows c1, c2 - c1, C - c2 apart: the
// x | B | C operands of the scan and their gradients -- instead of one [L, C] tensor.  Otherwise as
// ssd_conv1d_fwd / ssd_conv1d_bwd.
struct ConvSplit {
    void* p[3];
    int c1, c2;
};
int conv1d_fwd_split(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in,
                     const ConvSplit& out, void* state_out, hipStream_t st);
int conv1d_bwd_split(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in,
                     const ConvSplit& dout, const float* dstate_out, void* du, float* dw, float* dbias, float* dstate_in,
                     void* workspace, size_t workspace_bytes, uint32_t flags, hipStream_t st);

// ssd_fwd / ssd_bwd with the step sizes still to be formed (raw.dt set: dt is ignored; batch 1).
int scan_fwd(const ssd_shape_t* shape, const void* x, const void* dt, const RawDt& raw, const float* A, const void* B, const void* C,
             const float* D, const float* init_state, void* y, float* final_state, void* boundary_states, void* workspace,
             size_t workspace_bytes, uint32_t flags, hipStream_t st);
int scan_bwd(const ssd_shape_t* shape, const void* x, const void* dt, const RawDt& raw, const float* A, const void* B, const void* C,
             const float* D, const float* init_state, const void* dy, const float* dfinal_state, const void* boundary_states, void* dx,
             void* ddt, float* dA, void* dB, void* dC, float* dD, float* dinit_state, void* workspace, size_t workspace_bytes,
             uint32_t flags, hipStream_t st);

// sum = a + b, rounded to bf16, dense rows of `dim`, and out = RMS normalisation of the rounded sum times w, in one pass;
// copy_bytes bytes (a multiple of 16) moved from copy_src to copy_dst by the same launch.  sum may be a or b.
struct ResidualJob {
    int64_t rows;
    int dim;
    const void *a, *b;
    void* sum;
    const float* w;
    void* out;
    float eps;
    const void* copy_src;
    void* copy_dst;
    size_t copy_bytes;
};
bool residual_norm_supported(const ResidualJob& j);
hipError_t launch_residual_norm(const ResidualJob& j, hipStream_t st);
// ssd_gated_norm_bwd without a gate, with dy = (its dy) + res, rounded once; all rows dense, dy may be res.
bool norm_bwd_residual_supported(const ssd_norm_shape_t* sh, const void* y, const void* dout, const void* res, const void* dy);
int norm_bwd_residual(const ssd_norm_shape_t* sh, const void* y, const float* w, const void* dout, const void* res, void* dy, float* dw,
                      void* workspace, size_t workspace_bytes, uint32_t flags, hipStream_t st);

// True when everything is to stay on the caller's stream (SSD_MAGC_SERIAL=1 in the environment, or ssd_prof_serialize).
bool serial_mode();

// The library's side stream of the current device (default priority, created on first use) with a pair of
// events for the caller to fork it from and join it into its own stream; NULL in serial mode or on failure.
struct SideStream {
    hipStream_t st;
    hipEvent_t fork, join;
};
SideStream* side_stream();

// Generation (few_rows.hip): products and the block's middle steps for at most FEW_ROWS tokens, bf16 storage.
constexpr int FEW_ROWS = 16;
// Up to this many rows the product runs on the vector ALUs, above on the matrix cores.
constexpr int FEW_ROWS_VALU = 2;
// out[r, n] = sum_k f(x)[r, k] w[n, k] (+ res[r, n]); w [N, K] dense.  mode 0: f = identity; 1: RMS normalisation
// over all of K times in_w.  Row strides in elements.
struct FewRowsJob {
    int rows, K, N, mode;
    const void* x;
    int64_t ldx;
    const void* w;
    void* out;
    int64_t ldo;
    const float* in_w;
    float eps;
    const void* res;
    int64_t ldres;
    // optional: copy_chunks (0 = 1) pieces of copy_bytes bytes (a multiple of 16; at most 16 N vectors in all), the
    // pieces copy_src_stride / copy_dst_stride bytes apart, moved from copy_src to copy_dst by the same launch
    const void* copy_src;
    void* copy_dst;
    size_t copy_bytes;
    int copy_chunks;
    size_t copy_src_stride, copy_dst_stride;
    // matrix-core kernel only (rows > FEW_ROWS_VALU).  mode 2: x is the packed operand the kernel before left, already
    // times the norm's weight, `ssq` its partial sums of squares (null: no normalisation), nparts for each of `groups`
    // equal pieces of K (multiples of 256).  pack_out: leave the rounded output times pack_w (null: as it is) packed for the
    // next such product, with one part of sums of squares per 16 columns in pack_ssq.
    const float* ssq;
    int nparts, groups;
    void* pack_out;
    const float* pack_w;
    float* pack_ssq;
    // one token for each of `rows` sequences: columns [off_xbc, off_dt) through the convolution step + SiLU on the states cs
    // ([3, off_dt - off_xbc] each, cs_bs elements apart, replaced in place), columns from off_dt on through
    // softplus(. + dt_bias).  cs null: the product alone.
    void* cs;
    int64_t cs_bs;
    const float *conv_w, *conv_b, *dt_bias;
    int off_xbc, off_dt;
    bool stream;  // w by streaming loads: it will not be in a cache when it is read again
};
bool few_rows_supported(const FewRowsJob& j);  // sizes, strides and 16-byte alignment the kernel relies on
hipError_t launch_linear_few_rows(const FewRowsJob& j, hipStream_t st);
// zx [T, ld] = (z | xBC | dt_raw) of T tokens -> y [T, H P]; state [H, P, N] in place; cs_in / cs_out [3, H P + 2 G N]
// (either may be null; never the same buffer).  nb > 1: that many independent sequences of T tokens each (nb T <=
// FEW_ROWS), sequence b in rows b T .. of zx and y, its states state_bs / cs_in_bs / cs_out_bs elements further on.
struct DecodeMidJob {
    int nb;
    int64_t state_bs, cs_in_bs, cs_out_bs;
    int T, H, P, G, N;
    const void* zx;
    int64_t ld;
    const float *conv_w, *conv_b, *dt_bias, *A, *D;
    const void* cs_in;
    void* cs_out;
    float* state;
    void* y;
    int gate;  // y silu(z) instead of y
    // one token per sequence whose product took the convolution step and softplus along (FewRowsJob.cs): the recurrence
    // only; cs_in, cs_out are not touched.  Where step_supported(j).
    int stepped;
    // stepped with gate: y silu(z) pack_w as the packed operand of a mode-2 product instead, step_parts(j) parts of sums of
    // squares (heads in order) in pack_ssq
    void* pack;
    const float* pack_w;
    float* pack_ssq;
    bool stream;  // stepped: the states by streaming accesses
};
bool step_supported(const DecodeMidJob& j);
int step_parts(const DecodeMidJob& j);
hipError_t launch_decode_mid(const DecodeMidJob& j, hipStream_t st);

}  // namespace ssdk
