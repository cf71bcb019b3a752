// Matrix-core (MFMA, bf16 in / fp32 accumulate) kernels of the chunked selective scan for gfx950.
// Shape: P = 64 channels per head, N = 128 states, chunk Q in {64, 128, 256}; wave64; every contraction
// runs on v_mfma_f32_32x32x16_bf16.
//
// Numerical scheme for the decay mask exp(cum_i - cum_j) of the dual form (Sec. 3.1, Eq. 1 unrolled
// over a chunk).  The chunk is cut into blocks of 64 tokens.  With
//     ein_i  = exp(cum_i - cum[start of i's block - 1])      (<= 1)
//     eout_j = exp(cum[end of j's block] - cum_j)            (<= 1)
//     s_K    = exp(cum[end of block K] - cum[start of K - 1]) (<= 1, the block's total decay)
// one has, for i in block I and j in block J < I,
//     exp(cum_i - cum_j) = ein_i * (prod_{J<K<I} s_K) * eout_j,
// so the off-diagonal blocks are pure MFMA work on the raw scores G = C B^T and on operands that were
// scaled once per token while being staged into LDS; the product over K is applied Horner-style by
// scaling the accumulator with the scalar s_K between blocks (this is the state recurrence at
// 64-token granularity), and ein / eout is applied once per output row.  Only the four diagonal
// 64 x 64 blocks evaluate exp() per element.  Every exponent is <= 0: nothing can overflow, and an
// underflow only happens where the exact value underflows too.
//
// Operands whose contraction index is the token index live token-major in memory; they are staged
// in LDS as [token][channel] and read with the LDS transpose load (ds_read_b64_tr_b16), which hands
// each lane four consecutive tokens of one channel -- the layout an MFMA operand needs.
#include "mfma_common.h"

namespace ssdk {
namespace {

using namespace mf;

// ---------------------------------------------------------------------------------------------
// Decay preparation of one chunk and head by one wave, lane l the tokens E l .. E l + E - 1: cum (chunk-local inclusive cumsum of
// dt*A), dt in fp32, ein, eout.  Nothing waits for other waves (over LDS the prefix sums took sixteen barriers), and the waves
// of a workgroup take neighbouring heads, i.e. read the same cache lines of dt.  In two halves, so that the loads can be under
// way while something else is worked on.
template <int Q>
struct Prep {
    static constexpr int E = Q / 64;
    typedef float vec __attribute__((ext_vector_type(E)));
    bf16_t dt[E];
    float A, bias;  // of the head: by scalar memory, asked for with the rest

    __device__ __forceinline__ void load(const SegParams& sp, int b, int c, int h, int lane, int rows) {
        const bool raw = sp.raw.dt;
        const int64_t rs = raw ? sp.raw.rs : sp.H;
        const bf16_t* src = (raw ? (const bf16_t*)sp.raw.dt : (const bf16_t*)sp.dt + (int64_t)b * sp.dts_b) + (int64_t)c * Q * rs + h;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = E * lane + e, il = i < rows ? i : rows - 1;
            dt[e] = src[il * rs];
        }
        typedef const __attribute__((address_space(4))) float* scalars;
        A = ((scalars)sp.A)[h];
        bias = ((scalars)(raw ? sp.raw.bias : sp.A))[h];
    }
    // vc: cum, vd: dt; returns cum at the end of the chunk
    __device__ __forceinline__ float form(const SegParams& sp, int b, int c, int h, int lane, int rows, vec& vc, vec& vd) const {
        float d[E], a[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            d[e] = bf16_to_float(dt[e]);
            a[e] = 0.f;
        }
        if (sp.raw.dt) {  // uniform
#pragma unroll
            for (int e = 0; e < E; ++e) d[e] = bf16_to_float(float_to_bf16(softplus(d[e] + bias)));
        }
        if (sp.reset) {  // uniform
            const uint8_t* reset = sp.reset + (int64_t)b * sp.reset_bs + (int64_t)c * Q;
#pragma unroll
            for (int e = 0; e < E; ++e) a[e] = reset[E * lane + e < rows ? E * lane + e : rows - 1] ? RESET_LOG_DECAY : 0.f;
        }
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (E * lane + e >= rows) d[e] = a[e] = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) a[e] += d[e] * A;
        // prefix sums by doubling: token i adds token i - off, off = 1, 2, 4, ...
#pragma unroll
        for (int off = 1; off < Q; off <<= 1) {
            float v[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int src = off < E ? e - off : e;  // element, and how many lanes to the left of this one it lies
                const int left = off < E ? (src < 0 ? 1 : 0) : off / E;
                v[e] = left ? __shfl_up(a[(src + E) % E], left, 64) : a[(src + E) % E];
                if (lane < left) v[e] = 0.f;
            }
#pragma unroll
            for (int e = 0; e < E; ++e) a[e] += v[e];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            vc[e] = a[e];
            vd[e] = d[e];
        }
        return __shfl(a[E - 1], 63, 64);
    }
    __device__ __forceinline__ void store(const SegParams& sp, int b, int c, int h, int lane, const vec& vc, const vec& vd) const {
        // cum at the end of the lane's 64-token block and of the one in front of it
        constexpr int LPB = 64 / E;  // lanes of a block
        const float end = __shfl(vc[E - 1], lane | (LPB - 1), 64), prev = __shfl(vc[E - 1], (lane | (LPB - 1)) - LPB, 64);
        const float start = lane >= LPB ? prev : 0.f;
        vec vi, vo;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            vi[e] = __expf(vc[e] - start);
            vo[e] = __expf(end - vc[e]);
        }
        const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q + E * lane;
        *(vec*)(sp.cum + o) = vc;
        *(vec*)(sp.dtf + o) = vd;
        *(vec*)(sp.ein + o) = vi;
        *(vec*)(sp.eout + o) = vo;
    }
};

// ---------------------------------------------------------------------------------------------
// Scores of one chunk and group: G[i][j] = C_i . B_j and its transpose, bf16, for the 64 x 64 blocks
// on and below the diagonal.  Layout in the scratch area: G [Q][Q] then GT [Q][Q].
template <int Q>
__device__ __forceinline__ void cb_body(const SegParams& sp, int z, int pair, int w, int lane) {  // four waves
    constexpr int NB = Q / BLK;
    const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc);
    int I = 0, rem = pair;  // pair enumerates the block pairs (I, J <= I)
    while (rem > I) {
        rem -= I + 1;
        ++I;
    }
    const int J = rem;
    if (I >= NB) return;
    const int i0 = I * BLK + (w >> 1) * 32, j0 = J * BLK + (w & 1) * 32;
    const int64_t ts = (int64_t)sp.G * N_;
    const bf16_t* Cm = (const bf16_t*)sp.Cm + (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N_;
    const bf16_t* Bm = (const bf16_t*)sp.Bm + (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N_;
    const int nv = chunk_rows(sp, c, Q);
    const uint32_t rowbytes = (uint32_t)ts * 2;
    const rsrc_t cr = make_rows(Cm, nv, rowbytes), br = make_rows(Bm, nv, rowbytes);
    f32x16 a1 = zero16(), a2 = zero16();
#pragma unroll
    for (int ks = 0; ks < N_ / 16; ++ks) {
        const bf16x8 fc = frag_tokens(cr, rowbytes, i0, 16 * ks, lane);
        const bf16x8 fb = frag_tokens(br, rowbytes, j0, 16 * ks, lane);
        a1 = mfma(fc, fb, a1);  // a1[r] = G[i0 + acc_row(r)][j0 + lane%32]
        a2 = mfma(fb, fc, a2);  // a2[r] = G[i0 + lane%32][j0 + acc_row(r)]
    }
    bf16_t* Gd = (bf16_t*)sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * (2 * Q * Q);
    bf16_t* GTd = Gd + Q * Q;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        bf16x4 v1, v2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v1[e] = (__bf16)a1[4 * q + e];
            v2[e] = (__bf16)a2[4 * q + e];
        }
        const int rr = 8 * q + 4 * (lane >> 5);
        *(bf16x4*)(GTd + (int64_t)(j0 + (lane & 31)) * Q + i0 + rr) = v1;
        *(bf16x4*)(Gd + (int64_t)(i0 + (lane & 31)) * Q + j0 + rr) = v2;
    }
}

// ---------------------------------------------------------------------------------------------
// role 0: states_bf[b,c,h]  = sum_j exp(T - cum_j) dt_j x_j (x) B_j      (chunk state, bf16 [P][N])
// role 1: dstates_bf[b,c,h] = sum_i exp(cum_i) dY_i (x) C_i              (local state adjoint)
// (fp32 accumulation, one rounding to bf16: the consumers take these as bf16 MFMA operands anyway,
// and the scans carry the running state in fp32 registers.)
// One workgroup per (batch, chunk, group, role, head slice); eight waves, wave w owning the 32 x 32
// output tile (p half w / 4, state columns 32 (w % 4)).  The B (or C) rows of the chunk do not depend on
// the head: they go through LDS once and each wave keeps its Q/16 operand fragments in registers
// for every head of the slice.  Per head the token-major tile (x or dY, weighted per token) is
// prefetched in registers during the previous head, staged in LDS and read with transpose loads.
// The weights come from the decay preparation, which needs nothing but the inputs either: a wave does a head of the slice,
// eight heads ahead of their use (role 0 stores it for the kernels that follow), and the scores of the chunks are further workgroups
// of this launch.  As a launch in front of this one, which read the weights from memory, against now (us, two launches -> one):
// 10007 tokens of 80 heads 11.9 + 35.2 -> 37.8; 8192 of 24 8.8 + 13.1 -> 16.3, both roles 8.8 + 19.7 -> 23.2; 65536 tokens of
// 80 heads forward + backward, four segments in flight, 3110 -> 3048.
constexpr int OUTER_THR = 512, PREP_HEADS = OUTER_THR / 64, OUT_PITCH = 64 + 16;

template <int Q>
struct OuterLds {
    union {
        char bc[Q * BPITCH];  // B or C rows of the chunk (prologue only: each wave takes its fragments, then the space is free)
        struct {
            char xt[Q * XPITCH];                          // weight * x or weight * dY
            char out[OUTER_THR / 64][32 * OUT_PITCH];     // a wave's 32 x 32 tile on its way to whole rows (bf16)
        };
    };
    float wt[PREP_HEADS][Q];  // weights of eight heads
};

template <int Q>
struct OuterPre {
    static constexpr int NV = Q * 8 / OUTER_THR > 0 ? Q * 8 / OUTER_THR : 1;
    bf16x8 t[NV];
};

// Loads only: nothing waits for them before the next head's staging.
template <int Q>
__device__ __forceinline__ void outer_load(OuterPre<Q>& pr, const SegParams& sp, int role, int b, int c, int h, int tid) {
    const int64_t xt = (int64_t)sp.H * P_;
    const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P_;
    const bf16_t* src = role == 0 ? (const bf16_t*)sp.x + (int64_t)b * sp.xs_b + xrow
                                  : (const bf16_t*)sp.dy + (int64_t)b * sp.dys_b + xrow;
    // addresses = a wave-uniform base (scalar registers) + one 32-bit byte offset per lane
    const int t8 = tid % (Q * 8);  // Q = 64: one vector per thread
    const uint32_t rowbytes = (uint32_t)xt * 2, off = (uint32_t)(t8 >> 3) * rowbytes + (uint32_t)(t8 & 7) * 16;
    const rsrc_t rows = make_rows(src, chunk_rows(sp, c, Q), rowbytes);
#pragma unroll
    for (int k = 0; k < OuterPre<Q>::NV; ++k) {
        // one reader per launch: streaming load (keeps the L2 for the kernels of other segments that do share tiles)
        pr.t[k] = rows_load<AUX_NT>(rows, off + k * (OUTER_THR / 8) * rowbytes);
    }
}

// Two workgroups per compute unit (78 KB of LDS, at most 128 registers): one stages its next head while the
// other contracts.
template <int Q, bool F32OUT>
__global__ __launch_bounds__(OUTER_THR, 4) void mk_chunk_outer(SegParams sp, int nroles, int n_outer) {
    constexpr int KS = Q / 16;
    __shared__ __attribute__((aligned(16))) OuterLds<Q> L;
    int z = blockIdx.x;
    [[maybe_unused]] const int zlog = z;
    if (z >= n_outer) {  // scores: two block pairs a workgroup
        constexpr int NPAIR = (Q / BLK) * (Q / BLK + 1) / 2;
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = 2 * (z - n_outer) + (w >> 2);
        if (i < sp.Bt * sp.nc * sp.G * NPAIR) cb_body<Q>(sp, i / NPAIR, i % NPAIR, w & 3, threadIdx.x & 63);
        return;
    }
    if ((n_outer & 7) == 0) z = (z & 7) * (n_outer >> 3) + (z >> 3);
    const int ns = sp.outer_split, slice = z % ns;
    z /= ns;
    const int role = z % nroles;
    z /= nroles;
    const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc);
    const Slice sl = slice_of(sp.hpg, ns, slice);
    const int hps = sl.n, h0 = g * sp.hpg + sl.first;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), ph = w >> 2, nt = w & 3;
    const int64_t bt = (int64_t)sp.G * N_;
    const int nrows = chunk_rows(sp, c, Q);
    Prep<Q> pp;
    if (w < hps) pp.load(sp, b, c, h0 + w, lane, nrows);
    // B (role 0) or C (role 1) rows, then the first head: all under way before the first of them is waited for, and one trip to memory
    // (with the rows in a loop and A and the bias fetched where they are used three: 8192 tokens of 24 heads, forward and backward,
    // 164.4 -> 162.5 us)
    const bf16_t* rhs = (role == 0 ? (const bf16_t*)sp.Bm : (const bf16_t*)sp.Cm) + (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N_;
    const rsrc_t rows = make_rows(rhs, nrows, (uint32_t)bt * 2);
    constexpr int NB = Q * 16 / OUTER_THR;
    bf16x8 rv[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) rv[k] = rows_load(rows, (uint32_t)((tid >> 4) + k * (OUTER_THR / 16)) * (uint32_t)bt * 2 + (tid & 15) * 16);
    OuterPre<Q> pr;
    outer_load<Q>(pr, sp, role, b, c, h0, tid);
    // what is derived from such a value is formed where it is used and not kept in registers over the loop
    auto opaque = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    // the weights of this wave's head of the eight from hh on
    auto weights = [&](int hh) {
        if (hh + w >= hps) return;
        const int ln = opaque(lane);
        typename Prep<Q>::vec vc, vd, vw;
        const float T = pp.form(sp, b, c, h0 + hh + w, ln, nrows, vc, vd);
#pragma unroll
        for (int e = 0; e < Q / 64; ++e) vw[e] = role == 0 ? __expf(T - vc[e]) * vd[e] : __expf(vc[e]);
        *(typename Prep<Q>::vec*)(&L.wt[w][Q / 64 * ln]) = vw;
        if (role == 0) pp.store(sp, b, c, h0 + hh + w, ln, vc, vd);
    };
    // prologue: the rows -> LDS -> this wave's fragments
#pragma unroll
    for (int k = 0; k < NB; ++k) *(bf16x8*)(L.bc + ((tid >> 4) + k * (OUTER_THR / 16)) * BPITCH + (tid & 15) * 16) = rv[k];
    weights(0);
    __syncthreads();
    bf16x8 fb[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fb[ks] = frag_tr(L.bc, BPITCH, 16 * ks, 32 * nt, lane);
    wait_loads();
    for (int hh = 0; hh < hps; ++hh) {
        const int h = h0 + hh;
        SSDK_STAMP(4, 0);
        __syncthreads();
        SSDK_STAMP(4, 1);
#pragma unroll
        for (int k = 0; k < OuterPre<Q>::NV; ++k) {
            const int v = tid + OUTER_THR * k, row = v >> 3, seg = v & 7;
            if (v < Q * 8) *(bf16x8*)(L.xt + row * XPITCH + seg * 16) = scale8(pr.t[k], L.wt[hh % PREP_HEADS][row]);
        }
        SSDK_STAMP(4, 2);
        __syncthreads();
        SSDK_STAMP(4, 3);
        if (hh % PREP_HEADS == PREP_HEADS - 1 && hh + 1 + w < hps) pp.load(sp, b, c, h + 1 + w, lane, nrows);
        if (hh + 1 < hps) outer_load<Q>(pr, sp, role, b, c, h + 1, opaque(tid));
        SSDK_STAMP(4, 4);
        f32x16 acc = zero16();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = mfma(fb[ks], frag_tr(L.xt, XPITCH, 16 * ks, 32 * ph, lane), acc);
        // a lane holds four times four neighbours of a row
        const int64_t so = (((int64_t)b * sp.nc + c) * sp.H + h) * (P_ * N_) + 32 * ph * N_ + 32 * nt;
        const int ls = opaque(lane);
        if (F32OUT) {  // fp32 scan input, in an array of its own
            float* out = (role == 0 ? sp.states : sp.dstates) + so;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4*)(out + (ls & 31) * N_ + 8 * q + 4 * (ls >> 5)) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        } else {
            // bf16, into the slot where the scan will put the state entering the chunk (total adjoint leaving it); through
            // LDS, two stores of 16 bytes a lane instead of sixteen of two bytes
            __bf16* out = (__bf16*)(role == 0 ? sp.states_bf : sp.dstates_bf) + so;
            char* patch = L.out[w];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)acc[4 * q + e];
                *(bf16x4*)(patch + (ls & 31) * OUT_PITCH + (8 * q + 4 * (ls >> 5)) * 2) = v;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int row = 16 * it + (ls >> 2), seg = ls & 3;
                *(bf16x8*)(out + row * N_ + 8 * seg) = *(const bf16x8*)(patch + row * OUT_PITCH + 16 * seg);
            }
        }
        if (hh % PREP_HEADS == PREP_HEADS - 1) weights(hh + 1);  // of the next eight heads: the last of these is staged
        SSDK_STAMP(4, 5);
    }
}

// ---------------------------------------------------------------------------------------------
// Inter-chunk state passing over a span, four state elements per thread.  The running state is carried in fp32 registers
// (checkpoints and the final state are stored from them); the state entering each chunk is emitted as the bf16 copy the
// contraction kernels read, nothing else.  Bound by the trips of the chunk states through memory: the recurrence is serial,
// so the loads of a block of chunks are under way while the block before it is worked on.  (Two elements per thread, twice
// the waves: no faster at 24 heads, 10 % slower at 64.)
__device__ __forceinline__ f32x4 ld_state(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 ld_state(const bf16_t* p) { return __builtin_convertvector(*(const bf16x4*)p, f32x4); }
__device__ __forceinline__ void st_state(float* p, f32x4 v) { *(f32x4*)p = v; }
__device__ __forceinline__ void st_state(bf16_t* p, f32x4 v) { *(bf16x4*)p = __builtin_convertvector(v, bf16x4); }

// F32IN: the chunk states arrive in fp32 (SSD_FLAG_FP32_CHUNK_STATES, an array of their own), else as bf16 in place.
// BWD = false: one walk over all chunks of the span, putting the checkpoints of its segments down on the way.
// BWD = true: the walk to the right again, every segment restarted from its checkpoint, then the walk back over the
// chunk-state adjoints, which emits the bf16 adjoint leaving each chunk and the per-wave partial sums of
// exp(T_c) <dHnext_c, Hprev_c>, the gradient of the chunk's total decay through the carried state (fixed summation order).
// The way back finds the entering states that the same thread has just written in the L2 of its XCD.  As two launches the
// same work read them from memory and paid a second ramp: 32 chunks of 24 heads 21.5 -> 17.8 us, 24 chunks of 2 x 32 heads
// 25.6 -> 21.4.  Restarting every segment side by side, which two launches could, pays for one or two heads only: 153600 tokens
// of one head in eight segments 558 us backward, 575 so (with the forward pass 769, 766).
template <bool BWD, bool F32IN>
__global__ __launch_bounds__(NTH) void mk_scan(SegParams sp) {
    constexpr int PN = P_ * N_;
    constexpr int U = 8;  // chunks of a block: their loads are in flight together
    const int e = (blockIdx.x * NTH + threadIdx.x) * 4, h = blockIdx.y, b = blockIdx.z, nc = sp.nc;
    const int64_t bh = (int64_t)h * PN + e, HPN = (int64_t)sp.H * PN;
    const float* cum = sp.cum + ((int64_t)b * sp.H + h) * nc * sp.Q + sp.Q - 1;
    const int64_t base = (int64_t)b * nc * HPN + bh;
    f32x4 hc = (f32x4)(0.f), nxt = (f32x4)(0.f);
    struct Block {
        f32x4 s[U];
        float a[U];
    } A, B;
    auto load = [&](Block& R, int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u < nc ? c0 + u : nc - 1;
            R.s[u] = F32IN ? ld_state(sp.states + base + c * HPN) : ld_state(sp.states_bf + base + c * HPN);
            R.a[u] = cum[(int64_t)c * sp.Q];
        }
    };
    int64_t slot = (int64_t)b * sp.ckpt_bs + bh;
    // chunk at which the next segment of the span starts; its checkpoint is asked for a segment ahead
    int next = sp.ckpt || sp.ckpt16 ? sp.seg_chunks : nc;
    auto ask = [&] {
        if (BWD && next < nc) nxt = sp.ckpt16 ? ld_state(sp.ckpt16 + slot + HPN) : ld_state(sp.ckpt + slot + HPN);
    };
    if (sp.state_in) hc = ld_state(sp.state_in + (int64_t)b * sp.state_in_bs + bh);
    else if (sp.state_in16) hc = ld_state(sp.state_in16 + (int64_t)b * sp.state_in_bs + bh);  // bf16 checkpoint
    load(A, 0);
    ask();
    if (!BWD) {
        if (sp.bnd_write) st_state(sp.bnd_write + (int64_t)b * sp.bnd_write_bs + bh, hc);
        if (sp.bnd_write16) st_state(sp.bnd_write16 + (int64_t)b * sp.bnd_write_bs + bh, hc);
    }
    auto walk = [&](const Block& R, int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u;
            if (c >= nc) break;  // uniform
            if (c == next) {     // uniform
                next += sp.seg_chunks;
                slot += HPN;
                if (BWD) {
                    hc = nxt;
                    ask();
                } else {
                    if (sp.ckpt) st_state(sp.ckpt + slot, hc);
                    if (sp.ckpt16) st_state(sp.ckpt16 + slot, hc);
                }
            }
            st_state(sp.states_bf + base + c * HPN, hc);
            hc = __expf(R.a[u]) * hc + R.s[u];
        }
    };
    for (int c0 = 0; c0 < nc; c0 += 2 * U) {
        if (c0 + U < nc) load(B, c0 + U);
        walk(A, c0);
        if (c0 + 2 * U < nc) load(A, c0 + 2 * U);
        if (c0 + U < nc) walk(B, c0 + U);
    }
    if (!BWD) {
        if (sp.state_out) st_state(sp.state_out + (int64_t)b * sp.state_out_bs + bh, hc);
        if (sp.state_out2) st_state(sp.state_out2 + (int64_t)b * sp.state_out2_bs + bh, hc);
        if (sp.state_out16) st_state(sp.state_out16 + (int64_t)b * sp.state_out16_bs + bh, hc);
        return;
    }
    if (sp.first_span && blockIdx.x == 0 && b == 0 && threadIdx.x == 0) sp.param_count[(int64_t)h * sp.param_stride] = 0;
    const int64_t ce = (int64_t)b * HPN + bh;
    f32x4 g = sp.dcarry_in ? ld_state(sp.dcarry_in + ce) : (f32x4)(0.f);
    constexpr int UB = 4;  // two arrays a chunk on the way back
    struct Back {
        f32x4 l[UB], h[UB];
        float a[UB];
    } RA, RB;
    auto loadb = [&](Back& R, int c0) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int c = c0 - u >= 0 ? c0 - u : 0;
            R.l[u] = F32IN ? ld_state(sp.dstates + base + c * HPN) : ld_state(sp.dstates_bf + base + c * HPN);
            R.h[u] = ld_state(sp.states_bf + base + c * HPN);
            R.a[u] = cum[(int64_t)c * sp.Q];
        }
    };
    float* tail = sp.tail_part + ((int64_t)b * sp.H + h) * nc * sp.nslice + blockIdx.x * (NTH / 64) + (threadIdx.x >> 6);
    auto walkb = [&](const Back& R, int c0) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int c = c0 - u;
            if (c < 0) break;  // uniform
            st_state(sp.dstates_bf + base + c * HPN, g);  // the total adjoint is kept in bf16 only
            const float a = __expf(R.a[u]);
            float part = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) part += g[i] * R.h[u][i];
            part = wave_prefix(a * part);
            if ((threadIdx.x & 63) == 63) tail[(int64_t)c * sp.nslice] = part;  // one per wave; summed later in a fixed order
            g = a * g + R.l[u];
        }
    };
    loadb(RA, nc - 1);
    for (int c0 = nc - 1; c0 >= 0; c0 -= 2 * UB) {
        if (c0 >= UB) loadb(RB, c0 - UB);
        walkb(RA, c0);
        if (c0 >= 2 * UB) loadb(RA, c0 - 2 * UB);
        if (c0 >= UB) walkb(RB, c0 - UB);
    }
    st_state(sp.dcarry + ce, g);
    if (sp.dinit_out) st_state(sp.dinit_out + ce, g);
}

template <bool BWD>
hipError_t scan(const SegParams& sp, hipStream_t st) {
    const dim3 grid(P_ * N_ / 4 / NTH, sp.H, sp.Bt);
    if (sp.flags & SSD_FLAG_FP32_CHUNK_STATES)
        SSDK_LAUNCH(BWD ? K_SCAN_BWD : K_SCAN_FWD, st, (mk_scan<BWD, true>), grid, dim3(NTH), sp);
    else
        SSDK_LAUNCH(BWD ? K_SCAN_BWD : K_SCAN_FWD, st, (mk_scan<BWD, false>), grid, dim3(NTH), sp);
    return hipSuccess;
}

template <int Q>
hipError_t fwd_q(const SegParams& sp, bool need_y, hipStream_t st) {
    constexpr int NB = Q / BLK;
    const int n_cb = sp.Bt * sp.nc * sp.G * (NB * (NB + 1) / 2);
    {   // decay preparation, scores, chunk states; on the backward path (need_y false) the local state adjoints ride in the same launch
        SegParams so = sp;
        const int nroles = need_y ? 1 : 2;
        // alone on the machine (10007 tokens of 80 heads, eight slices -> ten: 40.2 -> 35.9 us); with others in flight as mk_dual
        const int64_t base = (int64_t)sp.Bt * sp.nc * sp.G * nroles;
        so.outer_split = sp.wg_target < 256 ? pick_split(sp.hpg, base, sp.wg_target) : pick_rounds(sp.hpg, base, 2, 140);
        const int n_outer = sp.Bt * sp.nc * sp.G * nroles * so.outer_split;
        const dim3 grid(n_outer + (n_cb + 1) / 2);
        if (sp.flags & SSD_FLAG_FP32_CHUNK_STATES)
            SSDK_LAUNCH(need_y ? K_MFMA_CHUNK_STATE : K_MFMA_DSTATE, st, (mk_chunk_outer<Q, true>), grid, dim3(OUTER_THR), so, nroles, n_outer);
        else
            SSDK_LAUNCH(need_y ? K_MFMA_CHUNK_STATE : K_MFMA_DSTATE, st, (mk_chunk_outer<Q, false>), grid, dim3(OUTER_THR), so, nroles, n_outer);
    }
    if (!need_y) return hipSuccess;  // the backward pass restores the entering states in the launch of its own scan
    // the scan is the only step that needs the previous segment (its leaving state)
    if (sp.ev_wait && hipStreamWaitEvent(st, sp.ev_wait, 0) != hipSuccess) return hipErrorUnknown;
    const hipError_t e = scan<false>(sp, st);
    if (e != hipSuccess) return e;
    if (sp.ev_record && hipEventRecord(sp.ev_record, st) != hipSuccess) return hipErrorUnknown;
    return mfma_launch_dual(sp, 0, st);
}

template <int Q>
hipError_t bwd_q(const SegParams& sp0, hipStream_t st) {
    SegParams sp = sp0;
    sp.nslice = P_ * N_ / 4 / 64;  // partial sums of the reverse scan: one per wave
    // the scan is the only step that needs the segment to the right (its entering-state adjoint)
    if (sp.ev_wait && hipStreamWaitEvent(st, sp.ev_wait, 0) != hipSuccess) return hipErrorUnknown;
    hipError_t e = scan<true>(sp, st);
    if (e != hipSuccess) return e;
    if (sp.ev_record && hipEventRecord(sp.ev_record, st) != hipSuccess) return hipErrorUnknown;
    // dx, dG and the dB / dC head sums (which also write the chunk-local part of the gradient of cum
    // and the state dot products): one launch when the three share a workgroup size
    const bool trio = Q >= 128;
    if (!trio) e = mfma_launch_dual(sp, 2, st);
    if (e != hipSuccess) return e;
    return mfma_launch_grad_bc(sp, st);  // ddt, dA and dD ride in its last launch
}

}  // namespace

bool mfma_path_supported(const ssd_shape_t& s) {
    return s.dtype == SSD_BF16 && s.headdim == P_ && s.dstate == N_ && (s.chunk == 64 || s.chunk == 128 || s.chunk == 256);
}

hipError_t mfma_forward_segment(const SegParams& sp, bool need_y, hipStream_t st) {
    switch (sp.Q) {
        case 64: return fwd_q<64>(sp, need_y, st);
        case 128: return fwd_q<128>(sp, need_y, st);
        case 256: return fwd_q<256>(sp, need_y, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t mfma_backward_segment(const SegParams& sp, hipStream_t st) {
    switch (sp.Q) {
        case 64: return bwd_q<64>(sp, st);
        case 128: return bwd_q<128>(sp, st);
        case 256: return bwd_q<256>(sp, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ssdk
