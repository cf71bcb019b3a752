// Causal depthwise convolution (kernel 4) + bias + SiLU of the Mamba-2 block, forward and backward,
// with the three-token convolution state that MA-GC keeps next to the SSM state in every sequence
// checkpoint (App. C, Tab. 7: the per-checkpoint constant counts the SSM state plus three tokens of the
// convolution's channels).  A segment is processed from its stored state exactly as the SSD segment is:
//     pre[t,c] = bias[c] + sum_{k=0..3} w[c,k] u[t-3+k, c]      (u[-3..-1] = state_in, zeros if absent)
//     out[t,c] = pre / (1 + exp(-pre))
// HBM-bound: every thread owns V consecutive channels (8 bytes: with 16 the backward kernel's state does not fit the registers) and walks `tt` consecutive tokens with
// the window in registers, so every input row is read once (plus a three-row halo per run).  The rows come in
// packed, four at a time and the four behind them under way, by loads without a branch around them (a row index
// beyond the run is clamped to its last): a load under a condition ends in a wait for all of them.
#include <string.h>

#include "column_sums.h"

namespace ssdk {
namespace {

constexpr int CONV_K = 4;
constexpr int MAX_TT = 64, MIN_TT = 8;  // tokens per thread; shorter runs re-read too much of the three-token halo
constexpr int U = 4;                    // rows requested together
constexpr int BWD_WAVES = 4;            // runs of a backward workgroup, whose sums of dw / dbias go out as one

struct ConvParams {
    const void* u;
    const void* dout;
    const void* state_in;   // [Bt][3][C] storage dtype or null
    const float* dstate_out;  // [Bt][3][C] fp32 or null: gradient reaching the last three rows of u from the right
    void* out;
    void* du;
    void* state_out;    // [Bt][3][C] storage dtype or null
    float* dstate_in;   // [Bt][3][C] fp32 or null
    const float* w;     // [C][4]
    const float* bias;  // [C] or null
    float* part;        // [nwg][5][C] partial sums of dw (k = 0..3) and dbias
    int64_t L, u_bs, o_bs;  // tokens; batch stride of u / du and of out / dout in elements
    int64_t u_rs;           // elements between consecutive tokens of u / du (out / dout: C)
    int C;
    uint32_t batch, nruns, nwg;  // backward: sequences, runs of one, workgroups side by side that share them out
    int tt;             // tokens per thread of this launch
    // out / dout as three dense tensors side by side instead of one: channels [cb[k], cb[k+1]) live in
    // part[k] with rows cb[k+1] - cb[k] apart (the block's x | B | C, each the shape the scan wants)
    int split;
    int cb[4];
    void* out3[3];
    const void* dout3[3];
};

// Where this thread's channels c0.. of out / dout live: base pointer, batch and row stride, first column.
struct OutSlot {
    void* out;
    const void* dout;
    int64_t bs, rs;
    int c;
};
__device__ __forceinline__ OutSlot out_slot(const ConvParams& cp, int c0) {
    OutSlot o;
    if (!cp.split) {
        o.out = cp.out;
        o.dout = cp.dout;
        o.bs = cp.o_bs;
        o.rs = cp.C;
        o.c = c0;
    } else {
        const int k = c0 >= cp.cb[2] ? 2 : c0 >= cp.cb[1] ? 1 : 0;
        o.out = cp.out3[k];
        o.dout = cp.dout3[k];
        o.rs = cp.cb[k + 1] - cp.cb[k];
        o.bs = cp.L * o.rs;
        o.c = c0 - cp.cb[k];
    }
    return o;
}

typedef uint32_t words2 __attribute__((ext_vector_type(2)));

template <typename T, int V>
struct Vec;
template <>
struct Vec<float, 1> {
    static __device__ __forceinline__ void ld(const void* p, int64_t i, float (&v)[1]) { v[0] = ((const float*)p)[i]; }
    static __device__ __forceinline__ void st(void* p, int64_t i, const float (&v)[1]) { ((float*)p)[i] = v[0]; }
    typedef float Raw;
    static __device__ __forceinline__ void open(Raw r, float (&v)[1]) { v[0] = r; }
    static __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, int at, const float (&v)[1]) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[0]), r, at, 0, 0); }
};
template <>
struct Vec<float, 2> {
    typedef float2 Raw;
    static __device__ __forceinline__ void open(Raw r, float (&v)[2]) { v[0] = r.x; v[1] = r.y; }
    static __device__ __forceinline__ void ld(const void* p, int64_t i, float (&v)[2]) { open(*(const Raw*)((const float*)p + i), v); }
    static __device__ __forceinline__ void st(void* p, int64_t i, const float (&v)[2]) { *(float2*)((float*)p + i) = make_float2(v[0], v[1]); }
    static __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, int at, const float (&v)[2]) {
        __builtin_amdgcn_raw_buffer_store_b64(words2{__float_as_uint(v[0]), __float_as_uint(v[1])}, r, at, 0, 0);
    }
};
template <>
struct Vec<bf16_t, 1> {
    static __device__ __forceinline__ void ld(const void* p, int64_t i, float (&v)[1]) { v[0] = bf16_to_float(((const bf16_t*)p)[i]); }
    static __device__ __forceinline__ void st(void* p, int64_t i, const float (&v)[1]) { ((bf16_t*)p)[i] = float_to_bf16(v[0]); }
    typedef bf16_t Raw;
    static __device__ __forceinline__ void open(Raw r, float (&v)[1]) { v[0] = bf16_to_float(r); }
    static __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, int at, const float (&v)[1]) { __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, float_to_bf16(v[0])), r, at, 0, 0); }
};
template <>
struct Vec<bf16_t, 4> {
    typedef words2 Raw;  // words: bf16 elements would take a register each
    typedef __bf16 b4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ void open(Raw r, float (&v)[4]) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t word = r[e];
            v[2 * e] = __uint_as_float(word << 16);
            v[2 * e + 1] = __uint_as_float(word & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void ld(const void* p, int64_t i, float (&v)[4]) { open(*(const Raw*)((const bf16_t*)p + i), v); }
    static __device__ __forceinline__ void st(void* p, int64_t i, const float (&v)[4]) {
        b4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = (__bf16)v[e];
        *(b4*)((bf16_t*)p + i) = t;
    }
    static __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, int at, const float (&v)[4]) {
        b4 t;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = (__bf16)v[e];
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(words2, t), r, at, 0, 0);
    }
};

// sigmoid through the hardware reciprocal (1 ulp) instead of an IEEE division: the kernels here are close
// enough to the VALU limit for the ten extra instructions per element to show
__device__ __forceinline__ float sigmoid_fast(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigmoid_fast(z); }
// d silu / dz = s (1 + z (1 - s)), s = sigmoid(z)
__device__ __forceinline__ float dsilu(float z) {
    const float s = sigmoid_fast(z);
    return s * (1.f + z * (1.f - s));
}

// The three rows in front of row t0 of u for this thread's channels: of the tensor, the entering state, or zeros (then something that is
// there is loaded and not used: a load under a condition would be waited for at the condition's end).
template <typename T, int V>
__device__ __forceinline__ void load_before(const ConvParams& cp, int64_t b, int64_t t0, int c0, typename Vec<T, V>::Raw (&v)[3]) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int64_t t = t0 - 3 + j;
        const T* p = t >= 0 ? (const T*)cp.u + b * cp.u_bs + t * cp.u_rs : cp.state_in ? (const T*)cp.state_in + (b * 3 + (t + 3)) * cp.C : (const T*)cp.w;
        v[j] = *(const typename Vec<T, V>::Raw*)(p + c0);
    }
}
template <typename T, int V>
__device__ __forceinline__ void open_before(const ConvParams& cp, int64_t t0, const typename Vec<T, V>::Raw (&r)[3], float (&v)[3][V]) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        Vec<T, V>::open(r[j], v[j]);
#pragma unroll
        for (int e = 0; e < V; ++e) v[j][e] = t0 - 3 + j >= 0 || cp.state_in ? v[j][e] : 0.f;
    }
}
// V floats that may not be there: zeros then.
template <int V>
__device__ __forceinline__ void load_if(const ConvParams& cp, const float* p, bool there, float (&v)[V]) {
    const float* q = there ? p : cp.w;
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = q[e];
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = there ? v[e] : 0.f;
}

// The rows t0 .. of one tensor for this thread's channels, `last` rows behind t0 at most.
template <typename T, int V, typename Stride>
struct Rows {
    typedef typename Vec<T, V>::Raw Raw;
    const T* p;  // row t0
    Stride rs;
    int last;
    __device__ __forceinline__ void ask(Raw (&r)[U], int row) const {
#pragma unroll
        for (int j = 0; j < U; ++j) r[j] = *(const Raw*)(p + (uint64_t)(uint32_t)(row + j < last ? row + j : last) * (uint64_t)rs);
    }
};

// What bounds it: the rows from and to memory (2 x 2 bytes a channel and token; 18 us for 4096 x 5376 at the rate of a copy), with the
// sigmoids at half of that time.  With four rows asked for under a condition each and none ahead, 16 bytes a thread, 4096 x 5376 and 6001
// x 5376 took 28 and 38 us alone, 34.5 and 40 inside a step; this takes 19 and 25, and 26 and 30.
// Sequences of a few tokens, a run each, ask for no rows that they do not have, or for four at most: 1024 of 3 tokens and 512 channels, fp32 7.2 -> 5.9 us,
// bf16 5.1 -> 4.5, 512 of 12 tokens and 768 channels fp32 12.4 -> 8.8 (with the whole pipeline of rows under way 16 loads instead of 4).
// WHOLE: every run has `tt` tokens (the last one starts early and stores some rows a second time, the same values): a store under a
// condition would make the waits for the rows count on it not being there.
template <typename T, int V, bool WHOLE>
__global__ __launch_bounds__(64) void k_conv_fwd(ConvParams cp) {
    typedef typename Vec<T, V>::Raw Raw;
    const int c0 = (blockIdx.x * 64 + threadIdx.x) * V;
    if (c0 >= cp.C) return;
    int64_t b = blockIdx.z, t0 = (int64_t)blockIdx.y * cp.tt;
    if (WHOLE && t0 > cp.L - cp.tt) t0 = cp.L - cp.tt;
    const int n = WHOLE ? cp.tt : (int)cp.L;  // tokens of the run
    const Rows<T, V, int64_t> rows = {(const T*)cp.u + b * cp.u_bs + t0 * cp.u_rs + c0, cp.u_rs, n - 1};
    Raw ra[U], rb[U];
    Raw before[3];
    if (n > 0) rows.ask(ra, 0);
    load_before<T, V>(cp, b, t0, c0, before);
    float w[V][CONV_K], bias[V];
    load_if<V>(cp, cp.bias + c0, cp.bias, bias);
#pragma unroll
    for (int e = 0; e < V; ++e) {
#pragma unroll
        for (int k = 0; k < CONV_K; ++k) w[e][k] = cp.w[(c0 + e) * CONV_K + k];
    }
    if (WHOLE ? n > 0 : n > U) rows.ask(rb, U);
    const OutSlot os = out_slot(cp, c0);
    T* out = (T*)os.out + b * os.bs + t0 * os.rs + os.c;
    float win[3][V];  // u[t-3], u[t-2], u[t-1]
    open_before<T, V>(cp, t0, before, win);
    auto use = [&](const Raw (&r)[U], int t) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (WHOLE || t + j < n) {
                float cur[V], o[V];
                Vec<T, V>::open(r[j], cur);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float pre = bias[e] + w[e][0] * win[0][e] + w[e][1] * win[1][e] + w[e][2] * win[2][e] + w[e][3] * cur[e];
                    o[e] = silu(pre);
                    win[0][e] = win[1][e];
                    win[1][e] = win[2][e];
                    win[2][e] = cur[e];
                }
                Vec<T, V>::st(out, 0, o);
                out += os.rs;
                __builtin_amdgcn_sched_barrier(0);  // a row at a time: registers
            }
        }
    };
    for (int t = 0; t < n; t += 2 * U) {
        use(ra, t);
        if (!WHOLE && t + U >= n) break;  // a run of a few tokens has nothing to ask for any more
        rows.ask(ra, t + 2 * U);
        use(rb, t + U);
        if (!WHOLE && t + 2 * U >= n) break;
        rows.ask(rb, t + 3 * U);
    }
    // the state leaving the segment: the last three rows of [state_in ; u]
    if (cp.state_out && t0 + n == cp.L) {
#pragma unroll
        for (int j = 0; j < 3; ++j) Vec<T, V>::st(cp.state_out, (b * 3 + j) * cp.C + c0, win[j]);
    }
}

// Backward.  g[t] = dout[t] silu'(pre[t]);  du[t] = sum_k w[k] g[t+3-k]  (g beyond the segment is 0; what
// the segment on the right contributes to the last three rows arrives as dstate_out);
// dw[k] = sum_t g[t] u[t-3+k];  dbias = sum_t g[t];  dstate_in[j] = du[-3+j].
// The waves of a workgroup take consecutive runs of the same channels, of one sequence or of several, and add up their sums in LDS.  Stores of rows that are not there go to
// an empty descriptor (see k_conv_fwd).  What bounds it: three rows' traffic a token (27 us for 4096 x 5376 at the rate of a copy), and
// nearly as long the vector ALUs.  4096 x 5376 bf16 inside a step, with a wave a workgroup, a row at a time and every run's sums to
// memory (a fifth of the traffic): 50 us and 6.7 for the sums' reduction; now 38 and 5.4.  64 sequences of 64 tokens, 5376 and 10752 channels, both
// launches: 57 and 144 us with the waves of a workgroup bound to one sequence, which had no runs for them, now 39 and 64.
template <typename T, int V>
__global__ __launch_bounds__(64 * BWD_WAVES, 2) void k_conv_bwd(ConvParams cp) {
    typedef typename Vec<T, V>::Raw Raw;
    __shared__ float sums[BWD_WAVES][5 * V][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first_c = blockIdx.x * 64 * V, c0 = first_c + lane * V;
    if (c0 >= cp.C) return;
    const uint32_t wg = blockIdx.z * gridDim.y + blockIdx.y;
    if (wg >= cp.nwg) return;
    const uint32_t run = wg * BWD_WAVES + wv, seq = run / cp.nruns;
    const int64_t b = seq, first = (int64_t)(run - seq * cp.nruns) * cp.tt;  // first own token
    float acc[5][V];
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[k][e] = 0.f;
    if (seq < cp.batch) {
        // the run: tokens 0 .. n - 1 from t0 on, of which those in front of `skip` are another's
        const int64_t t0 = first > cp.L - cp.tt ? (cp.L > cp.tt ? cp.L - cp.tt : 0) : first;
        const int n = (int)(cp.L < cp.tt ? cp.L : cp.tt), skip = (int)(first - t0);
        const int left = (int)(cp.L - t0 < n + 3 ? cp.L - t0 : n + 3);  // and those whose g they need
        const OutSlot os = out_slot(cp, c0);
        const Rows<T, V, int64_t> ru = {(const T*)cp.u + b * cp.u_bs + t0 * cp.u_rs + c0, cp.u_rs, left - 1};
        const Rows<T, V, uint32_t> rd = {(const T*)os.dout + b * os.bs + t0 * os.rs + os.c, (uint32_t)os.rs, left - 1};
        Raw ua[U], ub[U], da[U], db[U];
        if (left > 0) ru.ask(ua, 0), rd.ask(da, 0);
        Raw before[3];
        load_before<T, V>(cp, b, t0, c0, before);
        float w[V][CONV_K], bias[V];
        load_if<V>(cp, cp.bias + c0, cp.bias, bias);
#pragma unroll
        for (int e = 0; e < V; ++e) {
#pragma unroll
            for (int k = 0; k < CONV_K; ++k) w[e][k] = cp.w[(c0 + e) * CONV_K + k];
        }
        // what arrives from the right for the last three rows, and for those of the entering state that a sequence shorter than three
        // tokens passes straight through to the state it leaves (row j of it: row L - 3 + j of [state_in ; u])
        float right[3][V];
#pragma unroll
        for (int j = 0; j < 3; ++j) load_if<V>(cp, cp.dstate_out + (b * 3 + j) * cp.C + c0, cp.dstate_out && t0 + n > cp.L - 3, right[j]);
        if (left > 0) ru.ask(ub, U), rd.ask(db, U);
        float win[3][V];  // u[t-3], u[t-2], u[t-1]
        open_before<T, V>(cp, t0, before, win);
        float gw[3][V];   // g[t-3], g[t-2], g[t-1]; before the run (or the sequence) they are not needed: zeros
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int e = 0; e < V; ++e) gw[j][e] = 0.f;
        const T* du = (const T*)cp.du + b * cp.u_bs + (t0 - 3) * cp.u_rs + first_c;  // row t - 3
        const int width = (cp.C - first_c < 64 * V ? cp.C - first_c : 64 * V) * (int)sizeof(T);
        float few[5][V];  // sums of eight tokens: a chain of all of them would round more often on its way
        // one token: g[t] from its rows of u and dout (zeros beyond the sequence), then du[t-3]
        auto token = [&](int t, const Raw& ur, const Raw& dr) __attribute__((always_inline)) {
            float cur[V], dv[V], g[V], o[V];
            Vec<T, V>::open(ur, cur);
            Vec<T, V>::open(dr, dv);
            const bool in = t < left;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float pre = bias[e] + w[e][0] * win[0][e] + w[e][1] * win[1][e] + w[e][2] * win[2][e] + w[e][3] * cur[e];
                g[e] = in ? dv[e] * dsilu(pre) : 0.f;
            }
            if (t < n && t >= skip) {  // own token: its share of dw and dbias
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    few[0][e] += g[e] * win[0][e];
                    few[1][e] += g[e] * win[1][e];
                    few[2][e] += g[e] * win[2][e];
                    few[3][e] += g[e] * cur[e];
                    few[4][e] += g[e];
                }
            }
            // du[t-3] = w3 g[t-3] + w2 g[t-2] + w1 g[t-1] + w0 g[t]
            const int to = t - 3;
#pragma unroll
            for (int e = 0; e < V; ++e) o[e] = w[e][3] * gw[0][e] + w[e][2] * gw[1][e] + w[e][1] * gw[2][e] + w[e][0] * g[e];
            const int64_t behind = t0 + to - (cp.L - 3);
            if (behind >= 0) {
#pragma unroll
                for (int e = 0; e < V; ++e) o[e] += right[0][e], right[0][e] = right[1][e], right[1][e] = right[2][e], right[2][e] = 0.f;
            }
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)du, 0, to >= 0 && to < n ? width : 0, 0x00020000);
            Vec<T, V>::put(rsrc, lane * V * (int)sizeof(T), o);
            du += cp.u_rs;
            if (t0 == 0 && to < 0 && cp.dstate_in) {  // a row of the entering state
#pragma unroll
                for (int e = 0; e < V; ++e) cp.dstate_in[(b * 3 + (to + 3)) * cp.C + c0 + e] = o[e];
            }
#pragma unroll
            for (int e = 0; e < V; ++e) {
                gw[0][e] = gw[1][e];
                gw[1][e] = gw[2][e];
                gw[2][e] = g[e];
                win[0][e] = win[1][e];
                win[1][e] = win[2][e];
                win[2][e] = in ? cur[e] : 0.f;
            }
            __builtin_amdgcn_sched_barrier(0);  // a token at a time: registers
        };
        for (int t = 0; t < n + 3; t += 2 * U) {
#pragma unroll
            for (int k = 0; k < 5; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) few[k][e] = 0.f;
#pragma unroll
            for (int j = 0; j < U; ++j) token(t + j, ua[j], da[j]);
            if (left > 0) ru.ask(ua, t + 2 * U), rd.ask(da, t + 2 * U);
#pragma unroll
            for (int j = 0; j < U; ++j) token(t + U + j, ub[j], db[j]);
            if (left > 0) ru.ask(ub, t + 3 * U), rd.ask(db, t + 3 * U);
#pragma unroll
            for (int k = 0; k < 5; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) acc[k][e] += few[k][e];
        }
    }
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int e = 0; e < V; ++e) sums[wv][k * V + e][lane] = acc[k][e];
    __syncthreads();
    float* part = cp.part + ((int64_t)wg * 5) * cp.C;
    for (int i = wv; i < 5 * V; i += BWD_WAVES) {
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < BWD_WAVES; ++q) t += sums[q][i][lane];
        part[(int64_t)(i / V) * cp.C + c0 + i % V] = t;
    }
}

// dw and dbias from the tiles' partial sums, rows of [5][C], in a fixed order.
__global__ __launch_bounds__(COLSUM_THREADS) void k_conv_reduce(const float* part, int64_t nparts, int C, float* dw, float* dbias, int accumulate) {
    __shared__ ColsumLds L;
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);  // over 5 * C
    const float s = column_sum(L, part, nparts, 5 * (int64_t)C, i, i < 5 * C);
    if (threadIdx.x < 64 && i < 5 * C) {
        const int k = i / C, c = i - k * C;
        if (k < 4) {
            float* o = dw + (int64_t)c * 4 + k;
            *o = accumulate ? *o + s : s;
        } else if (dbias) {
            dbias[c] = accumulate ? dbias[c] + s : s;
        }
    }
}

int check(const ssd_conv_shape_t* sh) {
    if (!sh) return SSD_ERR_NULL;
    if (sh->dtype != SSD_F32 && sh->dtype != SSD_BF16) return SSD_ERR_DTYPE;
    if (sh->batch <= 0 || sh->batch > 65535 || sh->seqlen < 0 || sh->channels <= 0) return SSD_ERR_SHAPE;
    if ((sh->seqlen + MAX_TT - 1) / MAX_TT > 65535) return SSD_ERR_SHAPE;  // grid.y (long sequences run MAX_TT tokens per thread)
    if (sh->u_row_stride && sh->u_row_stride < sh->channels) return SSD_ERR_SHAPE;
    if (sh->batch_stride && sh->batch_stride < sh->seqlen * (sh->u_row_stride ? sh->u_row_stride : sh->channels)) return SSD_ERR_SHAPE;
    return SSD_OK;
}

// Tokens per thread, `less` fewer than a multiple of 2 U and than `most`: one round of `waves` waves, evenly filled, unless that makes the runs too short or
// too long.  Forward with 2048 / 3072 / 4096 / 5120 waves, 6001 x 5376: 25.9, 27.6, 24.9, 24.7 us; backward with 1024 / 2048 / 3072 / 4096:
// 53.9, 53.9, 48.4, 58.6 (3072 fit, of the others some run behind the rest).  Waves of V channels a thread: with four counted for two (fp32)
// or one, runs were too short, and the launch twice or four times as many waves as fit: 4096 x 1792 fp32 13.2 us, now 12.0.
int pick_tt(const ssd_conv_shape_t* sh, int V, int waves, int most, int less) {
    const int64_t cols = ((int64_t)sh->channels + 64 * V - 1) / (64 * V) * sh->batch;  // waves side by side, at least one
    const int64_t runs = cols < waves ? waves / cols : 1, tt = (sh->seqlen + runs - 1) / runs + less;
    return (tt > most - 2 * U ? most : tt < MIN_TT ? MIN_TT : (int)(tt + 2 * U - 1) / (2 * U) * (2 * U)) - less;
}
constexpr int FWD_FILL = 5120, BWD_FILL = 3072;  // waves that fit the registers of the chip
int fwd_tt(const ssd_conv_shape_t* sh, int V) { return pick_tt(sh, V, FWD_FILL, MAX_TT, 0); }
// (three tokens more go through the loop; a workgroup's sums stand for at least 256 tokens of a long sequence; the workspace's size
// follows, and a caller asks for it without the layout that decides how many channels a thread takes)
int bwd_tt(const ssd_conv_shape_t* sh) { return pick_tt(sh, 4, BWD_FILL, MAX_TT + 2 * U, 3); }
// Runs of a sequence (an empty one has one too) and workgroups for all of them: 65535 sequences of 65535 MAX_TT tokens stay below 2^32 runs.
uint32_t bwd_runs(const ssd_conv_shape_t* sh) { return sh->seqlen ? (uint32_t)((sh->seqlen + bwd_tt(sh) - 1) / bwd_tt(sh)) : 1; }
uint32_t bwd_wgs(const ssd_conv_shape_t* sh, uint64_t runs) { return (uint32_t)(((uint64_t)sh->batch * runs + BWD_WAVES - 1) / BWD_WAVES); }
// The most runs of any sequence up to this length: a longer one may have fewer (5376 channels, 730 and 731 tokens: 146 of 5, 57 of 13), and a buffer for the
// longest segment has to do for a shorter last one.  Runs of every length between the shortest and the longest: as many as one round holds at most.
uint64_t bwd_most_runs(const ssd_conv_shape_t* sh) {
    const uint64_t cols = (((uint64_t)sh->channels + 255) / 256) * (uint64_t)sh->batch, round = cols < BWD_FILL ? BWD_FILL / cols : 1;
    const uint64_t shortest = ((uint64_t)sh->seqlen + MIN_TT - 4) / (MIN_TT - 3), longest = ((uint64_t)sh->seqlen + MAX_TT + 2 * U - 4) / (MAX_TT + 2 * U - 3);
    const uint64_t fit = shortest < round ? shortest : round, most = fit > longest ? fit : longest;
    return most > 0 ? most : 1;
}
size_t bwd_bytes(const ssd_conv_shape_t* sh, uint64_t runs) { return ((size_t)bwd_wgs(sh, runs) * 5 * (size_t)sh->channels * 4 + 255) & ~(size_t)255; }

}  // namespace
}  // namespace ssdk

using namespace ssdk;

extern "C" size_t ssd_conv1d_workspace_bytes(const ssd_conv_shape_t* sh) {
    if (check(sh) != SSD_OK) return 0;
    return bwd_bytes(sh, bwd_most_runs(sh));
}

namespace ssdk {
namespace {

// split: the three-part form of out / dout; every boundary a multiple of the vector width or the kernels fall
// back to one channel per thread
bool bind_split(ConvParams& cp, const ConvSplit* sp, bool bwd) {
    if (!sp) return true;
    if (sp->c1 <= 0 || sp->c2 <= sp->c1 || sp->c2 >= cp.C) return false;
    cp.split = 1;
    cp.cb[0] = 0;
    cp.cb[1] = sp->c1;
    cp.cb[2] = sp->c2;
    cp.cb[3] = cp.C;
    for (int k = 0; k < 3; ++k) {
        if (cp.L > 0 && !sp->p[k]) return false;
        if (bwd) cp.dout3[k] = sp->p[k];
        else cp.out3[k] = sp->p[k];
    }
    return true;
}

int vec_width(const ConvParams& cp, bool bf) {
    int all = cp.C | (int)cp.u_rs;
    if (cp.split) all |= cp.cb[1] | cp.cb[2];
    return bf ? (all % 8 == 0 ? 4 : 1) : (all % 4 == 0 ? 2 : 1);
}

int conv_fwd_impl(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in, void* out,
                  const ConvSplit* split, void* state_out, void* hip_stream) {
    int rc = check(sh);
    if (rc != SSD_OK) return rc;
    if (!w) return SSD_ERR_NULL;
    if (sh->seqlen > 0 && (!u || (!out && !split))) return SSD_ERR_NULL;
    ConvParams cp;
    memset(&cp, 0, sizeof(cp));
    cp.u = u;
    cp.out = out;
    cp.state_in = state_in;
    cp.state_out = state_out;
    cp.w = w;
    cp.bias = bias;
    cp.L = sh->seqlen;
    cp.C = sh->channels;
    cp.u_rs = sh->u_row_stride ? sh->u_row_stride : sh->channels;
    cp.u_bs = sh->batch_stride ? sh->batch_stride : sh->seqlen * cp.u_rs;
    cp.o_bs = sh->batch_stride ? sh->batch_stride : sh->seqlen * sh->channels;
    if (!bind_split(cp, split, false)) return SSD_ERR_ARG;
    hipStream_t st = (hipStream_t)hip_stream;
    const bool bf = sh->dtype == SSD_BF16;
    const int V = vec_width(cp, bf);
    // an empty sequence still hands the state on: one tile, whose token loop is empty
    cp.tt = fwd_tt(sh, V);
    const dim3 grid((cp.C / V + 63) / 64, (unsigned)(cp.L > 0 ? (cp.L + cp.tt - 1) / cp.tt : 1), (unsigned)sh->batch);
    const bool whole = cp.L >= cp.tt;
#define CONV_FWD(T, W) \
    if (whole) hipLaunchKernelGGL((k_conv_fwd<T, W, true>), grid, dim3(64), 0, st, cp); \
    else hipLaunchKernelGGL((k_conv_fwd<T, W, false>), grid, dim3(64), 0, st, cp)
    if (bf && V == 4) CONV_FWD(bf16_t, 4);
    else if (bf) CONV_FWD(bf16_t, 1);
    else if (V == 2) CONV_FWD(float, 2);
    else CONV_FWD(float, 1);
#undef CONV_FWD
    return hipGetLastError() == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}

int conv_bwd_impl(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in, const void* dout,
                  const ConvSplit* split, const float* dstate_out, void* du, float* dw, float* dbias, float* dstate_in, void* workspace,
                  size_t workspace_bytes, uint32_t flags, void* hip_stream) {
    int rc = check(sh);
    if (rc != SSD_OK) return rc;
    if (flags & ~(uint32_t)SSD_FLAG_ACCUM_PARAM) return SSD_ERR_ARG;
    if (!w || !dw) return SSD_ERR_NULL;
    if (sh->seqlen > 0 && (!u || (!dout && !split) || !du)) return SSD_ERR_NULL;
    if (sh->seqlen > 0 && du == dout) return SSD_ERR_ARG;
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < bwd_bytes(sh, bwd_runs(sh))) return SSD_ERR_WORKSPACE;
    ConvParams cp;
    memset(&cp, 0, sizeof(cp));
    cp.u = u;
    cp.dout = dout;
    cp.du = du;
    cp.state_in = state_in;
    cp.dstate_out = dstate_out;
    cp.dstate_in = dstate_in;
    cp.w = w;
    cp.bias = bias;
    cp.part = (float*)workspace;
    cp.L = sh->seqlen;
    cp.C = sh->channels;
    cp.u_rs = sh->u_row_stride ? sh->u_row_stride : sh->channels;
    cp.u_bs = sh->batch_stride ? sh->batch_stride : sh->seqlen * cp.u_rs;
    cp.o_bs = sh->batch_stride ? sh->batch_stride : sh->seqlen * sh->channels;
    cp.tt = bwd_tt(sh);
    cp.batch = (uint32_t)sh->batch;
    cp.nruns = bwd_runs(sh);
    cp.nwg = bwd_wgs(sh, cp.nruns);
    if (!bind_split(cp, split, true)) return SSD_ERR_ARG;
    hipStream_t st = (hipStream_t)hip_stream;
    const bool bf = sh->dtype == SSD_BF16;
    const int V = vec_width(cp, bf);
    const uint32_t deep = (cp.nwg + 65534) / 65535;
    const dim3 grid((cp.C / V + 63) / 64, (cp.nwg + deep - 1) / deep, deep);
    if (bf && V == 4) hipLaunchKernelGGL((k_conv_bwd<bf16_t, 4>), grid, dim3(64 * BWD_WAVES), 0, st, cp);
    else if (bf) hipLaunchKernelGGL((k_conv_bwd<bf16_t, 1>), grid, dim3(64 * BWD_WAVES), 0, st, cp);
    else if (V == 2) hipLaunchKernelGGL((k_conv_bwd<float, 2>), grid, dim3(64 * BWD_WAVES), 0, st, cp);
    else hipLaunchKernelGGL((k_conv_bwd<float, 1>), grid, dim3(64 * BWD_WAVES), 0, st, cp);
    if (hipGetLastError() != hipSuccess) return SSD_ERR_LAUNCH;
    hipLaunchKernelGGL(k_conv_reduce, dim3((5 * cp.C + 63) / 64), dim3(COLSUM_THREADS), 0, st, cp.part, (int64_t)cp.nwg, cp.C,
                       dw, dbias, (flags & SSD_FLAG_ACCUM_PARAM) ? 1 : 0);
    return hipGetLastError() == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}

}  // namespace

int conv1d_fwd_split(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in,
                     const ConvSplit& out, void* state_out, hipStream_t st) {
    return conv_fwd_impl(sh, u, w, bias, state_in, nullptr, &out, state_out, st);
}

int conv1d_bwd_split(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias, const void* state_in,
                     const ConvSplit& dout, const float* dstate_out, void* du, float* dw, float* dbias, float* dstate_in,
                     void* workspace, size_t workspace_bytes, uint32_t flags, hipStream_t st) {
    return conv_bwd_impl(sh, u, w, bias, state_in, nullptr, &dout, dstate_out, du, dw, dbias, dstate_in, workspace, workspace_bytes,
                         flags, st);
}

}  // namespace ssdk

extern "C" int ssd_conv1d_fwd(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias,
                              const void* state_in, void* out, void* state_out, void* hip_stream) {
    return conv_fwd_impl(sh, u, w, bias, state_in, out, nullptr, state_out, hip_stream);
}

extern "C" int ssd_conv1d_bwd(const ssd_conv_shape_t* sh, const void* u, const float* w, const float* bias,
                              const void* state_in, const void* dout, const float* dstate_out, void* du, float* dw,
                              float* dbias, float* dstate_in, void* workspace, size_t workspace_bytes, uint32_t flags,
                              void* hip_stream) {
    return conv_bwd_impl(sh, u, w, bias, state_in, dout, nullptr, dstate_out, du, dw, dbias, dstate_in, workspace, workspace_bytes,
                         flags, hip_stream);
}
