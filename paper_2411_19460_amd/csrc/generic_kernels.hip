// Shape-generic kernels of the chunked selective scan: fp32 arithmetic, any P, N, Q within
// the documented limits, fp32 or bf16 storage.  They serve the fp32 configuration, odd shapes,
// and as an on-device cross-check of the bf16 matrix-core kernels.
//
// The chunked ("dual") form of the recurrence of Sec. 3.1, Eq. 1, per (batch, head) and per chunk
// of Q tokens with entering state Hprev (local indices i, j in [0, Q)):
//     a_j = dt_j A, cum_i = sum_{r<=i} a_r, T = cum_{Q-1}, G[i,j] = C_i . B_j
//     S      = sum_j exp(T - cum_j) dt_j x_j (x) B_j           Hnext = exp(T) Hprev + S
//     yhat_i = sum_{j<=i} G[i,j] exp(cum_i - cum_j) dt_j x_j + exp(cum_i) Hprev C_i,   y = yhat + D x
// and, given dY and dHnext,
//     dHprev = exp(T) dHnext + sum_i exp(cum_i) dY_i (x) C_i
//     u_j    = sum_{i>=j} G[i,j] exp(cum_i - cum_j) dY_i + exp(T - cum_j) dHnext B_j,   dx_j = dt_j u_j + D dY_j
//     dG     = sum_{heads of the group} [exp(cum_i - cum_j) dt_j (dY_i . x_j)]_{j<=i}
//     dC_i   = sum_j dG[i,j] B_j + sum_heads exp(cum_i) dY_i^T Hprev
//     dB_j   = sum_i dG[i,j] C_i + sum_heads exp(T - cum_j) dt_j x_j^T dHnext
//     da_r   = sum_{i>=r} dcum_i,  dcum_i = exp(cum_i) dY_i . (Hprev C_i) - s_i + rowsum_i(E) - colsum_i(E)  (+ at the
//              chunk end exp(T) <dHnext, Hprev> + sum_j s_j),  s_j = exp(T - cum_j) dt_j x_j . (dHnext B_j),
//              E[i][j] = G[i,j] exp(cum_i - cum_j) dt_j (dY_i . x_j)
//     ddt_j  = A da_j + x_j . u_j,  dA += sum_j dt_j da_j,  dD += sum dY . x
// Every exponent is formed from a difference that is <= 0, so nothing overflows.
//
// All contractions run on v_mfma_f32_32x32x2_f32: full fp32 products and sums at twice the rate of plain FMAs, and
// with one LDS operand read per four of them instead of five reads per four FMAs, which is what bounded the tiles
// this replaces.  A workgroup of four waves owns a 64 x 64 tile; K goes by in steps of 32, staged through two LDS
// buffers (one barrier a step) as [row][k] with the next step's global loads in flight during the MFMAs.  The weights
// (decays, dt, masks) are applied between the load and the LDS store.  Sums over the heads of a group are cut into head
// slices so that a sequence of a few chunks still fills the machine (1999 tokens of 24 heads in two segments, forward +
// backward: 1340 us with FMA tiles, serial heads and launches of their own for every segment, 253 us now).  Small problems are
// bound by launches: three forward, five backward here for segments that share them (512 tokens of 4 heads in two segments: 216
// us with 14 for each segment, 64 us now).
#include "ddt_finalize.h"
#include "ssd_internal.h"

namespace ssdk {
namespace {

template <typename T>
struct IO;
template <>
struct IO<float> {
    static __device__ __forceinline__ float ld(const void* p, size_t i) { return ((const float*)p)[i]; }
    static __device__ __forceinline__ float round(float v) { return v; }
    static __device__ __forceinline__ void st(void* p, int64_t i, float v) { ((float*)p)[i] = v; }
    static __device__ __forceinline__ void ld4(float (&v)[4], const void* p, size_t i) {  // i a multiple of 4, 16-byte aligned
        const float4 q = *(const float4*)((const float*)p + i);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
};
template <>
struct IO<bf16_t> {
    static __device__ __forceinline__ float ld(const void* p, size_t i) { return bf16_to_float(((const bf16_t*)p)[i]); }
    static __device__ __forceinline__ float round(float v) { return bf16_to_float(float_to_bf16(v)); }
    static __device__ __forceinline__ void st(void* p, int64_t i, float v) { ((bf16_t*)p)[i] = float_to_bf16(v); }
    static __device__ __forceinline__ void ld4(float (&v)[4], const void* p, size_t i) {
        const uint2 q = *(const uint2*)((const bf16_t*)p + i);
        v[0] = __builtin_bit_cast(float, q.x << 16); v[1] = __builtin_bit_cast(float, q.x & 0xffff0000u);
        v[2] = __builtin_bit_cast(float, q.y << 16); v[3] = __builtin_bit_cast(float, q.y & 0xffff0000u);
    }
};

typedef float f32x16 __attribute__((ext_vector_type(16)));

// exp of a difference of sums of dt A: at most 0 but for rounding.  A NaN stays one (fminf would take the number).
__device__ __forceinline__ float decay(float v) { return expf(v > 0.f ? 0.f : v); }

constexpr int NTHREADS = 256;
constexpr int TM = 64;   // tile edge
constexpr int TK = 32;   // contraction step
constexpr int KP = 36;   // floats per LDS row (32 + 4 pad: 16-byte aligned, and eight rows cover the banks)
constexpr int QMAX = 1024;
constexpr int SLICES = GENERIC_SLICES;
static_assert(SLICES == 4, "the sums over slices are written out");

struct Tiles {
    float a[2][TM][KP], b[2][TM][KP];
};
// LDS of the kernels that also keep per-token arrays of the chunk: the tiles, then `n` floats (sized at launch, so that
// four workgroups fit a compute unit up to chunks of 256 tokens).
inline size_t lds_bytes(int n) { return sizeof(Tiles) + (size_t)n * sizeof(float); }
extern __shared__ __attribute__((aligned(16))) char dyn_lds[];

// Four consecutive k (from k0 + k) of row row0 + r, k contiguous in memory; outside [0, rows) x [0, ks) reads as zero.
// The address is a wave-uniform base plus a 32-bit offset inside the tile, and out-of-range indices are clamped and
// their values dropped: no branches, so that a tile's loads leave together.  row0 < rows and k0 < ks.
template <typename T>
__device__ __forceinline__ void ld_k4(float (&v)[4], const void* p, int64_t base, int64_t row_stride, int row0, int r, int k0, int k, int rows,
                                      int ks, bool vec) {
    const T* u = (const T*)p + (base + row0 * row_stride + k0);
    const int rl = rows - row0 - 1, kl = ks - k0;
    if (vec && rl >= TM - 1 && kl >= TK) {  // uniform: a tile inside the matrix
        IO<T>::ld4(v, u, (uint32_t)r * (uint32_t)row_stride + (uint32_t)k);
        return;
    }
    const uint32_t o = (uint32_t)(r < rl ? r : rl) * (uint32_t)row_stride;
    if (vec) {  // ks is a multiple of 4 and rows are 4-element aligned
        IO<T>::ld4(v, u, o + (uint32_t)(k < kl ? k : 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = r <= rl && k < kl ? v[e] : 0.f;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float q = IO<T>::ld(u, o + (uint32_t)(k + e < kl ? k + e : 0));
            v[e] = r <= rl && k + e < kl ? q : 0.f;
        }
    }
}
// The same with the row index contiguous in memory.
template <typename T>
__device__ __forceinline__ void ld_r4(float (&v)[4], const void* p, int64_t base, int64_t k_stride, int r, int k0, int k, int rows, int ks) {
    const T* u = (const T*)p + (base + k0 * k_stride);
    const int kl = ks - k0;
    if (rows >= TM && kl >= TK) {  // uniform
        const uint32_t o = (uint32_t)k * (uint32_t)k_stride + (uint32_t)r;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = IO<T>::ld(u, o + (uint32_t)e * (uint32_t)k_stride);
        return;
    }
    const uint32_t row = (uint32_t)(r < rows ? r : 0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float q = IO<T>::ld(u, row + (uint32_t)(k + e < kl ? k + e : 0) * (uint32_t)k_stride);
        v[e] = r < rows && k + e < kl ? q : 0.f;
    }
}

// The thread index as the optimiser cannot see through: what is derived from it is formed anew in every turn of a loop
// instead of being kept in registers across it (half of the walks' registers otherwise).
__device__ __forceinline__ int opaque_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Where a thread's two groups of four k lie in a [64][32] tile: KC = k contiguous in memory, else the row index is
// (lanes run along what is contiguous).
template <bool KC>
__device__ __forceinline__ void place(int tid, int s, int& row, int& k) {
    const int t = tid + NTHREADS * s;
    row = KC ? t >> 3 : t & 63;
    k = KC ? (t & 7) * 4 : (t >> 6) * 4;
}

template <bool KC, class F>
__device__ __forceinline__ void tile_load(float (&r)[2][4], int k0, F ld) {
    const int tid = opaque_tid();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        int row, k;
        place<KC>(tid, s, row, k);
        ld(r[s], row, k, k0);
    }
}
template <bool KC, class W>
__device__ __forceinline__ void tile_store(float (&r)[2][4], float (*L)[KP], int k0, W wt) {
    const int tid = opaque_tid();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        int row, k;
        place<KC>(tid, s, row, k);
        wt(r[s], row, k0 + k);
        *(float4*)(&L[row][k]) = make_float4(r[s][0], r[s][1], r[s][2], r[s][3]);
    }
}

// acc += the wave's 32 x 32 quadrant of a [64][32] x [64][32]^T product.  Lane half h takes k = 8 j + 4 h .. + 3 of each
// row with one 16-byte read; the e-th MFMA contracts k = 8 j + e and 8 j + 4 + e.
__device__ __forceinline__ void tile_mma(f32x16& acc, const float (*A)[KP], const float (*B)[KP]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5;
    const float* pa = &A[32 * (w >> 1) + (lane & 31)][4 * half];
    const float* pb = &B[32 * (w & 1) + (lane & 31)][4 * half];
#pragma unroll
    for (int j = 0; j < TK / 8; ++j) {
        const float4 a = *(const float4*)(pa + 8 * j), b = *(const float4*)(pb + 8 * j);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
    }
}

// Row and column of accumulator register r of this lane inside the 64 x 64 tile.
__device__ __forceinline__ int tile_row(int r) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    return 32 * (w >> 1) + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
}
__device__ __forceinline__ int tile_col() { return 32 * ((threadIdx.x >> 6) & 1) + (threadIdx.x & 31); }

__device__ __forceinline__ f32x16 zero_acc() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

struct Staged {
    float a[2][4], b[2][4];
};

// acc += A B^T over k in [kbeg, kend), kbeg a multiple of 4.  la / lb load four k of a row (zeros outside), wa / wb then
// weight them in place.  `buf` alternates between the LDS buffers across calls: one barrier per step suffices.
// between() runs once the first loads are under way: what fills the arrays the weights are read from (its barriers
// included) costs no round trip to memory of its own.
template <bool AKC, bool BKC, class LA, class WA, class LB, class WB, class FB>
__device__ __forceinline__ void tile_gemm(f32x16& acc, int kbeg, int kend, LA la, WA wa, LB lb, WB wb, Tiles& L, int& buf, FB between) {
    Staged R0, R1;  // two steps of loads in flight
    auto load = [&](Staged& R, int k0) {
        tile_load<AKC>(R.a, k0, la);
        tile_load<BKC>(R.b, k0, lb);
    };
    auto step = [&](Staged& R, int k0) {
        tile_store<AKC>(R.a, L.a[buf], k0, wa);
        tile_store<BKC>(R.b, L.b[buf], k0, wb);
        __syncthreads();
        if (k0 + 2 * TK < kend) load(R, k0 + 2 * TK);
        tile_mma(acc, L.a[buf], L.b[buf]);
        buf ^= 1;
    };
    if (kbeg < kend) load(R0, kbeg);
    if (kbeg + TK < kend) load(R1, kbeg + TK);
    between();
    for (int k0 = kbeg; k0 < kend; k0 += 2 * TK) {
        step(R0, k0);
        if (k0 + TK < kend) step(R1, k0 + TK);
    }
}
template <bool AKC, bool BKC, class LA, class WA, class LB, class WB>
__device__ __forceinline__ void tile_gemm(f32x16& acc, int kbeg, int kend, LA la, WA wa, LB lb, WB wb, Tiles& L, int& buf) {
    tile_gemm<AKC, BKC>(acc, kbeg, kend, la, wa, lb, wb, L, buf, [] {});
}
struct NoWeight {
    __device__ __forceinline__ void operator()(float (&)[4], int, int) const {}
};

// Sum of each of the 16 registers over the 32 lanes of a half wave, by recursive halving; lane l (of the half) ends
// with the sum of register l / 2.
__device__ __forceinline__ float row_sums(const f32x16& v, int lane) {
    float a[8], b[4], c[2];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const float keep = lane & 16 ? v[r + 8] : v[r], give = lane & 16 ? v[r] : v[r + 8];
        a[r] = keep + __shfl_xor(give, 16, 64);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float keep = lane & 8 ? a[r + 4] : a[r], give = lane & 8 ? a[r] : a[r + 4];
        b[r] = keep + __shfl_xor(give, 8, 64);
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float keep = lane & 4 ? b[r + 2] : b[r], give = lane & 4 ? b[r] : b[r + 2];
        c[r] = keep + __shfl_xor(give, 4, 64);
    }
    const float keep = lane & 2 ? c[1] : c[0], give = lane & 2 ? c[0] : c[1];
    const float d = keep + __shfl_xor(give, 2, 64);
    return d + __shfl_xor(d, 1, 64);
}

__global__ void k_fill_zero(float* p, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0.f;
}

__global__ void k_copy_f32(float* dst, const float* src, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dst[i] = src[i];
}

// Which 16-byte loads along the contiguous dimension are possible.
struct Vec {
    bool x, bc;  // rows of x, dY (and dx, y are stored by element); rows of B, C and the states
};

// ---------------------------------------------------------------------------------------------
// Step 1, one launch: the scores and the chunk states (backward: and the local state adjoints).
// The first n_cb workgroups each do one 64 x 64 tile of  Gm[b,c,g,i,j] = C_i . B_j  on or below the diagonal; the
// others one 64 x 64 tile of
//   role 0: states[b,c,h,p,n]  = sum_j exp(T - cum_j) dt_j x_j[p] B_j[n]
//   role 1: dstates[b,c,h,p,n] = sum_i exp(cum_i) dY_i[p] C_i[n]
// after forming cum (the chunk-local inclusive cumsum of dt A) of their head for themselves; the workgroup of tile
// (0, 0) of role 0 stores cum and dt for the steps that follow.
// RAW: dt as it leaves a projection.  A template argument: as a branch it took 0.5 us of the 8.4 and 26.6 that the kernel
// takes of 512 and 2048 tokens (fp32, 8 and 24 heads).
template <typename T, bool RAW>
__global__ __launch_bounds__(NTHREADS, 4) void k_scores_states(SegParams sp, Vec vec, int n_cb, int nroles) {
    Tiles& L = *(Tiles*)dyn_lds;
    float* red = (float*)(dyn_lds + sizeof(Tiles));  // [4], then the tokens' weights [Q]
    float* wt = red + NTHREADS / 64;
    const int Q = sp.Q, N = sp.N, P = sp.P;
    const int64_t bt = (int64_t)sp.G * N;
    int z = blockIdx.x, buf = 0;
    f32x16 acc = zero_acc();
    if (z < n_cb) {
        const int NT = (Q + TM - 1) / TM, npair = NT * (NT + 1) / 2;
        int pair = z % npair, I = 0;
        z /= npair;
        while (pair > I) pair -= ++I;
        const int i0 = I * TM, j0 = pair * TM;
        const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc), V = chunk_rows(sp, c, Q);
        if (i0 >= V) return;
        const int64_t base = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
        tile_gemm<true, true>(
            acc, 0, N, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.Cm, base, bt, i0, r, k0, k, V, N, vec.bc); }, NoWeight{},
            [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.Bm, base, bt, j0, r, k0, k, V, N, vec.bc); }, NoWeight{}, L, buf);
        float* out = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = i0 + tile_row(r), j = j0 + tile_col();
            if (i < Q && j < Q) out[(int64_t)i * Q + j] = acc[r];
        }
        return;
    }
    z -= n_cb;
    const int NP = (P + TM - 1) / TM, NN = (N + TM - 1) / TM;
    const int n0 = (z % NN) * TM;
    z /= NN;
    const int p0 = (z % NP) * TM;
    z /= NP;
    const int role = z % nroles;
    z /= nroles;
    const int h = z % sp.H, c = (z / sp.H) % sp.nc, b = z / (sp.H * sp.nc), g = h / sp.hpg, V = chunk_rows(sp, c, Q);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    auto form_cum = [&] {  // thread t owns the E consecutive tokens from t E on
        const int E = (Q + NTHREADS - 1) / NTHREADS;
        const float A = sp.A[h];
        float d[QMAX / NTHREADS], a[QMAX / NTHREADS], run = 0.f;
        for (int e = 0; e < QMAX / NTHREADS; ++e) {
            const int i = tid * E + e;
            const bool live = e < E && i < V;
            if (RAW) d[e] = live ? IO<T>::round(softplus(IO<T>::ld(sp.raw.dt, ((int64_t)c * Q + i) * sp.raw.rs + h) + sp.raw.bias[h])) : 0.f;
            else d[e] = live ? IO<T>::ld(sp.dt, (int64_t)b * sp.dts_b + ((int64_t)c * Q + i) * sp.H + h) : 0.f;
            run += d[e] * A + ((live && sp.reset && sp.reset[(int64_t)b * sp.reset_bs + (int64_t)c * Q + i]) ? RESET_LOG_DECAY : 0.f);
            a[e] = run;
        }
        float incl = run;  // inclusive scan of the threads' totals over the wave, then over the waves
        for (int off = 1; off < 64; off <<= 1) {
            const float v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        if (lane == 63) red[w] = incl;
        __syncthreads();
        float before = incl - run, total = 0.f;
        for (int q = 0; q < NTHREADS / 64; ++q) {
            before += q < w ? red[q] : 0.f;
            total += red[q];
        }
        const bool keep = role == 0 && n0 == 0 && p0 == 0;
        const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
        for (int e = 0; e < QMAX / NTHREADS; ++e) {
            const int i = tid * E + e;
            if (e < E && i < Q) {
                const float cum = before + a[e];
                wt[i] = role == 0 ? decay(total - cum) * d[e] : expf(cum);
                if (keep) {
                    sp.cum[o + i] = i == Q - 1 ? total : cum;
                    sp.dtf[o + i] = d[e];
                }
            }
        }
        __syncthreads();
    };
    const void* lhs = role == 0 ? sp.x : sp.dy;
    const void* rhs = role == 0 ? sp.Bm : sp.Cm;
    const int64_t xt = (int64_t)sp.H * P;
    const int64_t xbase = (int64_t)b * (role == 0 ? sp.xs_b : sp.dys_b) + ((int64_t)c * Q * sp.H + h) * P + p0;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N + n0;
    tile_gemm<false, false>(
        acc, 0, V, [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, lhs, xbase, xt, r, k0, k, P - p0, V); },
        [&](float (&v)[4], int, int k) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + e < Q) v[e] *= wt[k + e];
        },
        [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, rhs, bbase, bt, r, k0, k, N - n0, V); }, NoWeight{}, L, buf, form_cum);
    float* out = role == 0 ? sp.states + (((int64_t)b * (sp.nc + 1) + c) * sp.H + h) * P * N
                           : sp.dstates + (((int64_t)b * sp.nc + c) * sp.H + h) * P * N;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int p = p0 + tile_row(r), n = n0 + tile_col();
        if (p < P && n < N) out[(int64_t)p * N + n] = acc[r];
    }
}

// ---------------------------------------------------------------------------------------------
// Step 2: inter-chunk state passing over one span, one thread per state element, sequential in chunks with the loads
// of SU chunks in flight.  Forward pass: one walk that puts the checkpoints of the span's segments down on the way.
// Backward pass (BWD): the states entering the chunks, every segment restarted from its checkpoint, then the way back
// over the chunk-state adjoints, with the partial sums (one per wave) of exp(T_c) <dHnext_c, Hprev_c>.
constexpr int SU = 8;

template <bool BWD>
__global__ __launch_bounds__(NTHREADS) void k_state_scan(SegParams sp) {
    const int PN = sp.P * sp.N, nc = sp.nc;
    const int e = blockIdx.x * NTHREADS + threadIdx.x, h = blockIdx.y, b = blockIdx.z;
    const bool live = e < PN;
    const int el = live ? e : PN - 1;
    const int64_t bh = (int64_t)h * PN + el, HPN = (int64_t)sp.H * PN;
    float hc = 0.f;
    if (sp.state_in) hc = sp.state_in[(int64_t)b * sp.state_in_bs + bh];
    else if (sp.state_in16) hc = bf16_to_float(sp.state_in16[(int64_t)b * sp.state_in_bs + bh]);  // bf16 checkpoint
    if (live && sp.bnd_write) sp.bnd_write[(int64_t)b * sp.bnd_write_bs + bh] = hc;
    if (live && sp.bnd_write16) sp.bnd_write16[(int64_t)b * sp.bnd_write_bs + bh] = float_to_bf16(hc);
    const float* cum = sp.cum + ((int64_t)b * sp.H + h) * nc * sp.Q + sp.Q - 1;
    float* S = sp.states + (int64_t)b * (nc + 1) * HPN + bh;
    int next = sp.ckpt || sp.ckpt16 ? sp.seg_chunks : nc;  // chunk at which the next segment of the span starts
    int64_t slot = (int64_t)b * sp.ckpt_bs + bh;
    for (int c0 = 0; c0 < nc; c0 += SU) {
        float sv[SU], av[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = c0 + u < nc ? c0 + u : nc - 1;
            sv[u] = S[c * HPN];
            av[u] = cum[(int64_t)c * sp.Q];
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = c0 + u;
            if (c >= nc) break;
            if (c == next) {
                next += sp.seg_chunks;
                slot += HPN;
                if (BWD) {
                    hc = sp.ckpt16 ? bf16_to_float(sp.ckpt16[slot]) : sp.ckpt[slot];
                } else if (live) {
                    if (sp.ckpt) sp.ckpt[slot] = hc;
                    if (sp.ckpt16) sp.ckpt16[slot] = float_to_bf16(hc);
                }
            }
            if (live) S[c * HPN] = hc;
            hc = expf(av[u]) * hc + sv[u];
        }
    }
    if (!BWD) {
        if (!live) return;
        if (sp.state_out) sp.state_out[(int64_t)b * sp.state_out_bs + bh] = hc;
        if (sp.state_out2) sp.state_out2[(int64_t)b * sp.state_out2_bs + bh] = hc;
        if (sp.state_out16) sp.state_out16[(int64_t)b * sp.state_out16_bs + bh] = float_to_bf16(hc);
        return;
    }
    if (sp.first_span && e == 0 && b == 0) sp.param_count[(int64_t)h * sp.param_stride] = 0;
    const int64_t ce = (int64_t)b * HPN + bh;
    float g = sp.dcarry_in ? sp.dcarry_in[ce] : 0.f;
    float* dS = sp.dstates + (int64_t)b * nc * HPN + bh;
    for (int c0 = nc - 1; c0 >= 0; c0 -= SU) {
        float lv[SU], hv[SU], av[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = c0 - u >= 0 ? c0 - u : 0;
            lv[u] = dS[c * HPN];
            hv[u] = S[c * HPN];
            av[u] = cum[(int64_t)c * sp.Q];
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = c0 - u;
            if (c < 0) break;
            if (live) dS[c * HPN] = g;
            const float a = expf(av[u]);
            float part = live ? a * g * hv[u] : 0.f;
            for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
            if ((threadIdx.x & 63) == 0)
                sp.tail_part[(((int64_t)b * sp.H + h) * nc + c) * sp.nslice + blockIdx.x * (NTHREADS / 64) + (threadIdx.x >> 6)] = part;
            g = a * g + lv[u];
        }
    }
    if (live) {
        sp.dcarry[ce] = g;
        if (sp.dinit_out) sp.dinit_out[ce] = g;
    }
}

// ---------------------------------------------------------------------------------------------
// Step 3 forward: y = (G o decay o dt) X + exp(cum) C Hprev^T + D x   (+ x under the residual flag); one 64 x 64 tile.
template <typename T>
__global__ __launch_bounds__(NTHREADS, 4) void k_chunk_out(SegParams sp, Vec vec) {
    const int Q = sp.Q, N = sp.N, P = sp.P;
    Tiles& L = *(Tiles*)dyn_lds;
    float *cum = (float*)(dyn_lds + sizeof(Tiles)), *dtf = cum + Q, *rowf = dtf + Q, *srow = rowf + TM;
    const int p0 = blockIdx.y * TM, i0 = ((int)gridDim.z - 1 - (int)blockIdx.z) * TM;  // the longest rows first
    const int z = blockIdx.x, h = z % sp.H, c = (z / sp.H) % sp.nc, b = z / (sp.H * sp.nc), g = h / sp.hpg, V = chunk_rows(sp, c, Q);
    if (i0 >= V) return;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
    const int kend = i0 + TM < V ? i0 + TM : V;
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const float* Hprev = sp.states + (((int64_t)b * (sp.nc + 1) + c) * sp.H + h) * P * N;
    const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P;
    const int64_t xbase = (int64_t)b * sp.xs_b + xrow, ybase = (int64_t)b * sp.ys_b + xrow;
    const int64_t xt = (int64_t)sp.H * P;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
    int buf = 0;
    f32x16 acc = zero_acc();
    auto la = [&](float (&v)[4], int r, int k, int k0) { ld_k4<float>(v, Gm, 0, Q, i0, r, k0, k, V, Q, (Q & 3) == 0); };
    auto lb = [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, sp.x, xbase + p0, xt, r, k0, k, P - p0, V); };
    // Tokens before the tile: exp(cum_i - cum_k) = exp(cum_i - cum_ref) exp(cum_ref - cum_k) with the token in front of
    // the tile as reference, both <= 1: one exp per token instead of one per score; the first factor scales the rows at
    // the end.  Only the diagonal tile takes an exp per score.  The entering state's weight exp(cum_i) too is applied to the
    // rows of its product.  (Weights in the operands of that product and the rows' exps in every lane: 600 instructions a
    // wave more, 4096 tokens of 24 heads 36.6 us, now 32.)
    const float ref = i0 > 0 ? sp.cum[cbase + i0 - 1] : 0.f;
    tile_gemm<true, false>(
        acc, 0, i0, la,
        [&](float (&v)[4], int, int k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= dtf[k + e];
        },
        lb, NoWeight{}, L, buf, [&] {
            for (int i = threadIdx.x; i < kend; i += NTHREADS) {
                const float c_ = sp.cum[cbase + i], d_ = sp.dtf[cbase + i];
                cum[i] = c_;
                dtf[i] = i < i0 ? decay(ref - c_) * d_ : d_;
                if (i >= i0) {
                    rowf[i - i0] = decay(c_ - ref);
                    srow[i - i0] = expf(c_);
                }
            }
            __syncthreads();
        });
    if (i0 > 0)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] *= i0 + tile_row(r) < V ? rowf[tile_row(r)] : 0.f;
    tile_gemm<true, false>(
        acc, i0, kend, la,
        [&](float (&v)[4], int r, int k) {
            const int i = i0 + r;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (i < V && k + e <= i) ? v[e] * expf(cum[i] - cum[k + e]) * dtf[k + e] : 0.f;
        },
        lb, NoWeight{}, L, buf);
    f32x16 t = zero_acc();
    tile_gemm<true, true>(
        t, 0, N, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.Cm, bbase, bt, i0, r, k0, k, V, N, vec.bc); }, NoWeight{},
        [&](float (&v)[4], int r, int k, int k0) { ld_k4<float>(v, Hprev, (int64_t)p0 * N, N, 0, r, k0, k, P - p0, N, (N & 3) == 0); }, NoWeight{}, L, buf);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = fmaf(t[r], i0 + tile_row(r) < V ? srow[tile_row(r)] : 0.f, acc[r]);
    const float Dh = sp.D[h] + ((sp.flags & SSD_FLAG_RESIDUAL) ? 1.f : 0.f);
    const int p = p0 + tile_col();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + tile_row(r);
        if (i < V && p < P) {
            const int64_t o = (int64_t)i * xt + p;
            IO<T>::st(sp.y, ybase + o, acc[r] + Dh * IO<T>::ld(sp.x, xbase + o));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Step 3 backward, one launch of three kinds of workgroups.  Sums over the tile's columns are left as partial sums per
// 32 columns (or rows) and added in a fixed order by the last step.
struct WalkLds {
    Tiles t;
    union {
        float ch[1];  // walk_u: cum [Q], dt [Q], the rows' factors [2][TM]
        struct { float row[2][TM], col[2][TM], dcol[2][TM]; } hd;
    };
};

// u rows j0.. of one (chunk, head): transposed masked scores (without dt) times dY, then the leaving-adjoint term;
// dx = dt u + D dY, and per token x . u (fterm) and dY . x (dDrow)
template <typename T>
__device__ __forceinline__ void walk_u(const SegParams& sp, const Vec& vec, WalkLds& L, int z) {
    const int Q = sp.Q, N = sp.N, P = sp.P, NT = (Q + TM - 1) / TM, NP = (P + TM - 1) / TM;
    const int j0 = (z % NT) * TM;  // tile 0 has the longest contraction
    z /= NT;
    const int p0 = (z % NP) * TM;
    z /= NP;
    const int h = z % sp.H, c = (z / sp.H) % sp.nc, b = z / (sp.H * sp.nc), g = h / sp.hpg, V = chunk_rows(sp, c, Q);
    if (j0 >= V) return;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
    float *cum = L.ch, *dtf = L.ch + Q, *rowf = dtf + Q, *srow = rowf + TM;
    const float T_ = sp.cum[cbase + Q - 1];
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const float* dHnext = sp.dstates + (((int64_t)b * sp.nc + c) * sp.H + h) * P * N;
    const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P;
    const int64_t xbase = (int64_t)b * sp.xs_b + xrow, dybase = (int64_t)b * sp.dys_b + xrow, dxbase = (int64_t)b * sp.dxs_b + xrow;
    const int64_t xt = (int64_t)sp.H * P;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
    const float Dh = sp.D[h] + ((sp.flags & SSD_FLAG_RESIDUAL) ? 1.f : 0.f);
    int buf = 0;
    f32x16 acc = zero_acc();
    auto la = [&](float (&v)[4], int r, int k, int k0) { ld_r4<float>(v, Gm, j0, Q, r, k0, k, V - j0, V); };
    auto lb = [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, sp.dy, dybase + p0, xt, r, k0, k, P - p0, V); };
    // tokens behind the tile: the decay split at the tile's last token, as in k_chunk_out
    const int j1 = j0 + TM < V ? j0 + TM : V;
    const float ref = sp.cum[cbase + j1 - 1];
    tile_gemm<false, false>(
        acc, j1, V, la,
        [&](float (&v)[4], int, int k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] *= k + e < V ? cum[k + e] : 0.f;
        },
        lb, NoWeight{}, L.t, buf, [&] {
            for (int i = threadIdx.x; i < V; i += NTHREADS) {
                const float c_ = sp.cum[cbase + i];
                cum[i] = i < j1 ? c_ : decay(c_ - ref);
                dtf[i] = sp.dtf[cbase + i];
                if (i >= j0 && i < j1) {
                    rowf[i - j0] = decay(ref - c_);
                    srow[i - j0] = expf(T_ - c_);
                }
            }
            __syncthreads();
        });
    if (j1 < V)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] *= rowf[tile_row(r)];
    tile_gemm<false, false>(
        acc, j0, j1, la,
        [&](float (&v)[4], int r, int k) {
            const int j = j0 + r;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (j < V && k + e < V && k + e >= j) ? v[e] * expf(cum[k + e] - cum[j]) : 0.f;
        },
        lb, NoWeight{}, L.t, buf);
    f32x16 t = zero_acc();
    tile_gemm<true, true>(
        t, 0, N, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.Bm, bbase, bt, j0, r, k0, k, V, N, vec.bc); }, NoWeight{},
        [&](float (&v)[4], int r, int k, int k0) { ld_k4<float>(v, dHnext, (int64_t)p0 * N, N, 0, r, k0, k, P - p0, N, (N & 3) == 0); }, NoWeight{}, L.t, buf);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = fmaf(t[r], j0 + tile_row(r) < V ? srow[tile_row(r)] : 0.f, acc[r]);
    const int p = p0 + tile_col();
    f32x16 dyx;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = j0 + tile_row(r);
        const bool live = j < V && p < P;
        const int64_t o = live ? (int64_t)j * xt + p : (int64_t)j0 * xt;
        const float dyv = IO<T>::ld(sp.dy, dybase + o), xv = IO<T>::ld(sp.x, xbase + o);
        if (live) IO<T>::st(sp.dx, dxbase + o, dtf[j] * acc[r] + Dh * dyv);
        acc[r] *= live ? xv : 0.f;
        dyx[r] = live ? dyv * xv : 0.f;
    }
    const int lane = threadIdx.x & 63, piece = 2 * (p0 / TM) + ((threadIdx.x >> 6) & 1);
    const float f = row_sums(acc, lane), d = row_sums(dyx, lane);
    if ((lane & 1) == 0) {  // lane l of a half holds the sum of register (l % 32) / 2
        const int j = j0 + tile_row((lane & 31) >> 1);
        if (j < V) {
            const int64_t o = piece * sp.tok_stride + cbase + j;
            sp.fterm[o] = f;
            sp.dDrow[o] = d;
        }
    }
}

// One 64 x 64 tile (on or below the diagonal) of dG[b,c,g,i,j] = sum over the heads of a slice of
// exp(cum_i - cum_j) dt_j (dY_i . x_j), and per head the row and column sums of E = that (.) G
template <typename T>
__device__ __forceinline__ void walk_dg(const SegParams& sp, const Vec& vec, WalkLds& L, int z) {
    const int Q = sp.Q, P = sp.P, NT = (Q + TM - 1) / TM, npair = NT * (NT + 1) / 2;
    int pair = z % npair, I = 0;
    z /= npair;
    while (pair > I) pair -= ++I;
    const int i0 = I * TM, j0 = pair * TM, ns = sp.dg_split, slice = z % ns;
    z /= ns;
    const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc), V = chunk_rows(sp, c, Q);
    if (i0 >= V) return;
    const int hps = sp.hpg / ns, h0 = g * sp.hpg + slice * hps, tid = threadIdx.x, lane = tid & 63;
    const int64_t xt = (int64_t)sp.H * P;
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const int col = tile_col(), j = j0 + col;
    float gv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + tile_row(r);
        gv[r] = (i < V && j <= i) ? Gm[(int64_t)i * Q + j] : 0.f;
    }
    f32x16 tot = zero_acc();
    const int KS = (P + TK - 1) / TK;
    float ra[2][4], rb[2][4], rc = 0.f, rf = 0.f;
    auto load = [&](int s) {  // contraction step s % KS of head s / KS; with the first one, that head's cum and dt
        const int h = h0 + s / KS, k0 = (s % KS) * TK;
        const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P;
        const int64_t xbase = (int64_t)b * sp.xs_b + xrow, dybase = (int64_t)b * sp.dys_b + xrow;
        tile_load<true>(ra, k0, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.dy, dybase, xt, i0, r, k0, k, V, P, vec.x); });
        tile_load<true>(rb, k0, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, sp.x, xbase, xt, j0, r, k0, k, V, P, vec.x); });
        if (k0 == 0 && tid < 3 * TM) {
            const int t = tid & (TM - 1), q = (tid < TM ? i0 : j0) + t;
            const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
            rc = q < V ? (tid < 2 * TM ? sp.cum : sp.dtf)[o + q] : 0.f;
            rf = i0 > j0 ? sp.cum[o + i0 - 1] : 0.f;
        }
    };
    f32x16 t = zero_acc();
    load(0);
    for (int s = 0; s < hps * KS; ++s) {
        const int hh = s / KS, ks = s % KS, buf = s & 1, hb = hh & 1;
        tile_store<true>(ra, L.t.a[buf], 0, NoWeight{});
        tile_store<true>(rb, L.t.b[buf], 0, NoWeight{});
        // off the diagonal the decay is a row factor times a column factor, split at the token in front of the rows
        if (ks == 0 && i0 > j0 && tid < 2 * TM) rc = decay(tid < TM ? rc - rf : rf - rc);
        if (ks == 0 && tid < 3 * TM) (tid < TM ? L.hd.row[hb] : (tid < 2 * TM ? L.hd.col[hb] : L.hd.dcol[hb]))[tid & (TM - 1)] = rc;
        __syncthreads();
        if (s + 1 < hps * KS) load(s + 1);
        tile_mma(t, L.t.a[buf], L.t.b[buf]);
        if (ks == KS - 1) {
            const float cj = L.hd.col[hb][col], dj = L.hd.dcol[hb][col], fj = cj * dj;
            float cs = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = tile_row(r), i = i0 + row;
                const float f = i0 > j0 ? L.hd.row[hb][row] * fj : decay(L.hd.row[hb][row] - cj) * dj;
                t[r] = (i < V && j <= i) ? t[r] * f : 0.f;
                tot[r] += t[r];
                t[r] *= gv[r];
                cs += t[r];
            }
            const int w = tid >> 6, h = h0 + hh;
            const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
            cs += __shfl_xor(cs, 32, 64);
            if (lane < 32 && j < V) sp.ecol[(2 * I + (w >> 1)) * sp.tok_stride + cbase + j] = cs;
            const float rs = row_sums(t, lane);
            if ((lane & 1) == 0) {
                const int i = i0 + tile_row((lane & 31) >> 1);
                if (i < V) sp.erow[(2 * pair + (w & 1)) * sp.tok_stride + cbase + i] = rs;
            }
            t = zero_acc();
        }
    }
    float* out = sp.dG + ((((int64_t)b * sp.nc + c) * sp.G + g) * ns + slice) * Q * Q;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + tile_row(r);
        if (i < V && j < V) out[(int64_t)i * Q + j] = tot[r];
    }
}

// One 64 x 64 tile of the head sums of a slice, with the per-token dot products through the boundary states:
//   role 0: part[i][n] = sum_h exp(cum_i) (dY_i . Hprev[:, n]),            gterm_i = exp(cum_i) dY_i . (Hprev C_i)
//   role 1: part[j][n] = sum_h exp(T - cum_j) dt_j (x_j . dHnext[:, n]),   sterm_j = exp(T - cum_j) dt_j x_j . (dHnext B_j)
template <typename T>
__device__ __forceinline__ void walk_part(const SegParams& sp, const Vec& vec, WalkLds& L, int z) {
    const int Q = sp.Q, N = sp.N, P = sp.P, NT = (Q + TM - 1) / TM, NN = (N + TM - 1) / TM;
    const int r0 = (z % NT) * TM;
    z /= NT;
    const int n0 = (z % NN) * TM;
    z /= NN;
    const int role = z & 1;
    z >>= 1;
    const int ns = sp.part_split, slice = z % ns;
    z /= ns;
    const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc), V = chunk_rows(sp, c, Q);
    if (r0 >= V) return;
    const int hps = sp.hpg / ns, h0 = g * sp.hpg + slice * hps, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t xt = (int64_t)sp.H * P;
    // The products come out with a lane per token and the columns n along the registers: a token's weight is one factor
    // after the product, and its dot product stays inside the lane.
    const int i = r0 + tile_col(), il = i < V ? i : V - 1;
    float cf[16];  // C_i[n] (role 1: B_j[n])
    {
        const int64_t o = (int64_t)b * sp.bcs_b + (((int64_t)c * Q + il) * sp.G + g) * N;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int n = n0 + tile_row(r);
            cf[r] = n < N ? IO<T>::ld(role ? sp.Bm : sp.Cm, o + n) : 0.f;
        }
    }
    const int KS = (P + TK - 1) / TK;
    float ra[2][4], rb[2][4], rc = 0.f, rd = 0.f, rT = 0.f;
    auto load = [&](int s) {  // with the first step of a head, its cum and dt
        const int h = h0 + s / KS, k0 = (s % KS) * TK;
        const int64_t xbase = (int64_t)b * (role ? sp.xs_b : sp.dys_b) + ((int64_t)c * Q * sp.H + h) * P;
        const float* S = role ? sp.dstates + (((int64_t)b * sp.nc + c) * sp.H + h) * P * N : sp.states + (((int64_t)b * (sp.nc + 1) + c) * sp.H + h) * P * N;
        tile_load<true>(ra, k0, [&](float (&v)[4], int r, int k, int k0) { ld_k4<T>(v, role ? sp.x : sp.dy, xbase, xt, r0, r, k0, k, V, P, vec.x); });
        tile_load<false>(rb, k0, [&](float (&v)[4], int r, int k, int k0) { ld_r4<float>(v, S, n0, N, r, k0, k, N - n0, P); });
        if (k0 == 0) {
            const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
            rc = sp.cum[o + il];
            rd = sp.dtf[o + il];
            rT = sp.cum[o + Q - 1];
        }
    };
    f32x16 tot = zero_acc(), d = zero_acc();
    float wgt = 0.f;
    load(0);
    for (int s = 0; s < hps * KS; ++s) {
        const int hh = s / KS, ks = s % KS, buf = s & 1;
        if (ks == 0) wgt = role ? decay(rT - rc) * rd : expf(rc);
        tile_store<true>(ra, L.t.a[buf], 0, NoWeight{});
        tile_store<false>(rb, L.t.b[buf], 0, NoWeight{});
        __syncthreads();
        if (s + 1 < hps * KS) load(s + 1);
        tile_mma(d, L.t.b[buf], L.t.a[buf]);
        if (ks == KS - 1) {
            float d0 = 0.f, d1 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                tot[r] = fmaf(d[r], wgt, tot[r]);
                tot[r + 1] = fmaf(d[r + 1], wgt, tot[r + 1]);
                d0 = fmaf(d[r], cf[r], d0);
                d1 = fmaf(d[r + 1], cf[r + 1], d1);
            }
            d0 += d1;
            d0 += __shfl_xor(d0, 32, 64);
            if (lane < 32 && i < V)
                (role ? sp.sterm : sp.gterm)[(2 * (n0 / TM) + (w >> 1)) * sp.tok_stride + (((int64_t)b * sp.H + h0 + hh) * sp.nc + c) * Q + i] = d0 * wgt;
            d = zero_acc();
        }
    }
    if (i >= V) return;
    float* out = sp.dbc_part + (((((int64_t)b * sp.nc + c) * sp.G + g) * ns + slice) * 2 + role) * ((int64_t)Q * N) + (int64_t)i * N;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = n0 + tile_row(4 * q);
        if ((N & 3) == 0) {
            if (n < N) *(float4*)(out + n) = make_float4(tot[4 * q], tot[4 * q + 1], tot[4 * q + 2], tot[4 * q + 3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) out[n + e] = tot[4 * q + e];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(NTHREADS, 3) void k_bwd_walk(SegParams sp, Vec vec, int n_part, int n_dg) {
    WalkLds& L = *(WalkLds*)dyn_lds;
    const int z = blockIdx.x;  // the workgroups that walk several heads first
    if (z < n_part) walk_part<T>(sp, vec, L, z);
    else if (z < n_part + n_dg) walk_dg<T>(sp, vec, L, z - n_part);
    else walk_u<T>(sp, vec, L, z - n_part - n_dg);
}

// ---------------------------------------------------------------------------------------------
// Step 4 backward, one launch: 64 x 64 tiles of dC (role 0) / dB (role 1) from the slices' partial sums (see the
// formulas at the top of the file), and per (chunk, head) ddt with the chunk's dA / dD partial sums.
__device__ __forceinline__ void add_slices(float (&v)[4], const float (&q)[SLICES][4], int n) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = q[0][e];
#pragma unroll
        for (int s = 1; s < SLICES; ++s) v[e] += s < n ? q[s][e] : 0.f;
    }
}

template <typename T>
__global__ __launch_bounds__(NTHREADS) void k_bwd_final(SegParams sp, Vec vec, int n_dbc) {
    __shared__ __attribute__((aligned(16))) Tiles L;
    __shared__ DdtLds D;
    const int Q = sp.Q, N = sp.N;
    int z = blockIdx.x;
    if (z >= n_dbc) {
        z -= n_dbc;
        const int h = z % sp.H, c = (z / sp.H) % sp.nc, b = z / (sp.H * sp.nc);
        const int n32 = 2 * ((N + TM - 1) / TM), p32 = 2 * ((sp.P + TM - 1) / TM);
        ddt_finalize_body<4>(
            sp, &D, c, h, b,
            [&](int64_t o, int i) {
                const int64_t ts = sp.tok_stride;
                const int own = 2 * (i / TM);  // tiles right of (above) a token's own 64 x 64 tile do not exist
                const int live = 2 * ((chunk_rows(sp, c, Q) + TM - 1) / TM);
                // everything that chunks of 256 tokens and states of 128 leave is asked for at once
                DdtIn v = {0.f, 0.f, sp.fterm[o] + sp.fterm[ts + o], sp.dDrow[o] + sp.dDrow[ts + o]};
                for (int k = 2; k < p32; ++k) {
                    v.f += sp.fterm[k * ts + o];
                    v.d += sp.dDrow[k * ts + o];
                }
                float rs = 0.f, cs = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v.g += k < n32 ? sp.gterm[k * ts + o] : 0.f;
                    v.s += k < n32 ? sp.sterm[k * ts + o] : 0.f;
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    rs += k < own + 2 ? sp.erow[k * ts + o] : 0.f;
                    cs += k >= own && k < live ? sp.ecol[k * ts + o] : 0.f;
                }
                for (int k = 4; k < n32; ++k) {
                    v.g += sp.gterm[k * ts + o];
                    v.s += sp.sterm[k * ts + o];
                }
                for (int k = 8; k < live; ++k) {
                    rs += k < own + 2 ? sp.erow[k * ts + o] : 0.f;
                    cs += k >= own ? sp.ecol[k * ts + o] : 0.f;
                }
                v.g += rs - cs;
                return v;
            },
            [&](int64_t idx, float v) { IO<T>::st(sp.ddt, idx, v); });
        return;
    }
    const int NT = (Q + TM - 1) / TM, NN = (N + TM - 1) / TM;
    const int r0 = (z % NT) * TM;
    z /= NT;
    const int n0 = (z % NN) * TM;
    z /= NN;
    const int role = z & 1;
    z >>= 1;
    const int g = z % sp.G, c = (z / sp.G) % sp.nc, b = z / (sp.G * sp.nc), V = chunk_rows(sp, c, Q);
    if (r0 >= V) return;
    const int64_t bcg = ((int64_t)b * sp.nc + c) * sp.G + g, QQ = (int64_t)Q * Q;
    const int dns = sp.dg_split, pns = sp.part_split;
    const float* dG = sp.dG + bcg * dns * QQ;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
    int buf = 0;
    f32x16 acc;
    const int n = n0 + tile_col();
    {   // start from the slices' head sums: their loads and the first tiles' are one round trip
        const float* part = sp.dbc_part + (bcg * pns * 2 + role) * ((int64_t)Q * N);
        float pv[SLICES][16];
#pragma unroll
        for (int s = 0; s < SLICES; ++s)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = r0 + tile_row(r);
                pv[s][r] = (s < pns && i < V && n < N) ? part[(int64_t)s * 2 * Q * N + (int64_t)i * N + n] : 0.f;
            }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[r] = pv[0][r];
#pragma unroll
            for (int s = 1; s < SLICES; ++s) acc[r] += pv[s][r];
        }
    }
    if (role == 0) {
        const int kend = r0 + TM < V ? r0 + TM : V;
        tile_gemm<true, false>(
            acc, 0, kend,
            [&](float (&v)[4], int r, int k, int k0) {
                float q[SLICES][4];
#pragma unroll
                for (int s = 0; s < SLICES; ++s)
                    ld_k4<float>(q[s], dG, s < dns ? s * QQ : 0, Q, r0, r, k0, k, V, V, (Q & 3) == 0 && (V & 3) == 0);
                add_slices(v, q, dns);
            },
            [&](float (&v)[4], int r, int k) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e > r0 + r) v[e] = 0.f;
            },
            [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, sp.Bm, bbase + n0, bt, r, k0, k, N - n0, V); }, NoWeight{}, L, buf);
    } else {
        tile_gemm<false, false>(
            acc, r0, V,
            [&](float (&v)[4], int r, int k, int k0) {
                float q[SLICES][4];
#pragma unroll
                for (int s = 0; s < SLICES; ++s) ld_r4<float>(q[s], dG, (s < dns ? s * QQ : 0) + r0, Q, r, k0, k, V - r0, V);
                add_slices(v, q, dns);
            },
            [&](float (&v)[4], int r, int k) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < r0 + r) v[e] = 0.f;
            },
            [&](float (&v)[4], int r, int k, int k0) { ld_r4<T>(v, sp.Cm, bbase + n0, bt, r, k0, k, N - n0, V); }, NoWeight{}, L, buf);
    }
    void* out = role == 0 ? sp.dC : sp.dB;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = r0 + tile_row(r);
        if (i < V && n < N) IO<T>::st(out, bbase + (int64_t)i * bt + n, acc[r]);
    }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// 16-byte (fp32) / 8-byte (bf16) loads along P and N: sizes and every pointer and stride multiples of four elements
template <typename T>
Vec vec_of(const SegParams& sp) {
    const uintptr_t m = 4 * sizeof(T) - 1;
    Vec v;
    v.x = sp.P % 4 == 0 && (((uintptr_t)sp.x | (uintptr_t)sp.dy) & m) == 0 && (sp.xs_b | sp.dys_b) % 4 == 0;
    v.bc = sp.N % 4 == 0 && (((uintptr_t)sp.Bm | (uintptr_t)sp.Cm) & m) == 0 && sp.bcs_b % 4 == 0;
    return v;
}

template <typename T>
hipError_t scores_states(const SegParams& sp, int nroles, hipStream_t st) {
    const int NT = cdiv(sp.Q, TM);
    const int n_cb = sp.Bt * sp.nc * sp.G * (NT * (NT + 1) / 2);
    const int n_st = sp.Bt * sp.nc * sp.H * nroles * cdiv(sp.N, TM) * cdiv(sp.P, TM);
    if (sp.raw.dt) SSDK_LAUNCH_LDS(K_CHUNK_STATE, st, (k_scores_states<T, true>), dim3(n_cb + n_st), dim3(NTHREADS), lds_bytes(sp.Q + NTHREADS / 64), sp, vec_of<T>(sp), n_cb, nroles);
    else SSDK_LAUNCH_LDS(K_CHUNK_STATE, st, (k_scores_states<T, false>), dim3(n_cb + n_st), dim3(NTHREADS), lds_bytes(sp.Q + NTHREADS / 64), sp, vec_of<T>(sp), n_cb, nroles);
    return hipSuccess;
}

template <typename T>
hipError_t fwd_segment(const SegParams& sp, bool need_y, hipStream_t st) {
    if (!need_y) return hipSuccess;  // the backward pass restores the states inside its own launches
    const hipError_t e = scores_states<T>(sp, 1, st);
    if (e != hipSuccess) return e;
    SSDK_LAUNCH(K_SCAN_FWD, st, k_state_scan<false>, dim3(cdiv(sp.P * sp.N, NTHREADS), sp.H, sp.Bt), dim3(NTHREADS), sp);
    SSDK_LAUNCH_LDS(K_CHUNK_OUT, st, k_chunk_out<T>, dim3(sp.Bt * sp.nc * sp.H, cdiv(sp.P, TM), cdiv(sp.Q, TM)), dim3(NTHREADS), lds_bytes(2 * sp.Q + 2 * TM), sp, vec_of<T>(sp));
    return hipSuccess;
}

template <typename T>
hipError_t bwd_segment(const SegParams& sp0, hipStream_t st) {
    SegParams sp = sp0;
    sp.nslice = cdiv(sp.P * sp.N, NTHREADS) * (NTHREADS / 64);  // partial sums written by k_state_scan: one per wave
    const int NT = cdiv(sp.Q, TM), NN = cdiv(sp.N, TM), bcg = sp.Bt * sp.nc * sp.G;
    const hipError_t e = scores_states<T>(sp, 2, st);
    if (e != hipSuccess) return e;
    SSDK_LAUNCH(K_SCAN_BWD, st, k_state_scan<true>, dim3(cdiv(sp.P * sp.N, NTHREADS), sp.H, sp.Bt), dim3(NTHREADS), sp);
    const int n_part = bcg * sp.part_split * 2 * NN * NT, n_dg = bcg * sp.dg_split * (NT * (NT + 1) / 2), n_u = sp.Bt * sp.nc * sp.H * NT * cdiv(sp.P, TM);
    const int per_token = 2 * sp.Q + 2 * TM > 6 * TM ? 2 * sp.Q + 2 * TM : 6 * TM;
    SSDK_LAUNCH_LDS(K_BWD_MAIN, st, k_bwd_walk<T>, dim3(n_part + n_dg + n_u), dim3(NTHREADS), lds_bytes(per_token), sp, vec_of<T>(sp), n_part, n_dg);
    const int n_dbc = bcg * 2 * NN * NT;
    SSDK_LAUNCH(K_DBC, st, k_bwd_final<T>, dim3(n_dbc + sp.Bt * sp.nc * sp.H), dim3(NTHREADS), sp, vec_of<T>(sp), n_dbc);
    return hipSuccess;
}

}  // namespace

hipError_t launch_fill_zero(float* p, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const size_t blocks = (n + 255) / 256;
    SSDK_LAUNCH(K_FILL, st, k_fill_zero, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), p, n);
    return hipSuccess;
}

hipError_t launch_copy_f32(float* dst, const float* src, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const size_t blocks = (n + 255) / 256;
    SSDK_LAUNCH(K_COPY, st, k_copy_f32, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), dst, src, n);
    return hipSuccess;
}

hipError_t generic_forward_segment(const SegParams& sp, bool is_bf16, bool need_y, hipStream_t st) {
    return is_bf16 ? fwd_segment<bf16_t>(sp, need_y, st) : fwd_segment<float>(sp, need_y, st);
}

hipError_t generic_backward_segment(const SegParams& sp, bool is_bf16, hipStream_t st) {
    return is_bf16 ? bwd_segment<bf16_t>(sp, st) : bwd_segment<float>(sp, st);
}

}  // namespace ssdk
