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
// buffers (one barrier a step) with two steps of global loads in flight, 16 bytes a lane (chain()).  The weights
// (decays, dt, masks) are applied between the load and the LDS store.  Sums over the heads of a group are cut into head
// slices so that a sequence of a few chunks still fills the machine.  1999 tokens of 24 heads in two segments, forward +
// backward: 1340 us with FMA tiles, serial heads and launches of their own for every segment, 229 with tiles loaded element by
// element across the contraction and row sums by lane shuffles, 170 now: 28 + 11.5 + 16 of them are the MFMAs of the walk, the
// output and the states at their rate, beside as many vector instructions.  Small problems are bound by launches and what a
// kernel's first loads take: three forward, four backward (512 tokens of 4 heads in two segments: 216 us with 14 for each segment,
// 62 before, 46 now).
#include <numeric>
#include <type_traits>

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
};
template <>
struct IO<bf16_t> {
    static __device__ __forceinline__ float ld(const void* p, size_t i) { return bf16_to_float(((const bf16_t*)p)[i]); }
    static __device__ __forceinline__ float round(float v) { return bf16_to_float(float_to_bf16(v)); }
    static __device__ __forceinline__ void st(void* p, int64_t i, float v) { ((bf16_t*)p)[i] = float_to_bf16(v); }
};

typedef float f32x16 __attribute__((ext_vector_type(16)));

// exp of a difference of sums of dt A: at most 0 but for rounding.  A NaN stays one (fminf would take the number).
__device__ __forceinline__ float decay(float v) { return expf(v > 0.f ? 0.f : v); }

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NTHREADS = 256;
constexpr int TM = 64;   // tile edge
constexpr int TK = 32;   // contraction step
constexpr int QMAX = 1024;
constexpr int SLICES = GENERIC_SLICES;
static_assert(SLICES == 4, "the sums over slices are written out");

// An operand of a contraction step in LDS, laid out as it lies in memory: [64 rows][32 k] where k is contiguous there (KC),
// else [32 k][64 rows].  The pitches keep 16-byte rows aligned and the reads of a half wave in distinct banks, and both come to
// the same size, so that a buffer serves either.
constexpr int KPITCH = 36, RPITCH = 72, OPERAND = TM * KPITCH;
static_assert(OPERAND == TK * RPITCH, "one buffer");

struct Tiles {
    float a[2][OPERAND], b[2][OPERAND];
};
// LDS of the kernels that also keep per-token arrays of the chunk: the tiles, then `n` floats (sized at launch, so that
// four workgroups fit a compute unit up to chunks of 256 tokens).
inline size_t lds_bytes(int n) { return sizeof(Tiles) + (size_t)n * sizeof(float); }
// Tokens of a chunk's tiles: what an array needs that is read for whole tiles, rows that do not exist included.
__host__ __device__ __forceinline__ int whole_tiles(int Q) { return (Q + TM - 1) / TM * TM; }
extern __shared__ __attribute__((aligned(16))) char dyn_lds[];

// The part of a matrix that a contraction step takes, from its first element on: `outer` rows `stride` bytes apart (rows of a
// k-contiguous operand, else k), `inner` contiguous elements of each.  A buffer descriptor, wave-uniform: whatever lies outside
// reads as zero, without branches or clamped indices, so that a step's loads leave together.  (64 rows of 65535 heads of 256
// channels of fp32 stay below 4 GB.)
struct Part {
    const void* p;
    uint32_t stride;
    int outer, inner;
};
template <typename T>
__device__ __forceinline__ Part part_of(const void* p, int64_t first, int64_t stride, int outer, int inner) {
    return {(const T*)p + first, (uint32_t)stride * (uint32_t)sizeof(T), outer, inner};
}
// (By value: a cast of a vector's element in place reads the vector's first.)
__device__ __forceinline__ uint32_t bits_of(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float float_of(uint32_t v) { return __builtin_bit_cast(float, v); }
// Four elements as they come from memory: fp32, or bf16 in two registers (not SINGLE) or in the low halves of four.  Nothing is done to
// them before they are put down: that would wait for them.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// How they are asked for.  ALIGNED: `inner` and the elements in front of every row are multiples of four.  SHIFTED: any multiples of four bytes,
// all that a load of several words asks for, in rows of four elements at least; four that would reach beyond the end of their row
// are the row's last four, and move up on their way to LDS.  SINGLE: element by element, four times as many instructions and requests.
enum Loads { ALIGNED, SHIFTED, SINGLE };
template <typename T, Loads M>
__device__ __forceinline__ u32x4 fetch4(__amdgpu_buffer_rsrc_t r, uint32_t bytes, uint32_t row, int lo, int inner) {
    u32x4 v;
    if constexpr (M != SINGLE) {
        const int at = M == SHIFTED && lo > inner - 4 ? inner - 4 : lo;
        const uint32_t o = lo < inner ? row + (uint32_t)at * (uint32_t)sizeof(T) : bytes;
        if constexpr (sizeof(T) == 4) {
            v = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
        } else {
            const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
            v[0] = q[0];
            v[1] = q[1];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t o = lo + e < inner ? row + (uint32_t)(lo + e) * (uint32_t)sizeof(T) : bytes;
            if constexpr (sizeof(T) == 4) v[e] = __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
            else v[e] = __builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0);
        }
    }
    return v;
}
template <typename T, Loads M>
__device__ __forceinline__ f32x4 unpack(const u32x4& v) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(f32x4, v);
    else if constexpr (M != SINGLE) return f32x4{float_of(v[0] << 16), float_of(v[0] & 0xffff0000u), float_of(v[1] << 16), float_of(v[1] & 0xffff0000u)};
    else return f32x4{float_of(v[0] << 16), float_of(v[1] << 16), float_of(v[2] << 16), float_of(v[3] << 16)};
}
// Elements lo .. lo + 3 from the last four of a row of `inner` (beyond its end: all of them are zero already).
__device__ __forceinline__ f32x4 moved_up(f32x4 v, int lo, int inner) {
    const int by = lo + 4 - inner;
    const bool two = by > 0 && (by & 2), one = by > 0 && (by & 1);
    v = f32x4{two ? v[2] : v[0], two ? v[3] : v[1], two ? 0.f : v[2], two ? 0.f : v[3]};
    return f32x4{one ? v[1] : v[0], one ? v[2] : v[1], one ? v[3] : v[2], one ? 0.f : v[3]};
}

// A value (the thread index) that the optimiser cannot see through: what is derived from it is formed anew in every turn of a loop
// instead of being kept in registers across it (half of the walks' registers otherwise).
__device__ __forceinline__ int opaque(int t) {
    asm volatile("" : "+v"(t));
    return t;
}

// Where a thread's two pieces of four elements lie: row hi of 32, elements lo .. lo + 3, and 32 rows (k-contiguous operand) or 32
// elements further on.
__device__ __forceinline__ int piece_hi(int tid) { return tid >> 3; }
__device__ __forceinline__ int piece_lo(int tid) { return (tid & 7) * 4; }

// (kc as an argument, not a template one: where the products of a chain differ in it, the loads stay outside of branches.)
template <typename T, Loads M>
__device__ __forceinline__ void fetch(u32x4 (&r)[2], bool kc, const Part& s, bool live) {
    const int tid = opaque(threadIdx.x), lo = piece_lo(tid);
    // the last elements of a row that is longer than four: its last four begin in front of the part
    const uint32_t back = M == SHIFTED && s.inner < 4 ? 4 * (uint32_t)sizeof(T) : 0u;
    const uint32_t row = (uint32_t)piece_hi(tid) * s.stride + back, bytes = live ? (uint32_t)s.outer * s.stride + back : 0u;
    // uniform by construction; said again, or a part that the compiler has in vector registers makes it loop over the lanes' values
    const uint64_t p = (uint64_t)s.p - back;
    const uint32_t a0 = __builtin_amdgcn_readfirstlane((uint32_t)p), a1 = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)a1 << 32 | a0), 0, bytes, 0x00020000);
    r[0] = fetch4<T, M>(rs, bytes, row, lo, s.inner);
    r[1] = fetch4<T, M>(rs, bytes, row + (kc ? 32u * s.stride : 0u), lo + (kc ? 0 : 32), s.inner);
}
// wt(v, hi, lo, piece) weights a piece in place on its way to LDS.  `inner`: the part's.
template <typename T, Loads M, class W>
__device__ __forceinline__ void put(const u32x4 (&r)[2], bool kc, float* L, int inner, W wt) {
    const int tid = opaque(threadIdx.x), hi = piece_hi(tid), lo = piece_lo(tid);
    const bool shifted = M == SHIFTED && inner < (kc ? 32 : 64);  // uniform
    float* at = L + hi * (kc ? KPITCH : RPITCH) + lo;
    f32x4 v = unpack<T, M>(r[0]);
    if (shifted) v = moved_up(v, lo, inner);
    wt(v, hi, lo, 0);
    *(f32x4*)at = v;
    v = unpack<T, M>(r[1]);
    if (shifted) v = moved_up(v, lo + (kc ? 0 : 32), inner);
    wt(v, hi, lo, 1);
    *(f32x4*)(at + (kc ? 32 * KPITCH : 32)) = v;
}
// Four consecutive values of a per-token array in LDS, from a multiple of four on.
__device__ __forceinline__ f32x4 ld4(const float* p) { return *(const f32x4*)p; }
struct NoWeight {
    __device__ __forceinline__ void operator()(f32x4&, int, int, int) const {}
};

// acc += the wave's 32 x 32 quadrant of a 64 x 32 by 32 x 64 product (rows 32 (w / 2) .. of A, columns 32 (w % 2) .. of B).  Lane
// half h takes k = 8 j + 4 h .. + 3 of each row; the e-th MFMA contracts k = 8 j + e and 8 j + 4 + e.
template <bool KC>
__device__ __forceinline__ f32x4 operand4(const float* L, int row, int k) {
    if (KC) return *(const f32x4*)(L + row * KPITCH + k);
    const float* p = L + k * RPITCH + row;
    return f32x4{p[0], p[RPITCH], p[2 * RPITCH], p[3 * RPITCH]};
}
template <bool AKC, bool BKC>
__device__ __forceinline__ void tile_mma(f32x16& acc, const float* A, const float* B) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5;
    const int ra = 32 * (w >> 1) + (lane & 31), rb = 32 * (w & 1) + (lane & 31);
#pragma unroll
    for (int j = 0; j < TK / 8; ++j) {
        const f32x4 a = operand4<AKC>(A, ra, 8 * j + 4 * half), b = operand4<BKC>(B, rb, 8 * j + 4 * half);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
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

// A chain of contraction steps: load(stage, s, live) asks for step s, put(stage, s, la, lb) weights it and leaves it in LDS,
// use(s, la, lb) contracts it.  AHEAD steps are on their way from memory while one is contracted, and a tile's products -- through
// the state, with other tokens, on the diagonal -- are one chain, so that it fills once.  A step beyond the end is asked for like the
// others, with live = false: nothing is fetched, but the count of loads in flight stays known, where a branch around them would have
// every step wait for all of them.  (Two steps in flight as it seemed, with such branches, and a chain for each product, k_chunk_out
// took 35.7 us of 1999 tokens of 24 heads and the backward walk 110: now 30 and 78, of which their MFMAs alone are 11.5 and 28.  Three
// steps in flight are no faster, and the longer code costs small problems 2 us of 10.)
// Two LDS buffers: one barrier a step.  between() runs once the first loads are under way: what fills the arrays the weights are
// read from (its barriers included) costs no round trip to memory of its own.
template <int AHEAD, class Stage, class LD, class PUT, class USE, class FB>
__device__ __forceinline__ void chain(int steps, Tiles& L, LD load, PUT put_, USE use, FB between) {
    Stage R[AHEAD];
    int buf = 0;
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) load(R[a], a, a < steps);
    between();
    auto step = [&](int a, int s) {
        put_(R[a], s, L.a[buf], L.b[buf]);
        __syncthreads();
        load(R[a], s + AHEAD, s + AHEAD < steps);
        use(s, L.a[buf], L.b[buf]);
        buf ^= 1;
    };
    int s0 = 0;
    for (; s0 + AHEAD <= steps; s0 += AHEAD) {  // no way out in the middle: the same for the count of loads
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) step(a, s0 + a);
    }
#pragma unroll
    for (int a = 0; a < AHEAD - 1; ++a)
        if (s0 + a < steps) step(a, s0 + a);
}
struct Staged {
    u32x4 a[2], b[2];
};
__device__ __forceinline__ int least(int a, int b) { return a < b ? a : b; }

// A lane's value of v from the lane that CTRL permutes it with.
template <int CTRL>
__device__ __forceinline__ float from_lane(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// Sum of each of the 16 registers over the 32 lanes of a half wave, by recursive halving; lane l (of the half) ends
// with the sum of register l / 2.  On the exchanges of the vector ALUs: rows of sixteen lanes swapped between two registers, then
// inside the rows (by lane shuffles through LDS it was 550 instructions, a quarter of the dG walk).
__device__ __forceinline__ float row_sums(const f32x16& v, int lane) {
    float a[8], b[4], c[2];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const u32x2 q = __builtin_amdgcn_permlane16_swap(bits_of(v[r]), bits_of(v[r + 8]), false, false);
        a[r] = float_of(q[0]) + float_of(q[1]);
    }
    const bool h8 = lane & 8, h4 = lane & 4, h2 = lane & 2;
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r] = (h8 ? a[r + 4] : a[r]) + from_lane<0x140>(h8 ? a[r] : a[r + 4]);  // row_mirror
#pragma unroll
    for (int r = 0; r < 2; ++r) c[r] = (h4 ? b[r + 2] : b[r]) + from_lane<0x141>(h4 ? b[r] : b[r + 2]);  // row_half_mirror
    const float d = (h2 ? c[1] : c[0]) + from_lane<0x4E>(h2 ? c[0] : c[1]);                              // quad_perm 2 3 0 1
    return d + from_lane<0xB1>(d);                                                                       // quad_perm 1 0 3 2
}

// Four values each of a per-row array of a tile, for this lane's accumulator registers.
__device__ __forceinline__ void rows_of(const float* L, float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 t = *(const f32x4*)(L + tile_row(4 * q));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = t[e];
    }
}
__device__ __forceinline__ void scale_rows(f32x16& acc, const float* L) {
    float f[16];
    rows_of(L, f);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] *= f[r];
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

// Workgroups are dealt to the eight XCDs in turn, and each XCD has a cache (4 MB) of its own.  The work of a launch is listed chunk by
// chunk (and slice of heads by slice), and every XCD takes a contiguous part of the list: what works on the same rows, scores and
// states finds them in one cache.
__device__ __forceinline__ int xcd_order(int id, int n) {
    const int q = n >> 3;
    return id < 8 * q ? (id & 7) * q + (id >> 3) : id;
}

// (batch, chunk, workgroup of the chunk) from a place in the list.  Divisions that do not wait for one another.
struct Place {
    int b, c, z;
};
__device__ __forceinline__ Place place(int id, int per, int nc) {
    const uint32_t u = id, q = u / (uint32_t)per, b = u / ((uint32_t)per * (uint32_t)nc);
    return {(int)b, (int)(q - b * nc), (int)(u - q * per)};
}

// ---------------------------------------------------------------------------------------------
// Step 1, one launch: the scores and the chunk states (backward: and the local state adjoints).
// Of a chunk's workgroups the first each do one 64 x 64 tile of  Gm[b,c,g,i,j] = C_i . B_j  on or below the diagonal; the
// others one 64 x 64 tile of
//   role 0: states[b,c,h,p,n]  = sum_j exp(T - cum_j) dt_j x_j[p] B_j[n]
//   role 1: dstates[b,c,h,p,n] = sum_i exp(cum_i) dY_i[p] C_i[n]
// after forming cum (the chunk-local inclusive cumsum of dt A) of their head for themselves; the workgroup of tile
// (0, 0) of role 0 stores cum and dt for the steps that follow.
// RAW: dt as it leaves a projection.  A template argument: as a branch it took 0.5 us of the 8.4 and 26.6 that the kernel
// takes of 512 and 2048 tokens (fp32, 8 and 24 heads).
template <typename T, bool RAW, Loads LT, Loads LF>
__global__ __launch_bounds__(NTHREADS, 4) void k_scores_states(SegParams sp, int nroles) {
    Tiles& L = *(Tiles*)dyn_lds;
    float* red = (float*)(dyn_lds + sizeof(Tiles));  // [4], then the tokens' weights [Q]
    float* wt = red + NTHREADS / 64;
    const int Q = sp.Q, N = sp.N, P = sp.P;
    const int64_t bt = (int64_t)sp.G * N;
    const int NT = (Q + TM - 1) / TM, npair = NT * (NT + 1) / 2, NP = (P + TM - 1) / TM, NN = (N + TM - 1) / TM;
    const int n_cb = sp.G * npair, per = n_cb + sp.H * nroles * NN * NP;  // of a chunk
    const Place at = place(xcd_order(blockIdx.x, gridDim.x), per, sp.nc);
    const int c = at.c, b = at.b, V = chunk_rows(sp, c, Q);
    int z = at.z;
    f32x16 acc = zero_acc();
    if (z < n_cb) {
        int pair = z % npair, I = 0;
        const int g = z / npair;
        while (pair > I) pair -= ++I;
        const int i0 = I * TM, j0 = pair * TM;
        if (i0 >= V) return;
        const int64_t base = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
        chain<2, Staged>(
            (N + TK - 1) / TK, L,
            [&](Staged& R, int s, bool live) {
                const int k0 = s * TK;
                fetch<T, LT>(R.a, true, part_of<T>(sp.Cm, base + i0 * bt + k0, bt, least(TM, V - i0), N - k0), live);
                fetch<T, LT>(R.b, true, part_of<T>(sp.Bm, base + j0 * bt + k0, bt, least(TM, V - j0), N - k0), live);
            },
            [&](const Staged& R, int s, float* la, float* lb) {
                put<T, LT>(R.a, true, la, N - s * TK, NoWeight{});
                put<T, LT>(R.b, true, lb, N - s * TK, NoWeight{});
            },
            [&](int, const float* la, const float* lb) { tile_mma<true, true>(acc, la, lb); }, [] {});
        float* out = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = i0 + tile_row(r), j = j0 + tile_col();
            if (i < Q && j < Q) out[(int64_t)i * Q + j] = acc[r];
        }
        return;
    }
    z -= n_cb;
    const int n0 = (z % NN) * TM;
    z /= NN;
    const int p0 = (z % NP) * TM;
    z /= NP;
    const int role = z % nroles, h = z / nroles, g = h / sp.hpg;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // Thread t owns the E consecutive tokens from t E on.  What they need from memory is asked for in front of everything else.
    constexpr int EM = QMAX / NTHREADS;
    const int E = (Q + NTHREADS - 1) / NTHREADS;
    float d[EM], flag[EM];
#pragma unroll
    for (int e = 0; e < EM; ++e) {
        d[e] = flag[e] = 0.f;
        if (e < E) {  // uniform
            const int i = least(tid * E + e, V - 1);
            d[e] = RAW ? IO<T>::ld(sp.raw.dt, ((int64_t)c * Q + i) * sp.raw.rs + h) : IO<T>::ld(sp.dt, (int64_t)b * sp.dts_b + ((int64_t)c * Q + i) * sp.H + h);
            if (sp.reset) flag[e] = sp.reset[(int64_t)b * sp.reset_bs + (int64_t)c * Q + i] ? RESET_LOG_DECAY : 0.f;
        }
    }
    const float A = sp.A[h], bias = RAW ? sp.raw.bias[h] : 0.f;
    auto form_cum = [&] {
        float a[EM], run = 0.f;
#pragma unroll
        for (int e = 0; e < EM; ++e) {
            const bool live = e < E && tid * E + e < V;
            if (RAW) d[e] = IO<T>::round(softplus(d[e] + bias));
            d[e] = live ? d[e] : 0.f;
            run += d[e] * A + (live ? flag[e] : 0.f);
            a[e] = run;
        }
        const float incl = wave_prefix(run);  // over the wave, then over the waves
        if (lane == 63) red[w] = incl;
        __syncthreads();
        float before = incl - run, total = 0.f;
#pragma unroll
        for (int q = 0; q < NTHREADS / 64; ++q) {
            before += q < w ? red[q] : 0.f;
            total += red[q];
        }
        const bool keep = role == 0 && n0 == 0 && p0 == 0;
        const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
#pragma unroll
        for (int e = 0; e < EM; ++e) {
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
    chain<2, Staged>(
        (V + TK - 1) / TK, L,
        [&](Staged& R, int s, bool live) {
            const int k0 = s * TK;
            fetch<T, LT>(R.a, false, part_of<T>(lhs, xbase + k0 * xt, xt, least(TK, V - k0), P - p0), live);
            fetch<T, LT>(R.b, false, part_of<T>(rhs, bbase + k0 * bt, bt, least(TK, V - k0), N - n0), live);
        },
        [&](const Staged& R, int s, float* la, float* lb) {
            put<T, LT>(R.a, false, la, P - p0, [&](f32x4& v, int hi, int, int) { v *= s * TK + hi < Q ? wt[s * TK + hi] : 0.f; });
            put<T, LT>(R.b, false, lb, N - n0, NoWeight{});
        },
        [&](int, const float* la, const float* lb) { tile_mma<false, false>(acc, la, lb); }, form_cum);
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
//
// One chain of steps: through the state, the tokens before the tile, the diagonal tile.  With the token in front of the tile as
// reference, exp(cum_i - cum_k) = exp(cum_i - ref) exp(ref - cum_k), both factors <= 1: one exp per token instead of one per score,
// the first factor scales the rows; only the diagonal tile takes an exp per score.  The state's weight exp(cum_i) is applied to the
// rows of its product.
template <typename T, Loads LT, Loads LF>
__global__ __launch_bounds__(NTHREADS, 4) void k_chunk_out(SegParams sp) {
    const int Q = sp.Q, N = sp.N, P = sp.P;
    Tiles& L = *(Tiles*)dyn_lds;
    float *rowf = (float*)(dyn_lds + sizeof(Tiles)), *rowm = rowf + TM, *colm = rowm + TK, *srow = colm + TK, *cum = srow + TM, *dtf = cum + whole_tiles(Q);
    const int NT = (Q + TM - 1) / TM, NP = (P + TM - 1) / TM;
    const Place at = place(xcd_order(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y), NP * sp.H * NT, sp.nc);
    const int c = at.c, b = at.b, V = chunk_rows(sp, c, Q);
    const uint32_t q = (uint32_t)at.z / (uint32_t)NP, it = (uint32_t)at.z / (uint32_t)(NP * sp.H);
    const int p0 = (at.z - (int)q * NP) * TM, h = (int)(q - it * sp.H), g = (uint32_t)h / (uint32_t)sp.hpg;
    const int i0 = (NT - 1 - (int)it) * TM;  // the longest rows first
    if (i0 >= V) return;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
    const int kend = i0 + TM < V ? i0 + TM : V, rows = kend - i0;
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const float* Hprev = sp.states + (((int64_t)b * (sp.nc + 1) + c) * sp.H + h) * P * N;
    const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P;
    const int64_t xbase = (int64_t)b * sp.xs_b + xrow, ybase = (int64_t)b * sp.ys_b + xrow;
    const int64_t xt = (int64_t)sp.H * P;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
    const float Dh = sp.D[h] + ((sp.flags & SSD_FLAG_RESIDUAL) ? 1.f : 0.f);
    // what the weights are made from: asked for in front of everything else
    const int tid = threadIdx.x, mine = least(tid, kend - 1), row = least(tid & (TM - 1), rows - 1);
    const float c0 = sp.cum[cbase + mine], d0 = sp.dtf[cbase + mine];
    const float ci = sp.cum[cbase + i0 + row], di = sp.dtf[cbase + i0 + row], cm = sp.cum[cbase + i0 + least(TK, rows) - 1];
    const float ref = i0 > 0 ? sp.cum[cbase + i0 - 1] : 0.f;
    const int nS = (N + TK - 1) / TK, nO = i0 / TK, nD = (rows + TK - 1) / TK;
    f32x16 acc = zero_acc(), t = zero_acc();
    chain<2, Staged>(
        nS + nO + nD, L,
        [&](Staged& R, int s, bool live) {
            const bool st = s < nS;
            const int k0 = (st ? s : s - nS) * TK;
            const Part sa = part_of<T>(sp.Cm, bbase + i0 * bt + k0, bt, rows, N - k0), ta = part_of<float>(Gm, (int64_t)i0 * Q + k0, Q, rows, Q - k0);
            const Part sb = part_of<float>(Hprev, (int64_t)p0 * N + k0, N, least(TM, P - p0), N - k0);
            const Part tb = part_of<T>(sp.x, xbase + p0 + k0 * xt, xt, least(TK, V - k0), P - p0);
            if constexpr (sizeof(T) == 4) {
                fetch<float, LF>(R.a, true, st ? sa : ta, live);
                fetch<float, LF>(R.b, st, st ? sb : tb, live);
            } else if (st) {
                fetch<T, LT>(R.a, true, sa, live);
                fetch<float, LF>(R.b, true, sb, live);
            } else {
                fetch<float, LF>(R.a, true, ta, live);
                fetch<T, LT>(R.b, false, tb, live);
            }
        },
        [&](const Staged& R, int s, float* la, float* lb) {
            if (s < nS) {
                put<T, LT>(R.a, true, la, N - s * TK, NoWeight{});
                put<float, LF>(R.b, true, lb, N - s * TK, NoWeight{});
                return;
            }
            const int k0 = (s - nS) * TK;
            put<T, LT>(R.b, false, lb, P - p0, NoWeight{});
            if (s < nS + nO) {
                put<float, LF>(R.a, true, la, Q - k0, [&](f32x4& v, int, int k, int) { v *= ld4(dtf + k0 + k); });
            } else {
                // Two steps of 32 tokens.  Of the first, the tile's upper rows take an exponential per score and the lower ones a
                // factor per row and one per token, split at the step's last token; the second is the lower rows' own.
                const int half = k0 > i0;
                put<float, LF>(R.a, true, la, Q - k0, [&](f32x4& v, int r, int k, int piece) {
                    if (piece == half) {
                        const float ci = cum[i0 + 32 * half + r];
                        const f32x4 ck = ld4(cum + k0 + k), dk = ld4(dtf + k0 + k);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float f = expf(ci - ck[e]) * dk[e];
                            v[e] = k + e <= r ? v[e] * f : 0.f;
                        }
                    } else if (piece == 1) {
                        v *= rowm[r] * *(const f32x4*)(colm + k);
                    } else {
                        v = (f32x4)(0.f);
                    }
                });
            }
        },
        [&](int s, const float* la, const float* lb) {
            if (s < nS) {
                tile_mma<true, true>(t, la, lb);
            } else {
                if (s == nS + nO && i0 > 0) scale_rows(acc, rowf);
                tile_mma<true, false>(acc, la, lb);
                if (s == nS + nO + (tid >> 7)) {  // the step whose tokens are the wave's rows, the last with a share in its sums: their x is here
                    float f[16];
                    rows_of(srow, f);
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = fmaf(Dh, lb[(tile_row(r) & (TK - 1)) * RPITCH + tile_col()], fmaf(t[r], f[r], acc[r]));
                }
            }
        },
        [&] {
            // (not needed before the second step of the chain: its barriers suffice)
            auto keep = [&](int i, float c_, float d_) {
                cum[i] = c_;
                dtf[i] = i < i0 ? decay(ref - c_) * d_ : d_;
            };
            if (tid < kend) keep(tid, c0, d0);
            for (int i = tid + NTHREADS; i < kend; i += NTHREADS) keep(i, sp.cum[cbase + i], sp.dtf[cbase + i]);
            if (tid < TM) {
                rowf[tid] = decay(ci - ref);  // rows that do not exist: those of the last one
                srow[tid] = expf(ci);
                if (tid < TK) colm[tid] = decay(cm - ci) * di;
                else rowm[tid - TK] = decay(ci - cm);
            }
        });
    const int left = opaque(V - i0), p = p0 + tile_col();
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (tile_row(r) < left && p < P) IO<T>::st(sp.y, ybase + (int64_t)(i0 + tile_row(r)) * xt + p, acc[r]);
}

// ---------------------------------------------------------------------------------------------
// Step 3 backward, one launch of three kinds of workgroups.  Sums over the tile's columns are left as partial sums per
// 32 columns (or rows) and added in a fixed order by the last step.
struct WalkLds {
    Tiles t;
    union {
        float ch[1];  // walk_u: the factors of rows and tokens [2 TM], cum [Q], dt [Q]
        struct { float row[2][TM], col[2][TM], dcol[2][TM]; } hd;
    };
};

// u rows j0.. of one (chunk, head): transposed masked scores (without dt) times dY, then the leaving-adjoint term;
// dx = dt u + D dY, and per token x . u (fterm) and dY . x (dDrow)
template <typename T, Loads LT, Loads LF>
__device__ __forceinline__ void walk_u(const SegParams& sp, WalkLds& L, int b, int c, int h, int z) {
    const int Q = sp.Q, N = sp.N, P = sp.P, NP = (P + TM - 1) / TM;
    const int p0 = (z % NP) * TM, j0 = (z / NP) * TM;  // tile 0 has the longest contraction
    const int g = h / sp.hpg, V = chunk_rows(sp, c, Q);
    if (j0 >= V) return;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
    float *rowf = L.ch, *rowm = rowf + TM, *colm = rowm + TK, *cum = colm + TK, *dtf = cum + Q;
    const float T_ = sp.cum[cbase + Q - 1];
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const float* dHnext = sp.dstates + (((int64_t)b * sp.nc + c) * sp.H + h) * P * N;
    const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P;
    const int64_t xbase = (int64_t)b * sp.xs_b + xrow, dybase = (int64_t)b * sp.dys_b + xrow, dxbase = (int64_t)b * sp.dxs_b + xrow;
    const int64_t xt = (int64_t)sp.H * P;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
    const float Dh = sp.D[h] + ((sp.flags & SSD_FLAG_RESIDUAL) ? 1.f : 0.f);
    // through the adjoint, tokens behind the tile, the diagonal tile, the decay split at the tile's last token: k_chunk_out's chain
    const int j1 = j0 + TM < V ? j0 + TM : V, rows = j1 - j0;
    // what the weights are made from: asked for in front of everything else
    const int tid = threadIdx.x, mine = least(tid, V - 1), row = least(tid & (TM - 1), rows - 1);
    const float c0 = sp.cum[cbase + mine], d0 = sp.dtf[cbase + mine];
    const float cj = sp.cum[cbase + j0 + row], cm = sp.cum[cbase + j0 + least(TK, rows) - 1], ref = sp.cum[cbase + j1 - 1];
    const int nS = (N + TK - 1) / TK, nO = (V - j1 + TK - 1) / TK, nD = (rows + TK - 1) / TK;
    const int p = p0 + tile_col();
    f32x16 acc = zero_acc();
    float xv[16], dyv[16];
    chain<2, Staged>(
        nS + nO + nD, L.t,
        [&](Staged& R, int s, bool live) {
            const bool st = s < nS;
            const int k0 = st ? s * TK : (s < nS + nO ? j1 + (s - nS) * TK : j0 + (s - nS - nO) * TK);
            const Part sa = part_of<T>(sp.Bm, bbase + j0 * bt + k0, bt, rows, N - k0), ta = part_of<float>(Gm, (int64_t)k0 * Q + j0, Q, least(TK, V - k0), Q - j0);
            const Part sb = part_of<float>(dHnext, (int64_t)p0 * N + k0, N, least(TM, P - p0), N - k0);
            const Part tb = part_of<T>(sp.dy, dybase + p0 + k0 * xt, xt, least(TK, V - k0), P - p0);
            if constexpr (sizeof(T) == 4) {
                fetch<float, LF>(R.a, st, st ? sa : ta, live);
                fetch<float, LF>(R.b, st, st ? sb : tb, live);
            } else if (st) {
                fetch<T, LT>(R.a, true, sa, live);
                fetch<float, LF>(R.b, true, sb, live);
            } else {
                fetch<float, LF>(R.a, false, ta, live);
                fetch<T, LT>(R.b, false, tb, live);
            }
        },
        [&](const Staged& R, int s, float* la, float* lb) {
            if (s < nS) {
                put<T, LT>(R.a, true, la, N - s * TK, NoWeight{});
                put<float, LF>(R.b, true, lb, N - s * TK, NoWeight{});
                return;
            }
            put<T, LT>(R.b, false, lb, P - p0, NoWeight{});
            if (s < nS + nO) {
                const int k0 = j1 + (s - nS) * TK;
                put<float, LF>(R.a, false, la, Q - j0, [&](f32x4& v, int k, int, int) { v *= k0 + k < V ? cum[k0 + k] : 0.f; });
            } else {
                // the first step is the tile's upper rows' own; of the second, the lower rows take an exponential per score, the
                // upper ones a factor per row and one per token
                const int half = s > nS + nO, k0 = j0 + half * TK;
                put<float, LF>(R.a, false, la, Q - j0, [&](f32x4& v, int k, int r, int piece) {
                    if (piece == half) {
                        const float ck = cum[least(k0 + k, V - 1)];
                        const f32x4 cj = ld4(cum + k0 + r);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float f = expf(ck - cj[e]);
                            v[e] = k >= r + e && k0 + k < V ? v[e] * f : 0.f;
                        }
                    } else if (piece == 0) {
                        v *= colm[k] * *(const f32x4*)(rowm + r);
                    } else {
                        v = (f32x4)(0.f);
                    }
                });
            }
        },
        [&](int s, const float* la, const float* lb) {
            if (s < nS) {
                tile_mma<true, true>(acc, la, lb);
            } else {
                if (s == nS) acc *= decay(T_ - ref);
                if (s == nS + nO) scale_rows(acc, rowf);
                tile_mma<false, false>(acc, la, lb);
            }
        },
        [&] {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t o = (int64_t)least(j0 + tile_row(r), V - 1) * xt + least(p, P - 1);  // clamped: no branches
                dyv[r] = IO<T>::ld(sp.dy, dybase + o);
                xv[r] = IO<T>::ld(sp.x, xbase + o);
            }
            // (not needed before the second step of the chain: its barriers suffice)
            auto keep = [&](int i, float c_, float d_) {
                cum[i] = i < j1 ? c_ : decay(c_ - ref);
                dtf[i] = d_;
            };
            if (tid < V) keep(tid, c0, d0);
            for (int i = tid + NTHREADS; i < V; i += NTHREADS) keep(i, sp.cum[cbase + i], sp.dtf[cbase + i]);
            if (tid < TM) {
                rowf[tid] = decay(ref - cj);  // rows that do not exist: those of the last one
                if (tid < TK) rowm[tid] = decay(cm - cj);
                else colm[tid - TK] = tid < rows ? decay(cj - cm) : 0.f;
            }
        });
    f32x16 dyx;
    const int left = opaque(V - j0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int j = j0 + tile_row(r);
        const bool live = tile_row(r) < left && p < P;
        if (live) IO<T>::st(sp.dx, dxbase + (int64_t)j * xt + p, dtf[j] * acc[r] + Dh * dyv[r]);
        acc[r] = live ? acc[r] * xv[r] : 0.f;
        dyx[r] = live ? dyv[r] * xv[r] : 0.f;
    }
    const int lane = tid & 63, piece = 2 * (p0 / TM) + ((tid >> 6) & 1);
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
template <typename T, Loads LT, Loads LF, bool DIAG>
__device__ __forceinline__ void walk_dg(const SegParams& sp, WalkLds& L, int b, int c, int g, int slice, int I, int J) {
    const int Q = sp.Q, P = sp.P, V = chunk_rows(sp, c, Q), ns = sp.dg_split;
    const int i0 = I * TM, j0 = J * TM;
    if (i0 >= V) return;
    const int hps = sp.hpg / ns, h0 = g * sp.hpg + slice * hps, tid = threadIdx.x, lane = tid & 63;
    const int64_t xt = (int64_t)sp.H * P;
    const float* Gm = sp.Gm + (((int64_t)b * sp.nc + c) * sp.G + g) * Q * Q;
    const int col = tile_col(), j = j0 + col;
    float gv[16];  // the tile's scores: clamped indices, no branches, and zeros where there is none
#pragma unroll
    for (int r = 0; r < 16; ++r) gv[r] = Gm[(int64_t)least(i0 + tile_row(r), V - 1) * Q + least(j, Q - 1)];
#pragma unroll
    for (int r = 0; r < 16; ++r) gv[r] = i0 + tile_row(r) < V && j <= i0 + tile_row(r) ? gv[r] : 0.f;
    f32x16 tot = zero_acc(), t = zero_acc();
    const int KS = (P + TK - 1) / TK;
    struct Stage : Staged {
        float c, f;  // the head's cum or dt, and its cum in front of the rows
    };
    int lh = 0, lk = 0, sh = 0, sk = 0, uh = 0, uk = 0;  // head of the slice and step of that head: of the next load, put and use
    auto next = [&](int& hh, int& ks) {
        if (++ks == KS) ks = 0, ++hh;
    };
    chain<2, Stage>(
        hps * KS, L.t,
        [&](Stage& R, int, bool live) {
            const int h = __builtin_amdgcn_readfirstlane(live ? h0 + lh : h0), k0 = __builtin_amdgcn_readfirstlane(lk * TK);
            const int64_t xrow = ((int64_t)c * Q * sp.H + h) * P + k0;
            fetch<T, LT>(R.a, true, part_of<T>(sp.dy, (int64_t)b * sp.dys_b + xrow + i0 * xt, xt, least(TM, V - i0), P - k0), live);
            fetch<T, LT>(R.b, true, part_of<T>(sp.x, (int64_t)b * sp.xs_b + xrow + j0 * xt, xt, least(TM, V - j0), P - k0), live);
            const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;  // (every step: see chain)
            R.c = (tid < 2 * TM ? sp.cum : sp.dtf)[o + least((tid < TM ? i0 : j0) + (tid & (TM - 1)), V - 1)];
            if (!DIAG) R.f = sp.cum[o + i0 - 1];
            next(lh, lk);
        },
        [&](Stage& R, int, float* la, float* lb) {
            put<T, LT>(R.a, true, la, P - sk * TK, NoWeight{});
            put<T, LT>(R.b, true, lb, P - sk * TK, NoWeight{});
            const int hb = sh & 1;
            if (sk == 0 && tid < 3 * TM) {
                // off the diagonal the decay is a row factor times a column factor, split at the token in front of the rows
                const float v = !DIAG && tid < 2 * TM ? decay(tid < TM ? R.c - R.f : R.f - R.c) : R.c;
                (tid < TM ? L.hd.row[hb] : (tid < 2 * TM ? L.hd.col[hb] : L.hd.dcol[hb]))[tid & (TM - 1)] = v;
            }
            next(sh, sk);
        },
        [&](int, const float* la, const float* lb) {
            tile_mma<true, true>(t, la, lb);
            const int hh = uh, hb = uh & 1;
            next(uh, uk);
            if (uk != 0) return;
            float cj = L.hd.col[hb][col];
            asm volatile("" : "+v"(cj));  // or the exponentials move up into every step
            const float dj = L.hd.dcol[hb][col], fj = cj * dj;
            float cs = 0.f;
            const int left = opaque(V - i0);  // or a mask of every register stays in scalar registers
            float f[16];
            rows_of(L.hd.row[hb], f);
            if constexpr (!DIAG) {
#pragma unroll
                for (int r = 0; r < 16; ++r) t[r] *= f[r] * fj;
                if (i0 + TM > V) {  // uniform
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] = tile_row(r) < left ? t[r] : 0.f;
                }
            } else {
                const int above = opaque(col);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool live = tile_row(r) < left && tile_row(r) >= above;
                    f[r] = decay(f[r] - cj) * dj;
                    t[r] = live ? t[r] * f[r] : 0.f;
                    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // four exponentials at a time: sixteen take the registers of a wave
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
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
                if (i < V) sp.erow[(2 * J + (w & 1)) * sp.tok_stride + cbase + i] = rs;
            }
            t = zero_acc();
        },
        [] {});
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
template <typename T, Loads LT, Loads LF>
__device__ __forceinline__ void walk_part(const SegParams& sp, WalkLds& L, int b, int c, int g, int slice, int z) {
    const int Q = sp.Q, N = sp.N, P = sp.P, NT = (Q + TM - 1) / TM, NN = (N + TM - 1) / TM, V = chunk_rows(sp, c, Q), ns = sp.part_split;
    const int r0 = (z % NT) * TM;
    z /= NT;
    const int n0 = (z % NN) * TM, role = z / NN;
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
    struct Stage : Staged {
        float c, d, T_;  // the head's cum and dt, its cum at the end
    };
    int lh = 0, lk = 0, sk = 0, uh = 0, uk = 0;  // head of the slice and step of that head: of the next load, put and use
    auto next = [&](int& hh, int& ks) {
        if (++ks == KS) ks = 0, ++hh;
    };
    f32x16 tot = zero_acc(), d = zero_acc();
    float wgt = 0.f;
    chain<2, Stage>(
        hps * KS, L.t,
        [&](Stage& R, int, bool live) {
            const int h = __builtin_amdgcn_readfirstlane(live ? h0 + lh : h0), k0 = __builtin_amdgcn_readfirstlane(lk * TK);
            const int64_t first = (int64_t)b * (role ? sp.xs_b : sp.dys_b) + (((int64_t)c * Q + r0) * sp.H + h) * P + k0;
            const float* S = role ? sp.dstates + (((int64_t)b * sp.nc + c) * sp.H + h) * P * N : sp.states + (((int64_t)b * (sp.nc + 1) + c) * sp.H + h) * P * N;
            fetch<T, LT>(R.a, true, part_of<T>(role ? sp.x : sp.dy, first, xt, least(TM, V - r0), P - k0), live);
            fetch<float, LF>(R.b, false, part_of<float>(S, (int64_t)k0 * N + n0, N, least(TK, P - k0), N - n0), live);
            const int64_t o = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;  // (every step: see chain)
            R.c = sp.cum[o + il];
            R.d = sp.dtf[o + il];
            R.T_ = sp.cum[o + Q - 1];
            next(lh, lk);
        },
        [&](Stage& R, int, float* la, float* lb) {
            if (sk == 0) wgt = role ? decay(R.T_ - R.c) * R.d : expf(R.c);
            put<T, LT>(R.a, true, la, P - sk * TK, NoWeight{});
            put<float, LF>(R.b, false, lb, N - n0, NoWeight{});
            if (++sk == KS) sk = 0;
        },
        [&](int, const float* la, const float* lb) {
            tile_mma<false, true>(d, lb, la);
            const int hh = uh;
            next(uh, uk);
            if (uk != 0) return;
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
        },
        [] {});
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

// The list: batch, chunk, group, and of the heads as many slices as the two slicings have boundaries in common.
template <typename T, Loads LT, Loads LF>
__global__ __launch_bounds__(NTHREADS, 3) void k_bwd_walk(SegParams sp, int ns) {
    WalkLds& L = *(WalkLds*)dyn_lds;
    const int NT = (sp.Q + TM - 1) / TM, NN = (sp.N + TM - 1) / TM, NP = (sp.P + TM - 1) / TM, npair = NT * (NT + 1) / 2;
    const int ps = sp.part_split / ns, ds = sp.dg_split / ns, hs = sp.hpg / ns;  // slices, and heads, of one of these
    const int w_part = 2 * NN * NT, w_u = NT * NP, n_part = ps * w_part, n_dg = ds * npair, per = n_part + n_dg + hs * w_u;
    const Place at = place(xcd_order(blockIdx.x, gridDim.x), per, ns * sp.G * sp.nc);
    const Place gs = place(at.c, ns, sp.G);  // b: chunk, c: group, z: slice
    const int b = at.b, c = gs.b, g = gs.c, s = gs.z;
    int z = at.z;
    // the workgroups that walk several heads first
    if (z < n_part) {
        walk_part<T, LT, LF>(sp, L, b, c, g, s * ps + z / w_part, z % w_part);
        return;
    }
    z -= n_part;
    if (z < n_dg) {
        int J = z % npair, I = 0;
        while (J > I) J -= ++I;
        if (I == J) walk_dg<T, LT, LF, true>(sp, L, b, c, g, s * ds + z / npair, I, J);
        else walk_dg<T, LT, LF, false>(sp, L, b, c, g, s * ds + z / npair, I, J);
        return;
    }
    z -= n_dg;
    walk_u<T, LT, LF>(sp, L, b, c, g * sp.hpg + s * hs + z % hs, z / hs);
}

// ---------------------------------------------------------------------------------------------
// Step 4 backward, one launch: 64 x 64 tiles of dC (role 0) / dB (role 1) from the slices' partial sums (see the
// formulas at the top of the file), and per (chunk, head) ddt with the chunk's dA / dD partial sums.
template <typename T, Loads LT, Loads LF>
__global__ __launch_bounds__(NTHREADS) void k_bwd_final(SegParams sp) {
    __shared__ __attribute__((aligned(16))) Tiles L;
    __shared__ DdtLds D;
    const int Q = sp.Q, N = sp.N, NT = (Q + TM - 1) / TM, NN = (N + TM - 1) / TM, n_dbc = sp.G * 2 * NN * NT, per = n_dbc + sp.H;
    const Place at = place(xcd_order(blockIdx.x, gridDim.x), per, sp.nc);
    const int c = at.c, b = at.b;
    int z = at.z;
    if (z >= n_dbc) {
        const int h = z - n_dbc;
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
    const int r0 = (z % NT) * TM;
    z /= NT;
    const int n0 = (z % NN) * TM;
    z /= NN;
    const int role = z & 1, g = z >> 1, V = chunk_rows(sp, c, Q);
    if (r0 >= V) return;
    const int64_t bcg = ((int64_t)b * sp.nc + c) * sp.G + g, QQ = (int64_t)Q * Q;
    const int dns = sp.dg_split, pns = sp.part_split;
    const float* dG = sp.dG + bcg * dns * QQ;
    const int64_t bbase = (int64_t)b * sp.bcs_b + ((int64_t)c * Q * sp.G + g) * N;
    const int64_t bt = (int64_t)sp.G * N;
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
    struct Stage {
        u32x4 a[SLICES][2], b[2];
    };
    // dG (role 0), or its transpose, with the slices added up on the way, times rows of B (role 1: C)
    auto walk = [&](auto rows_along_k, int first, int steps, const void* rhs) {
        constexpr bool KC = decltype(rows_along_k)::value;
        chain<2, Stage>(
            steps, L,
            [&](Stage& R, int s, bool live) {
                const int k0 = first + s * TK, kn = least(TK, V - k0);
#pragma unroll
                for (int q = 0; q < SLICES; ++q) {
                    const float* G = dG + (q < dns ? q * QQ : 0);
                    if (KC) fetch<float, LF>(R.a[q], true, part_of<float>(G, (int64_t)r0 * Q + k0, Q, least(TM, V - r0), Q - k0), live);
                    else fetch<float, LF>(R.a[q], false, part_of<float>(G, (int64_t)k0 * Q + r0, Q, kn, Q - r0), live);
                }
                fetch<T, LT>(R.b, false, part_of<T>(rhs, bbase + n0 + k0 * bt, bt, kn, N - n0), live);
            },
            [&](Stage& R, int s, float* la, float* lb) {
                u32x4 v[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    f32x4 t = unpack<float, LF>(R.a[0][e]);
#pragma unroll
                    for (int q = 1; q < SLICES; ++q) t += q < dns ? unpack<float, LF>(R.a[q][e]) : (f32x4)(0.f);
                    v[e] = __builtin_bit_cast(u32x4, t);
                }
                put<float, LF>(v, KC, la, KC ? Q - (first + s * TK) : Q - r0, [&](f32x4& t, int hi, int lo, int piece) {  // on or below the diagonal
                    const int k = first + s * TK, r = r0 + 32 * piece;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (KC ? k + lo + e > r + hi : k + hi < r + lo + e) t[e] = 0.f;
                });
                put<T, LT>(R.b, false, lb, N - n0, NoWeight{});
            },
            [&](int, const float* la, const float* lb) { tile_mma<KC, false>(acc, la, lb); }, [] {});
    };
    if (role == 0) walk(std::true_type{}, 0, (least(r0 + TM, V) + TK - 1) / TK, sp.Bm);
    else walk(std::false_type{}, r0, (V - r0 + TK - 1) / TK, sp.Cm);
    void* out = role == 0 ? sp.dC : sp.dB;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = r0 + tile_row(r);
        if (i < V && n < N) IO<T>::st(out, bbase + (int64_t)i * bt + n, acc[r]);
    }
}

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// How T's tensors, and the fp32 arrays of the passes before, are asked for: sizes, strides and every pointer in elements of four, or in words, or neither.
template <typename T>
bool in_units(const SegParams& sp, int unit) {  // of x, dY, B and C
    const uintptr_t m = unit * sizeof(T) - 1;
    return (sp.P | sp.N) % unit == 0 && (((uintptr_t)sp.x | (uintptr_t)sp.dy | (uintptr_t)sp.Bm | (uintptr_t)sp.Cm) & m) == 0 &&
           (sp.xs_b | sp.dys_b | sp.bcs_b) % unit == 0;
}
template <typename T, Loads LT, Loads LF>
hipError_t scores_states(const SegParams& sp, int nroles, hipStream_t st) {
    const int NT = cdiv(sp.Q, TM);
    const int n_cb = sp.Bt * sp.nc * sp.G * (NT * (NT + 1) / 2);
    const int n_st = sp.Bt * sp.nc * sp.H * nroles * cdiv(sp.N, TM) * cdiv(sp.P, TM);
    if (sp.raw.dt) SSDK_LAUNCH_LDS(K_CHUNK_STATE, st, (k_scores_states<T, true, LT, LF>), dim3(n_cb + n_st), dim3(NTHREADS), lds_bytes(sp.Q + NTHREADS / 64), sp, nroles);
    else SSDK_LAUNCH_LDS(K_CHUNK_STATE, st, (k_scores_states<T, false, LT, LF>), dim3(n_cb + n_st), dim3(NTHREADS), lds_bytes(sp.Q + NTHREADS / 64), sp, nroles);
    return hipSuccess;
}

template <typename T, Loads LT, Loads LF>
hipError_t fwd_segment(const SegParams& sp, hipStream_t st) {
    const hipError_t e = scores_states<T, LT, LF>(sp, 1, st);
    if (e != hipSuccess) return e;
    SSDK_LAUNCH(K_SCAN_FWD, st, k_state_scan<false>, dim3(cdiv(sp.P * sp.N, NTHREADS), sp.H, sp.Bt), dim3(NTHREADS), sp);
    // (two dimensions of the grid: a launch has at most 2^32 threads in one)
    SSDK_LAUNCH_LDS(K_CHUNK_OUT, st, (k_chunk_out<T, LT, LF>), dim3(sp.Bt * sp.nc * sp.H, cdiv(sp.P, TM) * cdiv(sp.Q, TM)), dim3(NTHREADS), lds_bytes(2 * whole_tiles(sp.Q) + 3 * TM), sp);
    return hipSuccess;
}

template <typename T, Loads LT, Loads LF>
hipError_t bwd_segment(const SegParams& sp0, hipStream_t st) {
    SegParams sp = sp0;
    sp.nslice = cdiv(sp.P * sp.N, NTHREADS) * (NTHREADS / 64);  // partial sums written by k_state_scan: one per wave
    const int NT = cdiv(sp.Q, TM), NN = cdiv(sp.N, TM), bcg = sp.Bt * sp.nc * sp.G;
    const hipError_t e = scores_states<T, LT, LF>(sp, 2, st);
    if (e != hipSuccess) return e;
    SSDK_LAUNCH(K_SCAN_BWD, st, k_state_scan<true>, dim3(cdiv(sp.P * sp.N, NTHREADS), sp.H, sp.Bt), dim3(NTHREADS), sp);
    const int n_part = bcg * sp.part_split * 2 * NN * NT, n_dg = bcg * sp.dg_split * (NT * (NT + 1) / 2), n_u = sp.Bt * sp.nc * sp.H * NT * cdiv(sp.P, TM);
    const int per_token = 2 * sp.Q + 2 * TM > 6 * TM ? 2 * sp.Q + 2 * TM : 6 * TM;
    SSDK_LAUNCH_LDS(K_BWD_MAIN, st, (k_bwd_walk<T, LT, LF>), dim3(n_part + n_dg + n_u), dim3(NTHREADS), lds_bytes(per_token), sp, std::gcd(sp.part_split, sp.dg_split));
    const int n_dbc = bcg * 2 * NN * NT;
    SSDK_LAUNCH(K_DBC, st, (k_bwd_final<T, LT, LF>), dim3(n_dbc + sp.Bt * sp.nc * sp.H), dim3(NTHREADS), sp);
    return hipSuccess;
}

template <typename T, Loads LT, Loads LF>
hipError_t segment(const SegParams& sp, bool bwd, hipStream_t st) {
    return bwd ? bwd_segment<T, LT, LF>(sp, st) : fwd_segment<T, LT, LF>(sp, st);
}
// ALIGNED wherever it can be: it takes no care of a row's end.  SHIFTED for all else that is whole words apart: rows of scores in chunks of any length
// (in fours with every other operand, or all of them singly: chunks of 63 / 101 / 127 tokens, fp32, 24 heads, 2000 / 2000 / 8192 tokens backward 204
// / 205 / 594 us, with each operand by a flag of its own and single loads of the scores 160 / 180 / 498, so 149 / 152 / 428), odd widths and
// addresses (256 tokens, one element off, 180 -> 130; states of 31, 101 -> 85).  bf16 at odd widths or addresses has only SINGLE loads for
// its own tensors (states of 31 103 -> 90 us, from the fp32 arrays alone); rows of one to three elements have none of four.
template <typename T>
hipError_t any_segment(const SegParams& sp, bool bwd, hipStream_t st) {
    if (sp.Q % 4 == 0 && in_units<T>(sp, 4)) return segment<T, ALIGNED, ALIGNED>(sp, bwd, st);
    if (sp.P < 4 || sp.N < 4 || sp.Q < 4) return segment<T, SINGLE, SINGLE>(sp, bwd, st);
    if (in_units<T>(sp, 4 / sizeof(T))) return segment<T, SHIFTED, SHIFTED>(sp, bwd, st);
    if constexpr (sizeof(T) == 2) return segment<T, SINGLE, SHIFTED>(sp, bwd, st);
    return segment<T, SINGLE, SINGLE>(sp, bwd, st);
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
    if (!need_y) return hipSuccess;  // the backward pass restores the states inside its own launches
    return is_bf16 ? any_segment<bf16_t>(sp, false, st) : any_segment<float>(sp, false, st);
}

hipError_t generic_backward_segment(const SegParams& sp, bool is_bf16, hipStream_t st) {
    return is_bf16 ? any_segment<bf16_t>(sp, true, st) : any_segment<float>(sp, true, st);
}

}  // namespace ssdk
