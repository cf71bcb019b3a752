// Generation: a token or a few at a time through a block (the recurrence of Sec. 3.1, Eq. 1 around which the
// block's other steps shrink to vectors).  Every kernel here is bound by reading each parameter once and the
// SSM state twice per call.  Up to two rows (a sequence on its own) the block's steps are folded into three
// launches that do exactly that, on the vector ALUs:
//   k_linear_few<1>  zxbcdt = RMSNorm(u) pre_norm_w W_in^T   (or plain u W_in^T)
//                    (one token a sequence: with the convolution step + SiLU and softplus(dt) on the finished columns)
//   k_decode_step    the state update and g = (C h + D x) silu(z)   (several tokens: k_decode_mid, convolution included)
//   k_linear_few<1>  out = RMSNorm(g) norm_w W_out^T (+ the residual)
// With more rows (several sequences generated together) the per-row arithmetic would bound the products, which then
// run as small MFMAs (k_linear_few_mfma): three launches as well.
#include "ssd_internal.h"

namespace ssdk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float sigmoid_fast(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// what storing a value in bf16 and reading it back leaves of it
__device__ __forceinline__ float through_bf16(float v) { return (float)(__bf16)v; }

// Streaming accesses: data that is gone from the last-level cache before it is read again would only push out of it what is not.
// Input product, output product and recurrence of a 2.7B block with 16 sequences, the layers whose weights do not stay in the
// cache: 17.9, 10.7, 19.1 us with plain accesses, 15.8, 10.3, 16.7 so; with one sequence 14.0, 8.6 -> 13.5, 8.5.  A template argument:
// as a branch around the loads it would end in a wait for them.
template <bool STREAM, typename V>
__device__ __forceinline__ V fetch(const V* p) {
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool STREAM, typename V>
__device__ __forceinline__ void put(V* p, V v) {
    if (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

struct FewParams {
    const __bf16 *x, *w, *res;
    __bf16* out;
    const float* in_w;
    int64_t ldx, ldo, ldres;
    int rows, K, N;
    float eps;
};

// out[r, n] = sum_k f(x)[r, k] w[n, k] (+ res[r, n]) for r < rows <= R.  MODE 0: f(x) = x.  MODE 1: f(x) = x / sqrt(mean x^2 +
// eps) * in_w; a workgroup sees whole rows, so the mean comes out of the same loop and scales the finished sums.
// Workgroup ids are dealt round-robin over the 8 XCDs: neighbouring columns, which share cache lines of everything but w,
// go to one XCD.
__device__ __forceinline__ int xcd_block() {
    const int n = gridDim.x, q = n >> 3, b = blockIdx.x;
    return b < 8 * q ? (b & 7) * q + (b >> 3) : b;
}
// The launch also moves `copy_chunks` pieces of `copy_n` 16-byte vectors from copy_src to copy_dst: a small
// state (one piece per sequence) that the kernel before this one still read in its old place.
struct FewOperands {
    const void* copy_src;
    void* copy_dst;
    int copy_n, copy_chunks;                   // vectors per chunk, chunks
    int64_t copy_src_stride, copy_dst_stride;  // vectors between chunks
    // matrix-core kernel with packed input: partial sums of squares of the rows (null: no normalisation), how many per
    // group, groups; and what it leaves for the next such product (pack_out null: nothing)
    const float* ssq;
    int nparts, groups;
    __bf16* pack_out;
    const float* pack_w;
    float* pack_ssq;
    // one token for each of several sequences (row r = sequence r): the columns [off_xbc, off_dt) of the output go through
    // the convolution step on the state cs (sequence r: cs_bs elements further on; replaced in place: a channel has one
    // owner), the H columns from off_dt on through softplus.  cs null: no such steps.
    __bf16* cs;
    int64_t cs_bs;
    const float *conv_w, *conv_b, *dt_bias;
    int off_xbc, off_dt, conv_dim;
    int ks, cols;  // waves of a workgroup, columns of one
    bool stream;  // w by streaming loads
};

// What the step of column n needs besides the product: asked for when the kernel starts, and not touched before the end
// (a conversion here would wait for it in front of the loads of w).
struct StepTaps {
    uint32_t s0, s1, s2;  // bf16 bits
    float b;
    f32x4 w;
};
__device__ __forceinline__ float bits_f(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ StepTaps step_taps(const FewOperands& fo, int r, int n) {  // no branches: clamped indices
    StepTaps t;
    const int last = fo.conv_dim - 1, c0 = n - fo.off_xbc, c = c0 < 0 ? 0 : (c0 < last ? c0 : last);
    const uint16_t* cs = (const uint16_t*)fo.cs + r * fo.cs_bs + c;
    t.s0 = cs[0];
    t.s1 = cs[fo.conv_dim];
    t.s2 = cs[2 * fo.conv_dim];
    const float* bias = n >= fo.off_dt ? fo.dt_bias + (n - fo.off_dt) : fo.conv_b + c;
    t.b = *bias;
    t.w = *(const f32x4*)(fo.conv_w + (int64_t)c * 4);
    return t;
}
// The rounded product u of (row r, column n) through its step; every intermediate is rounded as the block stores it.
__device__ __forceinline__ __bf16 step_finish(const FewOperands& fo, const StepTaps& t, int r, int n, __bf16 ub) {
    const float u = (float)ub;
    if (n >= fo.off_dt) {
        const float v = u + t.b;
        return (__bf16)(fmaxf(v, 0.f) + log1pf(__expf(-fabsf(v))));  // softplus
    }
    if (n < fo.off_xbc) return ub;
    const int c = n - fo.off_xbc;
    uint16_t* cs = (uint16_t*)fo.cs + r * fo.cs_bs + c;
    cs[0] = (uint16_t)t.s1;
    cs[fo.conv_dim] = (uint16_t)t.s2;
    cs[2 * fo.conv_dim] = __builtin_bit_cast(uint16_t, ub);
    const float pre = t.b + t.w[0] * bits_f(t.s0) + t.w[1] * bits_f(t.s1) + t.w[2] * bits_f(t.s2) + t.w[3] * u;
    return (__bf16)(pre * sigmoid_fast(pre));
}

// (The workgroup size comes as an argument: blockDim is a vector load that the whole kernel would wait for first.)
__device__ __forceinline__ void move_pieces(const FewOperands& fo, int threads) {
    const int total = fo.copy_n * fo.copy_chunks;
    for (int i = blockIdx.x * threads + threadIdx.x; i < total; i += gridDim.x * threads) {
        const int c = i / fo.copy_n, v = i - c * fo.copy_n;
        ((f32x4*)fo.copy_dst)[c * fo.copy_dst_stride + v] = ((const f32x4*)fo.copy_src)[c * fo.copy_src_stride + v];
    }
}

// Rows that one or two tokens multiply: the vector ALUs.  A workgroup owns `cols` consecutive columns and its waves share out the
// row in pieces of 512 k (16 bytes a lane); a wave keeps f(x) of its piece in registers and walks the columns four at a time, the
// eight behind them under way, so that w streams through without a pause while every other operand is read once a workgroup.  The
// partial sums of the columns meet in LDS once, at the end, where the threads that finish a column have had everything else
// they need since the start.  What bounds it is w from memory (5.5 TB/s of reads, 9.9 and 4.8 us for a 2.7B block's two), and what a
// launch takes until its first load has landed.  us of the two products of a 2.7B block, one token, in their places of a step (input with
// normalisation, convolution step and softplus; output with normalisation and residual): a workgroup per four columns with the row
// over its four waves, which fetched f(x) anew and paid two trips to memory in a row, 13.6 and 8.6, now 12.5 and 7.5; a step of eight blocks
// 203 -> 192, with two sequences 223 -> 197, at the width of 64 heads 143 -> 138 and 173 -> 155.
constexpr int FEW_PIECE = 512, FEW_WAVES = 12, FEW_COLS = 512;  // k of a piece; waves, columns of a workgroup at most

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t bits_of(float v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ float sum2(u32x2 q) {
    const uint32_t a = q[0], b = q[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// Sums of four values over the wave; the lanes 16 c .. 16 c + 15 have that of value c.
__device__ __forceinline__ float four_sums(const float (&a)[4]) {
    const float s0 = sum2(__builtin_amdgcn_permlane32_swap(bits_of(a[0]), bits_of(a[2]), false, false));
    const float s1 = sum2(__builtin_amdgcn_permlane32_swap(bits_of(a[1]), bits_of(a[3]), false, false));
    float v = sum2(__builtin_amdgcn_permlane16_swap(bits_of(s0), bits_of(s1), false, false));
    v = dpp_add<0x140, 0xF>(v);  // row_mirror
    v = dpp_add<0x141, 0xF>(v);  // row_half_mirror
    v = dpp_add<0x4E, 0xF>(v);   // quad_perm 2 3 0 1
    return dpp_add<0xB1, 0xF>(v);
}

// Longer rows than the waves have pieces go by in turns (two pieces of two rows to a wave do not fit the registers: 76 to 148 bytes of
// scratch a lane, and a step of 96 heads, whose d_inner is 6144, took 8 % longer).  STEP: with the convolution step (fo.cs).  Template
// arguments like MODE: a branch around loads ends in a wait for them.
template <int MODE, int R, bool STEP, bool STREAM>
__global__ __launch_bounds__(FEW_WAVES * 64) void k_linear_few(FewParams fp, FewOperands fo, int cols) {
    extern __shared__ float few_sums[];  // [columns, whole fours][R][NW], then the squares [R][NW]
    const int NW = fo.ks, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * cols, nc = fp.N - n0 < cols ? fp.N - n0 : cols, nb = (nc + 3) >> 2;
    float *red = few_sums, *sq = few_sums + ((cols + 3) & ~3) * R * NW;
    // columns and pieces beyond the end: nothing is fetched, zeros come back
    const uint32_t rowbytes = (uint32_t)fp.K * 2, bytes = (uint32_t)nc * rowbytes;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)(fp.w + (int64_t)n0 * fp.K), 0, bytes, 0x00020000);
    // (row fr, column n0 + fc) that thread tid finishes
    auto place = [&](int t, int& r, int& c) {
        r = R == 1 ? 0 : t / cols;
        c = t - r * cols;
        return r < fp.rows && c < nc;
    };
    int fr, fc;
    const bool finish = place(tid, fr, fc);
    const int frl = finish ? fr : 0, fnl = n0 + (finish ? fc : 0);
    const int range = FEW_PIECE * NW;
    float ss[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ss[r] = 0.f;
    StepTaps taps;
    float res = 0.f;
    for (int kb = 0; kb < fp.K; kb += range) {
        const int k = kb + FEW_PIECE * w + 8 * lane, kc = k < fp.K ? k : 0;
        const uint32_t off = k < fp.K ? (uint32_t)k * 2 : bytes;
        bf16x8 xv[R];
        f32x4 iw[2];
#pragma unroll
        for (int r = 0; r < R; ++r) xv[r] = *(const bf16x8*)(fp.x + (r < fp.rows ? r : 0) * fp.ldx + kc);
        if (MODE) {
            iw[0] = *(const f32x4*)(fp.in_w + kc);
            iw[1] = *(const f32x4*)(fp.in_w + kc + 4);
        }
        u32x4 W[2][4];
        auto load = [&](u32x4 (&b)[4], int n) {
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = __builtin_amdgcn_raw_buffer_load_b128(rw, off + (uint32_t)(4 * n + c) * rowbytes, 0, STREAM ? 2 : 0);
        };
        load(W[0], 0);
        load(W[1], 1);
        if (kb == 0) {
            if (STEP) taps = step_taps(fo, frl, fnl);
            if (fp.res) res = (float)fp.res[frl * fp.ldres + fnl];
        }
        float f[R][8];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool in = off < bytes && r < fp.rows;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = in ? (float)xv[r][e] : 0.f;
                if (MODE) {
                    ss[r] = fmaf(v, v, ss[r]);
                    v *= in ? iw[e >> 2][e & 3] : 0.f;
                }
                f[r][e] = v;
            }
        }
        auto use = [&](const u32x4 (&b)[4], int n) {
            float acc[R][4];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bf16x8 v = __builtin_bit_cast(bf16x8, b[c]);
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r][c] = fmaf(f[r][e], (float)v[e], acc[r][c]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float v = four_sums(acc[r]);
                float* at = red + ((4 * n + (lane >> 4)) * R + r) * NW + w;
                if ((lane & 15) == 0) *at = kb ? *at + v : v;
            }
        };
        int n = 0;
        for (; n + 2 <= nb; n += 2) {
            use(W[0], n);
            load(W[0], n + 2);
            use(W[1], n + 1);
            load(W[1], n + 3);
        }
        if (n < nb) use(W[0], n);
    }
    if (MODE) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float t = wave_total(ss[r]);
            if (lane == 0) sq[r * NW + w] = t;
        }
    }
    __syncthreads();
    for (int t = tid; t < R * cols; t += 64 * NW) {
        int r, c;
        if (!place(t, r, c)) continue;
        float v = 0.f, q2 = 0.f;
        for (int q = 0; q < NW; ++q) {  // fixed order: the result does not depend on which wave finished first
            v += red[(c * R + r) * NW + q];
            if (MODE) q2 += sq[r * NW + q];
        }
        const int n = n0 + c;
        if (MODE) v *= rsqrtf(q2 / (float)fp.K + fp.eps);
        if (fp.res) v += t == tid ? res : (float)fp.res[r * fp.ldres + n];
        const __bf16 ob = (__bf16)v;
        fp.out[r * fp.ldo + n] = STEP ? step_finish(fo, t == tid ? taps : step_taps(fo, r, n), r, n, ob) : ob;
    }
    move_pieces(fo, 64 * NW);
}

template <int MODE, bool STEP, bool STREAM>
hipError_t launch_few_kernel(const FewParams& fp, const FewOperands& fo, int cols, hipStream_t st) {
    const dim3 grid((unsigned)((fp.N + cols - 1) / cols)), block(64 * fo.ks);
    const size_t lds = (size_t)((cols + 3) / 4 * 4 + 1) * (fp.rows <= 1 ? 1 : FEW_ROWS_VALU) * fo.ks * sizeof(float);  // 49 KB at most
    if (fp.rows <= 1) hipLaunchKernelGGL((k_linear_few<MODE, 1, STEP, STREAM>), grid, block, lds, st, fp, fo, cols);
    else hipLaunchKernelGGL((k_linear_few<MODE, FEW_ROWS_VALU, STEP, STREAM>), grid, block, lds, st, fp, fo, cols);
    return hipGetLastError();
}

// N columns of K elements in as many rounds of `units` workgroups as they need with at most `most` columns each, all rounds full.  A
// workgroup's columns are addressed by 32 bits, with as much again beyond their end.
int even_columns(int N, int K, int units, int most) {
    most = most < (1 << 30) / K ? most : (1 << 30) / K;
    const int64_t round = (int64_t)units * most, all = (N + round - 1) / round * units;
    return (int)((N + all - 1) / all);
}

// As many waves a workgroup as share the row evenly, with one piece of it each, and as few columns, at least four, as give every compute
// unit about ten waves (80 KB of w under way), the same number of workgroups in each: eight a unit with some units holding twice as many as
// others took 3 % of a step.
// A product that stands alone has nothing but the way to its first load to hide, and more waves do: sixteen, where the registers hold
// them.  1536 x 3352 4.6 -> 4.4 us, 768 x 10576 with two rows 6.4 -> 6.0.  Better still are workgroups of four columns that start one after
// another, as many as fit: they keep the memory busier than a round that ends together, and do not meet on the same channels where 16 or
// 32 columns are a power of two of bytes.  us by rounds -> so: 5120 x 50288 85 -> 82, 8192 x 8192 24.9 -> 20.9, 16384 x 4096 26.1 -> 21.4; up to 4096
// columns one workgroup a unit, of whole fours, is a round that starts at once (5120 x 2560 5.2 with four columns, 4.6 with twelve).  Two rows,
// with twice the work to a load of w, are so where columns are many or rows long (8192 x 8192 25.8 -> 21.9, 4096 x 50288 72.5 -> 66.5, but 3072
// -> 6144 7.8 -> 8.1), and take four or five waves at most where they are many, and eight columns where five waves or two leave a unit's last
// ones idle (5120 x 50288 89.9 -> 85.3).
template <int MODE>
hipError_t launch_few(const FewParams& fp, FewOperands fo, hipStream_t st) {
    const int pieces = (fp.K + FEW_PIECE - 1) / FEW_PIECE;
    const bool alone = MODE == 0 && !fo.cs, two = fp.rows > 1, wide = fp.N >= 12288;
    const bool small = alone && pieces > 1 && (!two || wide || pieces > FEW_WAVES);
    const int most = !small ? FEW_WAVES : two && wide ? (pieces % 5 ? 4 : 5) : pieces > FEW_WAVES ? 8 : FEW_WAVES, turns = (pieces + most - 1) / most;
    fo.ks = (pieces + turns - 1) / turns;
    int cols = 4;
    if (small) {
        if (two && wide && (fo.ks == 5 || fo.ks <= 2)) cols = 8;
        if (!two && turns == 1 && fp.N <= 4096) cols = (fp.N + 1023) / 1024 * 4;
        if (cols < fp.N >> 22) cols = fp.N >> 22;  // a launch has at most 2^32 threads
    } else {
        cols = even_columns(fp.N, fp.K, 256 * (((alone && (!two || pieces <= 5) ? 16 : 10) + fo.ks / 2) / fo.ks), FEW_COLS);
        cols = cols < 4 ? 4 : cols;
    }
    if (fo.stream) return fo.cs ? launch_few_kernel<MODE, true, true>(fp, fo, cols, st) : launch_few_kernel<MODE, false, true>(fp, fo, cols, st);
    return fo.cs ? launch_few_kernel<MODE, true, false>(fp, fo, cols, st) : launch_few_kernel<MODE, false, false>(fp, fo, cols, st);
}

// More than a few rows (several sequences generated together): the same product on the matrix cores.  A workgroup owns `cols`
// consecutive columns; its waves share out the row in pieces of 256 k, one each up to rows of 3072 and two up to 6144, and keep the (at
// most 16) input rows of theirs as operands in registers while they walk the columns in tiles of 16, the next piece of w under way,
// one 16 x 16 x 32 MFMA per 32 k.  The partial tiles meet in LDS once, at the end.  The arithmetic is out of the way and the kernel
// again only streams w.  What bounds it is the number of cache lines an access touches: w is fetched as half rows of 512 contiguous
// bytes per half wave and turned into operands through LDS, and the input rows come in operand order (16 bytes per row and eight k,
// rows adjacent: `packed_at`) from the kernel before.  2560 x 10576 / 5120 x 2560 with 16 rows: 22 / 15 us with operands fetched
// straight from w's rows (16 lines an access), 16 / 11 with w through LDS, 13.4 / 8.6 with packed input too; reading w alone takes
// 9.9 / 5.9.  Then the way to the first load: everything the launch waits for is asked for before anything is waited for, w first (a
// sum that the compiler had moved in front of it, or a loop around a row that needs one turn, costs a trip to memory).  In their
// places of a step of 16 sequences a workgroup of eight waves per tile, two or three pieces to a wave one behind the other, took 15.7 /
// 10.3 us, this 13.2 / 9.6; the step of eight blocks 340 -> 315, with three sequences 257 -> 225.
typedef float f32x4v __attribute__((ext_vector_type(4)));

// Where (row, k) lies in the packed order.
__device__ __forceinline__ int64_t packed_at(int row, int k) { return ((int64_t)(k >> 3) * 16 + row) * 8 + (k & 7); }

constexpr int PIECE = 256, WPITCH = PIECE * 2 + 16;  // k per piece; bytes per LDS row of a piece of w
constexpr int MFMA_WAVES = 12, MFMA_COLS = 16, MAX_GROUPS = 8;  // waves of a workgroup at most, columns at least
__host__ __device__ constexpr int mfma_tiles(int ks) { return ks > 10 ? 4 : 6; }  // tiles of 16 columns at most: LDS
// Up to eight rows leave rows of a tile free: they carry what rounding the operand x in_w to bf16 left of the live rows, and
// the finished sums of a row's parts are added.  Up to four rows take three parts (rows r, r + 4, r + 8: all 24 bits, what the
// vector ALUs compute one and two rows with), up to eight two (r, r + 8: 16 bits); more rows one.  The extra parts cost
// nothing (three and four rows on fp32 operands on the vector ALUs took twice the time).
__host__ __device__ __forceinline__ int row_parts(int rows) { return rows <= 4 ? 3 : rows <= 8 ? 2 : 1; }
__host__ __device__ constexpr int part_step(int parts) { return parts == 3 ? 4 : parts == 2 ? 8 : 16; }  // rows between a row's parts
// What rounding v to b left of it: nothing of an infinity (of the row, or of the row times the norm's weight), which the first
// part carries alone.
__device__ __forceinline__ float rest_of(float v, __bf16 b) { return __builtin_isinf((float)b) ? 0.f : v - (float)b; }
__device__ __forceinline__ void pack_operand(__bf16* pack, int row, int k, float v, int parts) {
    const __bf16 hi = (__bf16)v;
    pack[packed_at(row, k)] = hi;
    if (parts == 1) return;
    v = rest_of(v, hi);
    const __bf16 mid = (__bf16)v;
    pack[packed_at(row + part_step(parts), k)] = mid;
    if (parts == 3) pack[packed_at(row + 8, k)] = (__bf16)(v - (float)mid);
}
inline size_t few_mfma_lds(int ks, int tiles) { return (size_t)ks * 16 * WPITCH + (size_t)tiles * ks * 1024 + 16 * 17 * 4; }
static_assert(MAX_GROUPS * 16 <= 16 * 17, "");
static_assert(10 * 16 * WPITCH + mfma_tiles(10) * 10 * 1024 <= MFMA_WAVES * 16 * WPITCH + mfma_tiles(MFMA_WAVES) * MFMA_WAVES * 1024, "");

// SRC 0: rows of x.  SRC 1: RMS normalisation over all of K times in_w, its squares summed on the way (the operand is
// x in_w, 1 / rms scales the finished sums).  SRC 2: packed rows, already times in_w, with `ssq` the partial
// sums of squares of their producer (nparts per group of K / groups, row r of part i at ssq[16 i + r]).  SRC 3: packed rows,
// no normalisation.  PARTS: row_parts(rows) (SRC 0: 1, rows of x are bf16 values as they are).
// PPW: pieces of a wave that it keeps operands of; longer rows go by in turns (SRC 1: one, two of them and what their
// normalisation takes do not fit the registers).  The first of w of a turn is asked for in front of the last tile of the turn before: with three
// rows 5120 x 50288 at its best split 89 us, 94 where it was asked for behind it.
template <int SRC, bool STEP, int PARTS, bool STREAM, int PPW, bool TURNS>
__global__ __launch_bounds__(MFMA_WAVES * 64) void k_linear_few_mfma(FewParams fp, FewOperands fo) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int KS = fo.ks, nthr = 64 * KS, tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    char* wt = lds + wv * 16 * WPITCH;
    const int blk = xcd_block(), n0 = blk * fo.cols, tiles = (fo.cols + 15) / 16, ncols = fp.N - n0 < fo.cols ? fp.N - n0 : fo.cols;
    float* part = (float*)(lds + KS * 16 * WPITCH);  // [tiles][KS][256]
    float* rs = part + tiles * KS * 256;             // [groups][16]: 1 / rms, or (one group) [16][17]: shares of the squares
    const int col = lane & 15, kq = lane >> 4;   // operand lanes: row of x / column of w, quarter of a 32-wide k step
    const int r2 = lane >> 5, l32 = lane & 31;   // fetching lanes: two columns of w at a time, 32 vectors of a piece each
    constexpr int pstep = part_step(PARTS);
    const int xrow = SRC == 1 ? col & (pstep - 1) : col;
    const __bf16* xr = fp.x + (SRC >= 2 ? (int64_t)0 : (int64_t)(xrow < fp.rows ? xrow : 0) * fp.ldx);
    constexpr bool norm = SRC == 2;
    // columns and k beyond the end: nothing is fetched, zeros come back
    const uint32_t rowbytes = (uint32_t)fp.K * 2, bytes = (uint32_t)ncols * rowbytes;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)(fp.w + (int64_t)n0 * fp.K), 0, bytes, 0x00020000);
    // the packed operand: zeros from its end on
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)fp.x, 0, SRC >= 2 ? (uint32_t)fp.K * 32 : 0, 0x00020000);
    constexpr int PU = 10;  // partial sums of squares asked for ahead (per thread)
    float sp[PU];
    const int TQ = nthr < 256 ? nthr >> 4 : 16;  // threads that share a row's sum
    // One group: its 1 / rms scales the finished sums, so nothing waits for it here.  Several: each piece of k lies inside
    // one group and is scaled before it is added.
    const bool norm_late = norm && fo.groups == 1;
    auto row_share = [&](int g, bool ahead) {  // this thread's share of the squares of row tid % 16
        const float* q = fo.ssq + (int64_t)16 * g * fo.nparts;
        float t = 0.f;
        if (ahead) {
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                float s = sp[u];
                asm volatile("" : "+v"(s));  // here: the sum is not to move to where everything would wait for these loads
                t += (tid >> 4) + TQ * u < fo.nparts ? s : 0.f;
            }
        }
        for (int i = (tid >> 4) + (ahead ? TQ * PU : 0); i < fo.nparts; i += TQ) t += q[16 * i + (tid & 15)];
        return t;
    };
    // the (row, column) of output t: a wave of t has four rows, all 16 columns
    auto row_of = [&](int t) { return 4 * ((t >> 6) & 3) + (t & 3); };
    auto col_of = [&](int t) { return 16 * (t >> 8) + ((t >> 2) & 15); };  // (from n0 on)
    StepTaps taps;  // of the thread's first output
    float ss = 0.f;
    uint32_t off[PPW];
    u32x4 v[8];
    auto aim = [&](int kb) {
#pragma unroll
        for (int j = 0; j < PPW; ++j) {
            const int kk = kb + (wv + KS * j) * PIECE + 8 * l32;
            off[j] = kk < fp.K ? (uint32_t)kk * 2 + (uint32_t)r2 * rowbytes : bytes;
        }
    };
    auto load = [&](int t, int j) {
        const uint32_t o = off[j] + (uint32_t)t * 16 * rowbytes;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, o + (uint32_t)(2 * i) * rowbytes, 0, STREAM ? 2 : 0);
    };
    aim(0);
    load(0, 0);
    bf16x8 a[PPW][8];
    auto operands = [&](int kb) {
#pragma unroll
        for (int j = 0; j < PPW; ++j)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int k = kb + (wv + KS * j) * PIECE + 32 * s + 8 * kq;
                if (SRC >= 2) a[j][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rx, (uint32_t)packed_at(col, k) * 2, 0, 0));
                if (SRC == 0) a[j][s] = *(const bf16x8*)(xr + (k < fp.K ? k : 0));
            }
    };
    operands(0);
    __builtin_amdgcn_sched_barrier(0);  // first what the whole product waits for
    auto taps_of = [&](int t) {
        const int r = row_of(t), n = n0 + col_of(t);
        return step_taps(fo, r < fp.rows ? r : 0, n < fp.N ? n : fp.N - 1);
    };
    if (STEP) taps = taps_of(tid);
    if (norm) {
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int i = (tid >> 4) + TQ * u;
            sp[u] = fo.ssq[16 * (i < fo.nparts ? i : 0) + (tid & 15)];
        }
    }
    for (int kb = 0;;) {
        if (norm && !norm_late && kb == 0) {
            for (int g = 0; g < fo.groups; ++g) {
                if (tid < 256) part[(tid & 15) * 16 + (tid >> 4)] = row_share(g, g == 0);
                __syncthreads();
                if (tid < 16) {
                    float t = 0.f;
                    for (int q = 0; q < TQ; ++q) t += part[tid * 16 + q];
                    rs[g * 16 + tid] = rsqrtf(t / (float)(fp.K / fo.groups) + fp.eps);
                }
                __syncthreads();
            }
        }
#pragma unroll
        for (int j = 0; j < PPW; ++j)
#pragma unroll
            for (int h = 0; h < 8; h += 4) {
                const int k0 = kb + (wv + KS * j) * PIECE + 32 * h + 8 * kq;
                f32x4 iw[4][2];
                if (SRC == 1) {
                    __builtin_amdgcn_sched_barrier(0);  // not all of the loads at once: registers
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int kc = k0 + 32 * s < fp.K ? k0 + 32 * s : 0;
                        a[j][h + s] = *(const bf16x8*)(xr + kc);
#pragma unroll
                        for (int e = 0; e < 2; ++e) iw[s][e] = *(const f32x4*)(fp.in_w + kc + 4 * e);
                    }
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const bool in = k0 + 32 * s < fp.K;
                    bf16x8 av = a[j][h + s];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        if (SRC == 1) {
                            const float x = in ? (float)av[e] : 0.f;
                            ss = fmaf(x, x, ss);
                            float xw = in ? x * iw[s][e >> 2][e & 3] : 0.f;
                            av[e] = (__bf16)xw;
                            if (PARTS > 1) {
                                xw = rest_of(xw, av[e]);
                                if (col >= pstep) av[e] = (__bf16)xw;
                            }
                            if (PARTS > 2) {
                                xw = rest_of(xw, av[e]);
                                if (col >= 2 * pstep) av[e] = (__bf16)xw;
                            }
                        } else if (SRC == 0 && !in) {
                            av[e] = (__bf16)0.f;
                        }
                    }
                    u32x4 words = __builtin_bit_cast(u32x4, av);
                    if (SRC == 1) asm volatile("" : "+v"(words));  // packed from here on: eight registers each otherwise
                    a[j][h + s] = __builtin_bit_cast(bf16x8, words);
                }
            }
        for (int t = 0; t < tiles; ++t) {
            f32x4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < PPW; ++j) {
#pragma unroll
                for (int i = 0; i < 8; ++i) *(u32x4*)(wt + (2 * i + r2) * WPITCH + 16 * l32) = v[i];
                if (j + 1 < PPW || t + 1 < tiles) {
                    load(j + 1 < PPW ? t : t + 1, j + 1 < PPW ? j + 1 : 0);
                } else if (TURNS && kb + PIECE * PPW * KS < fp.K) {  // the next turn's first
                    aim(kb + PIECE * PPW * KS);
                    load(0, 0);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // a wave's own rows: no barrier
                f32x4v d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 8; ++s)  // d[i] = out[row 4 kq + i][column col of the tile]
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][s], *(const bf16x8*)(wt + col * WPITCH + 64 * s + 16 * kq), d, 0, 0, 0);
                asm volatile("" ::: "memory");  // the next rows come in behind these reads
                if (norm && !norm_late) {
                    const int g = (int)((int64_t)(kb + (wv + KS * j) * PIECE) * fo.groups / fp.K);
                    const float4 q = *(const float4*)(rs + (g < fo.groups ? g : 0) * 16 + 4 * (kq & (pstep / 4 - 1)));
                    acc[0] += d[0] * q.x;
                    acc[1] += d[1] * q.y;
                    acc[2] += d[2] * q.z;
                    acc[3] += d[3] * q.w;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i] += d[i];
                }
            }
            f32x4v* at = (f32x4v*)(part + (t * KS + wv) * 256 + lane * 4);
            if (TURNS && kb) acc += *at;
            *at = acc;
        }
        kb += PIECE * PPW * KS;
        if (!TURNS || kb >= fp.K) break;
        operands(kb);
        // vmcnt(0): the compiler would otherwise have the first turn wait as well, where it has more under way
        if (SRC != 0 || STEP) __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    if (SRC == 1) {  // the row's squares of this wave's pieces
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (lane < 16) ((float*)wt)[lane] = ss;  // the wave's rows of w are used up
    }
    if (norm_late && tid < 256) rs[(tid & 15) * 17 + (tid >> 4)] = row_share(0, true);
    __syncthreads();
    auto finish = [&](int t, const StepTaps& tap) {
        const float* p = part + (t >> 8) * KS * 256;
        const int tt = t & 255;
        float o = 0.f;
        for (int q = 0; q < KS; ++q) o += p[q * 256 + tt];
        if (PARTS > 1 && tt < 128) {  // row r + pstep
            for (int q = 0; q < KS; ++q) o += p[q * 256 + tt + 16 * pstep];
            if (PARTS > 2 && tt < 64)  // row r + 8
                for (int q = 0; q < KS; ++q) o += p[q * 256 + tt + 128];
        }
        const int r = row_of(t), n = n0 + col_of(t);
        if (SRC == 1) {
            float m = 0.f;
            for (int q = 0; q < KS; ++q) m += ((const float*)(lds + q * 16 * WPITCH))[r];
            o *= rsqrtf(m / (float)fp.K + fp.eps);
        }
        if (norm_late) {
            float m = 0.f;
            for (int q = 0; q < TQ; ++q) m += rs[r * 17 + q];
            o *= rsqrtf(m / (float)fp.K + fp.eps);
        }
        const bool live = r < fp.rows && n < n0 + ncols;
        if (live && fp.res) o += (float)fp.res[r * fp.ldres + n];
        const __bf16 ob = (__bf16)o;
        if (live) fp.out[r * fp.ldo + n] = STEP ? step_finish(fo, tap, r, n, ob) : ob;
        if (fo.pack_out) {  // the next product's operand, and the squares its normalisation needs
            const float x = live ? (float)ob : 0.f;
            if (live) pack_operand(fo.pack_out, r, n, fo.pack_w ? x * fo.pack_w[n] : x, SRC ? PARTS : row_parts(fp.rows));
            float q = x * x;
            for (int off = 4; off < 64; off <<= 1) q += __shfl_xor(q, off, 64);
            if (((t >> 2) & 15) == 0 && n < fp.N) fo.pack_ssq[16 * (n >> 4) + r] = q;
        }
    };
    for (int t = tid; t < tiles * 256; t += nthr) {  // (whole waves)
        if (STEP && t != tid) taps = taps_of(t);
        finish(t, taps);
    }
    move_pieces(fo, nthr);
}

template <int SRC, bool STEP, int PARTS, bool STREAM, int PPW, bool TURNS>
hipError_t launch_few_mfma_kernel(const FewParams& fp, const FewOperands& fo, int wgs, size_t lds, hipStream_t st) {
    static bool raised[64];  // per device: more dynamic LDS than the default limit
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!raised[dev]) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_linear_few_mfma<SRC, STEP, PARTS, STREAM, PPW, TURNS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)few_mfma_lds(MFMA_WAVES, mfma_tiles(MFMA_WAVES)));
        if (e != hipSuccess) return e;
        raised[dev] = true;
    }
    hipLaunchKernelGGL((k_linear_few_mfma<SRC, STEP, PARTS, STREAM, PPW, TURNS>), dim3(wgs), dim3(fo.ks * 64), lds, st, fp, fo);
    return hipGetLastError();
}

template <int SRC, int PARTS, int PPW, bool TURNS>
hipError_t launch_few_mfma_pieces(const FewParams& fp, const FewOperands& fo, int wgs, size_t lds, hipStream_t st) {
    if (fo.stream)
        return fo.cs ? launch_few_mfma_kernel<SRC, true, PARTS, true, PPW, TURNS>(fp, fo, wgs, lds, st)
                     : launch_few_mfma_kernel<SRC, false, PARTS, true, PPW, TURNS>(fp, fo, wgs, lds, st);
    return fo.cs ? launch_few_mfma_kernel<SRC, true, PARTS, false, PPW, TURNS>(fp, fo, wgs, lds, st)
                 : launch_few_mfma_kernel<SRC, false, PARTS, false, PPW, TURNS>(fp, fo, wgs, lds, st);
}

template <int SRC, int PARTS>
hipError_t launch_few_mfma_parts(const FewParams& fp, const FewOperands& fo, int ppw, int wgs, size_t lds, hipStream_t st) {
    constexpr int most = SRC == 1 ? 1 : 2;
    if constexpr (SRC == 0)
        if (ppw == 1 && fp.K > PIECE * fo.ks) return launch_few_mfma_pieces<SRC, PARTS, 1, true>(fp, fo, wgs, lds, st);
    if (fp.K > PIECE * most * fo.ks) return launch_few_mfma_pieces<SRC, PARTS, most, true>(fp, fo, wgs, lds, st);
    return ppw == most ? launch_few_mfma_pieces<SRC, PARTS, most, false>(fp, fo, wgs, lds, st) : launch_few_mfma_pieces<SRC, PARTS, 1, false>(fp, fo, wgs, lds, st);
}

template <int SRC>
hipError_t launch_few_mfma_src(const FewParams& fp, const FewOperands& fo, int ppw, int wgs, size_t lds, hipStream_t st) {
    const int parts = row_parts(fp.rows);
    if (parts == 3) return launch_few_mfma_parts<SRC, 3>(fp, fo, ppw, wgs, lds, st);
    if (parts == 2) return launch_few_mfma_parts<SRC, 2>(fp, fo, ppw, wgs, lds, st);
    return launch_few_mfma_parts<SRC, 1>(fp, fo, ppw, wgs, lds, st);
}

// Waves by the row, as launch_few: up to twelve where that saves a second turn, else up to ten.  (With ten at most the rows of a block of 96 heads,
// of 3072 and 6144, went by in two turns of six waves: three blocks for three sequences 131 us, 112 so; 6144 x 2560 alone 9.1 and 8.6.  In more turns
// anyway, three turns of eleven waves are 4 % slower than four of eight, and four of seven 6 % faster than three of ten that do not have work for
// all: 14336 x 4096 with sixteen rows 27.4 and 25.9.)  One round of workgroups (or as many as are full), the same number in every compute unit, of at least
// MFMA_COLS columns: with less of w than that to each, the operands of the rows would be most of what they fetch.
// A product that stands alone takes single tiles of a few waves, which start one after another (see launch_few), where its rows cost little to fetch
// again: up to eight where four waves hold a row, up to four where a round would be long.  us by rounds -> so: 1024 x 50288 with three rows 21.3
// -> 17.8, 2048 x 50288 34.4 -> 31.6, 4096 x 50288 75 -> 72, 5120 x 50288 97 -> 92, 16384 x 16384 101 -> 88; with eight rows 1024 x 50288 21.4 -> 18.1
// but 2560 x 50288 40.8 -> 45.4 (eight waves of a piece each, 4096 x 50288, 78 -> 75).  With more rows three tiles are better than the five or six of a
// round where four waves hold a row (1024 x 131072 43 -> 40).
struct FewSplit {
    int ks, ppw, cols, wgs;
};
FewSplit few_split(int K, int N, bool two, bool whole, int lone) {  // two pieces a wave where one is not enough; whole tiles; rows of a product alone (else 0)
    FewSplit f;
    const int pieces = (K + PIECE - 1) / PIECE;
    const bool longer = (lone <= 4 || K % 2048 == 0) && (N >= 32768 || (int64_t)N * K >= 1 << 27), single = lone && lone <= 8 && pieces > 1 && (pieces <= 4 || longer);
    f.ppw = two && !single && (pieces > MFMA_WAVES || (pieces > 10 && N > 256 * 64)) ? 2 : 1;  // (twelve waves have four tiles: one round, or six waves with six)
    const int need = (pieces + f.ppw - 1) / f.ppw;
    auto waves = [&](int turns) { return (need + turns - 1) / turns; };
    int turns = single ? (need % 8 ? (need + 3) / 4 : need / 8) : need <= MFMA_WAVES ? 1 : (need + 9) / 10;
    if (!single && turns > 1 && waves(turns + 1) > 5 && waves(turns + 1) * (turns + 1) < waves(turns) * turns) ++turns;
    f.ks = waves(turns);
    const int cols = even_columns(N, K, 256 * ((10 + f.ks / 2) / f.ks), 16 * mfma_tiles(f.ks));
    f.cols = single || cols < MFMA_COLS ? MFMA_COLS : lone && pieces <= 4 && cols > 48 ? 48 : cols;
    if (whole) f.cols = (f.cols + 15) / 16 * 16;
    f.wgs = (N + f.cols - 1) / f.cols;
    return f;
}

hipError_t launch_few_mfma(const FewParams& fp, FewOperands fo, int src, hipStream_t st) {
    const FewSplit f = few_split(fp.K, fp.N, src != 1, fo.pack_out != nullptr, src == 0 && !fo.cs ? fp.rows : 0);
    const int ppw = f.ppw, wgs = f.wgs;
    const size_t lds = few_mfma_lds(f.ks, (f.cols + 15) / 16);
    fo.ks = f.ks;
    fo.cols = f.cols;
    if (src == 2 && !fo.ssq) src = 3;
    if (src == 0) return launch_few_mfma_parts<0, 1>(fp, fo, ppw, wgs, lds, st);
    if (src == 1) return launch_few_mfma_src<1>(fp, fo, ppw, wgs, lds, st);
    if (src == 2) return launch_few_mfma_src<2>(fp, fo, ppw, wgs, lds, st);
    return launch_few_mfma_src<3>(fp, fo, ppw, wgs, lds, st);
}

struct MidParams {
    const __bf16* zx;   // [T, ld]: (z | xBC | dt_raw) of the tokens
    int64_t ld;
    const float *conv_w, *conv_b, *dt_bias, *A, *D;
    const __bf16* cs_in;  // [3, conv_dim] or null: the convolution's inputs of the three tokens before
    __bf16* cs_out;       // [3, conv_dim] or null; never the same buffer as cs_in
    float* state;         // [H, P, N], updated in place
    __bf16* y;            // [T, d_inner]
    int T, H, P, G, N, hpg, d_inner, conv_dim, off_xbc, off_dt;
    // several independent sequences in one launch (blockIdx.y): sequence b owns rows b T .. b T + T - 1 of zx and y
    // and the states `b` strides (elements) further on
    int64_t state_bs, cs_in_bs, cs_out_bs;
    int gate;  // y is y silu(z), rounded once: what the normalisation behind takes the squares of
    // with both: y silu(z) pack_w goes to the packed operand of the output product instead, its squares (before pack_w)
    // summed over the workgroup's rows to pack_ssq[16 (h gridDim.z + z) + row]
    __bf16* pack;
    const float* pack_w;
    float* pack_ssq;
};

// input of the convolution, channel c, token `pos` of this call (negative: from the entering state)
__device__ __forceinline__ float conv_input(const MidParams& mp, int pos, int c) {
    if (pos >= 0) return (float)mp.zx[pos * mp.ld + mp.off_xbc + c];
    return mp.cs_in ? (float)mp.cs_in[(3 + pos) * mp.conv_dim + c] : 0.f;
}

// silu(bias + four taps), rounded as the block stores it between its steps
__device__ __forceinline__ float conv_output(const MidParams& mp, int t, int c) {
    const float* w = mp.conv_w + (int64_t)c * 4;
    const float pre = mp.conv_b[c] + w[0] * conv_input(mp, t - 3, c) + w[1] * conv_input(mp, t - 2, c) + w[2] * conv_input(mp, t - 1, c) +
                      w[3] * conv_input(mp, t, c);
    return through_bf16(pre * sigmoid_fast(pre));
}

// What is stored for channel c of token t: y, or y times silu of its gate.
__device__ __forceinline__ __bf16 mid_out(const MidParams& mp, int t, int c, float y) {
    if (mp.gate) {
        const float z = (float)mp.zx[t * mp.ld + c];
        y *= z * sigmoid_fast(z);
    }
    return (__bf16)y;
}

// Workgroup (head h, sequence b, z): wave w owns the RPW state rows p = (4 z + w) RPW + rr, lane l their columns
// n = l, l + 64, ..., which stay in registers over the tokens of the call (requested first: nothing below waits
// for them until the first update).  Per token the workgroup convolves the B and C channels of its group into
// LDS (every workgroup of the group does: a few hundred channels against the P N elements of a head's state --
// which is why several sequences at once take more rows per wave and fewer workgroups), each wave the x channels
// of its rows.
constexpr int MID_NPL = 8;  // state columns per lane at most (N <= 512)

template <int RPW>
__global__ __launch_bounds__(256) void k_decode_mid(MidParams mp) {
    extern __shared__ float bc[];  // B[0..N), C[0..N) of the group, this token
    {  // this workgroup's sequence
        const int64_t b = blockIdx.y;
        mp.zx += b * mp.T * mp.ld;
        mp.y += b * mp.T * mp.d_inner;
        mp.state += b * mp.state_bs;
        if (mp.cs_in) mp.cs_in += b * mp.cs_in_bs;
        if (mp.cs_out) mp.cs_out += b * mp.cs_out_bs;
    }
    const int h = blockIdx.x, g = h / mp.hpg;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p0 = (4 * blockIdx.z + w) * RPW;
    float* S = mp.state + (int64_t)h * mp.P * mp.N;
    float s[RPW][MID_NPL];
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr)
#pragma unroll
        for (int i = 0; i < MID_NPL; ++i) {
            const int n = lane + 64 * i;
            s[rr][i] = p0 + rr < mp.P && n < mp.N ? S[(int64_t)(p0 + rr) * mp.N + n] : 0.f;
        }
    const float Ah = mp.A[h], Dh = mp.D[h], bias_h = mp.dt_bias[h];
    const int cB = mp.d_inner + g * mp.N, cC = mp.d_inner + (mp.G + g) * mp.N;
    for (int t = 0; t < mp.T; ++t) {
        for (int i = threadIdx.x; i < 2 * mp.N; i += 256) bc[i] = conv_output(mp, t, i < mp.N ? cB + i : cC + (i - mp.N));
        const float v = (float)mp.zx[t * mp.ld + mp.off_dt + h] + bias_h;
        const float dtv = through_bf16(fmaxf(v, 0.f) + log1pf(__expf(-fabsf(v))));  // softplus
        const float a = __expf(dtv * Ah);
        float xv[RPW];
#pragma unroll
        for (int rr = 0; rr < RPW; ++rr) xv[rr] = p0 + rr < mp.P ? conv_output(mp, t, h * mp.P + p0 + rr) : 0.f;
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < RPW; ++rr) {
            if (p0 + rr < mp.P) {
                const float dx = dtv * xv[rr];
                float acc = 0.f;
#pragma unroll
                for (int i = 0; i < MID_NPL; ++i) {
                    const int n = lane + 64 * i;
                    if (n < mp.N) {
                        s[rr][i] = a * s[rr][i] + dx * bc[n];
                        acc += bc[mp.N + n] * s[rr][i];
                    }
                }
                acc = wave_sum(acc);
                if (lane == 0) mp.y[(int64_t)t * mp.d_inner + h * mp.P + p0 + rr] = mid_out(mp, t, h * mp.P + p0 + rr, acc + Dh * xv[rr]);
            }
        }
        __syncthreads();  // the next token's B and C replace these
    }
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr)
#pragma unroll
        for (int i = 0; i < MID_NPL; ++i) {
            const int n = lane + 64 * i;
            if (p0 + rr < mp.P && n < mp.N) S[(int64_t)(p0 + rr) * mp.N + n] = s[rr][i];
        }
    if (mp.cs_out) {  // the last three inputs of [entering state ; this call's tokens]
        for (int i = lane; i < 3 * RPW; i += 64) {
            const int rr = i / 3, j = i - 3 * rr;
            if (p0 + rr < mp.P) mp.cs_out[j * mp.conv_dim + h * mp.P + p0 + rr] = (__bf16)conv_input(mp, mp.T - 3 + j, h * mp.P + p0 + rr);
        }
        if (h % mp.hpg == 0 && blockIdx.z == 0)  // the group's B and C channels: once
            for (int i = threadIdx.x; i < 6 * mp.N; i += 256) {
                const int j = i / (2 * mp.N), ii = i % (2 * mp.N);
                const int c = ii < mp.N ? cB + ii : cC + (ii - mp.N);
                mp.cs_out[j * mp.conv_dim + c] = (__bf16)conv_input(mp, mp.T - 3 + j, c);
            }
    }
}

// One token for each of several sequences whose product has been through the convolution step and softplus already:
// the recurrence and the gate, nothing else.  16-byte accesses to the state (N a multiple of 4, N <= 128 NV): half a
// wave owns U consecutive rows, lane l of the half the columns 4 l .. 4 l + 3 (+ 128 i).  Everything is asked for at once,
// so what bounds it is the state's way in and out (16 sequences of 80 heads: 84 MB).
template <int NV, int U, bool STREAM>
__global__ __launch_bounds__(256) void k_decode_step(MidParams mp) {
    __shared__ float sq[8];
    const int h = blockIdx.x, b = blockIdx.y, g = h / mp.hpg, N = mp.N, tid = threadIdx.x, l32 = tid & 31, hw = tid >> 5;
    const int p0 = 8 * U * blockIdx.z + U * hw;
    const __bf16* zx = mp.zx + (int64_t)b * mp.ld;
    const __bf16* xb = zx + mp.off_xbc;
    float* S = mp.state + b * mp.state_bs + (int64_t)h * mp.P * N;
    f32x4 s[U][NV];
    bf16x4 bv[NV], cv[NV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int p = p0 + u < mp.P ? p0 + u : mp.P - 1, n = 4 * l32 + 128 * i;
            s[u][i] = fetch<STREAM>((const f32x4*)(S + (int64_t)p * N + (n < N ? n : 0)));
        }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int n = 4 * l32 + 128 * i;
        bv[i] = *(const bf16x4*)(xb + mp.d_inner + g * N + (n < N ? n : 0));
        cv[i] = *(const bf16x4*)(xb + mp.d_inner + (mp.G + g) * N + (n < N ? n : 0));
    }
    float xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = (float)xb[h * mp.P + (p0 + u < mp.P ? p0 + u : mp.P - 1)];
    // after the sums over the half wave: the row this lane finishes (all lanes of a group of 32 / U the same one)
    const int p_mine = p0 + ((l32 * U) >> 5), c_mine = h * mp.P + (p_mine < mp.P ? p_mine : mp.P - 1);
    const bool mine = (l32 & (32 / U - 1)) == 0 && p_mine < mp.P;
    const float x_mine = (float)xb[c_mine], z = mp.gate ? (float)zx[c_mine] : 0.f, pw = mp.pack ? mp.pack_w[c_mine] : 1.f;
    const float dtv = (float)zx[mp.off_dt + h], a = __expf(dtv * mp.A[h]), Dh = mp.D[h];
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float dx = dtv * xv[u];
        acc[u] = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            f32x4& q = s[u][i];
            q[0] = a * q[0] + dx * (float)bv[i][0];
            q[1] = a * q[1] + dx * (float)bv[i][1];
            q[2] = a * q[2] + dx * (float)bv[i][2];
            q[3] = a * q[3] + dx * (float)bv[i][3];
            const int p = p0 + u, n = 4 * l32 + 128 * i;
            if (n < N) {
                acc[u] += ((float)cv[i][0] * q[0] + (float)cv[i][1] * q[1]) + ((float)cv[i][2] * q[2] + (float)cv[i][3] * q[3]);
                if (p < mp.P) put<STREAM>((f32x4*)(S + (int64_t)p * N + n), q);
            }
        }
    }
    // halve the rows with the lanes until a lane has one, then sum over the lanes that share it
    int off = 16;
#pragma unroll
    for (int k = U; k > 1; k >>= 1, off >>= 1)
#pragma unroll
        for (int u = 0; u < k / 2; ++u) {
            const bool up = l32 & off;
            const float keep = up ? acc[u + k / 2] : acc[u], give = up ? acc[u] : acc[u + k / 2];
            acc[u] = keep + __shfl_xor(give, off, 64);
        }
    for (; off > 0; off >>= 1) acc[0] += __shfl_xor(acc[0], off, 64);
    float y = acc[0] + Dh * x_mine;
    if (mp.gate) y *= z * sigmoid_fast(z);
    if (!mp.pack) {
        if (mine) mp.y[(int64_t)b * mp.d_inner + c_mine] = (__bf16)y;
        return;
    }
    if (mine) pack_operand(mp.pack, b, c_mine, y * pw, row_parts(gridDim.y));
    float q = mine ? y * y : 0.f;
    for (int o = 16; o >= 32 / U; o >>= 1) q += __shfl_xor(q, o, 64);
    if (l32 == 0) sq[hw] = q;
    __syncthreads();
    if (tid == 0) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += sq[i];
        mp.pack_ssq[16 * (h * gridDim.z + blockIdx.z) + b] = sum;
    }
}

// rows per half wave: as many as still leave every compute unit a workgroup or a few (and with packed output, fewer
// workgroups leave fewer partial sums of squares to add up)
int step_rows(int H, int P, int nb) {
    const int64_t hn = (int64_t)H * nb;
    return hn * ((P + 63) / 64) >= 768 ? 8 : hn * ((P + 31) / 32) >= 256 ? 4 : 1;
}

template <int NV, bool STREAM>
void launch_step(const MidParams& mp, int nb, hipStream_t st) {
    const int u = step_rows(mp.H, mp.P, nb);
    const dim3 grid(mp.H, nb, (mp.P + 8 * u - 1) / (8 * u));
    if (u == 8) hipLaunchKernelGGL((k_decode_step<NV, 8, STREAM>), grid, dim3(256), 0, st, mp);
    else if (u == 4) hipLaunchKernelGGL((k_decode_step<NV, 4, STREAM>), grid, dim3(256), 0, st, mp);
    else hipLaunchKernelGGL((k_decode_step<NV, 1, STREAM>), grid, dim3(256), 0, st, mp);
}

bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool few_rows_supported(const FewRowsJob& j) {
    if (j.rows < 1 || j.rows > FEW_ROWS || j.K <= 0 || j.N <= 0 || ((j.K | j.N) & 7) || j.K > 1 << 24) return false;  // (offsets within a workgroup's columns of w: 32 bits)
    if (!j.x || !j.w || !j.out || !al16(j.x) || !al16(j.w) || (j.mode != 2 && ((j.ldx & 7) || j.ldx < j.K)) || j.ldo < j.N) return false;
    if (j.mode < 0 || j.mode > 2) return false;
    if (j.mode == 2 || j.pack_out) {
        if (j.rows <= FEW_ROWS_VALU) return false;
        if (j.mode == 2 && j.ssq && (j.groups < 1 || j.groups > MAX_GROUPS || j.nparts < 1 || (j.groups > 1 && j.K % (j.groups * PIECE)))) return false;
        if (j.pack_out && (!j.pack_ssq || !al16(j.pack_out))) return false;
    }
    if (j.mode == 1 && (!j.in_w || !al16(j.in_w))) return false;
    if (j.res && j.ldres < j.N) return false;
    if (j.copy_bytes) {
        const size_t chunks = j.copy_chunks > 0 ? j.copy_chunks : 1;
        if (!j.copy_src || !j.copy_dst || !al16(j.copy_src) || !al16(j.copy_dst) || (j.copy_bytes & 15) || j.copy_chunks < 0 ||
            ((j.copy_src_stride | j.copy_dst_stride) & 15) || j.copy_bytes / 16 * chunks > (size_t)j.N * 16)  // a few vectors per thread at most
            return false;
    }
    return true;
}

hipError_t launch_linear_few_rows(const FewRowsJob& j, hipStream_t st) {
    if (!few_rows_supported(j)) return hipErrorInvalidValue;
    FewParams fp;
    fp.x = (const __bf16*)j.x;
    fp.w = (const __bf16*)j.w;
    fp.res = (const __bf16*)j.res;
    fp.out = (__bf16*)j.out;
    fp.in_w = j.in_w;
    fp.ldx = j.ldx;
    fp.ldo = j.ldo;
    fp.ldres = j.ldres;
    fp.rows = j.rows;
    fp.K = j.K;
    fp.N = j.N;
    fp.eps = j.eps;
    FewOperands fo;
    fo.copy_src = j.copy_src;
    fo.copy_dst = j.copy_dst;
    fo.copy_n = (int)(j.copy_bytes / 16);
    fo.copy_chunks = j.copy_bytes ? (j.copy_chunks > 0 ? j.copy_chunks : 1) : 0;
    fo.copy_src_stride = (int64_t)(j.copy_src_stride / 16);
    fo.copy_dst_stride = (int64_t)(j.copy_dst_stride / 16);
    fo.ssq = j.ssq;
    fo.nparts = j.nparts;
    fo.groups = j.groups;
    fo.pack_out = (__bf16*)j.pack_out;
    fo.pack_w = j.pack_w;
    fo.pack_ssq = j.pack_ssq;
    fo.stream = j.stream;
    fo.cs = (__bf16*)j.cs;
    fo.cs_bs = j.cs_bs;
    fo.conv_w = j.conv_w;
    fo.conv_b = j.conv_b;
    fo.dt_bias = j.dt_bias;
    fo.off_xbc = j.off_xbc;
    fo.off_dt = j.off_dt;
    fo.conv_dim = j.off_dt - j.off_xbc;
    if (j.rows > FEW_ROWS_VALU) return launch_few_mfma(fp, fo, j.mode, st);
    return j.mode ? launch_few<1>(fp, fo, st) : launch_few<0>(fp, fo, st);
}

bool step_supported(const DecodeMidJob& j) {
    return j.T == 1 && j.N % 4 == 0 && j.N <= 256 && al16(j.state) && j.state_bs % 4 == 0 && al16(j.zx) && j.ld % 4 == 0 && (j.H * j.P) % 4 == 0 &&
           al16(j.conv_w);
}
int step_parts(const DecodeMidJob& j) {
    const int u = step_rows(j.H, j.P, j.nb > 0 ? j.nb : 1);
    return j.H * ((j.P + 8 * u - 1) / (8 * u));
}

hipError_t launch_decode_mid(const DecodeMidJob& j, hipStream_t st) {
    const int nb = j.nb > 0 ? j.nb : 1;
    if (nb > 65535 || (int64_t)nb * j.T > FEW_ROWS) return hipErrorInvalidValue;
    if (j.T < 1 || j.T > FEW_ROWS || j.H <= 0 || j.H > 65535 || j.P <= 0 || j.G <= 0 || j.N <= 0 || j.H % j.G) return hipErrorInvalidValue;
    if (!j.zx || !j.conv_w || !j.conv_b || !j.dt_bias || !j.A || !j.D || !j.state || !j.y || (j.cs_out && j.cs_out == j.cs_in))
        return hipErrorInvalidValue;
    if (j.N > 64 * MID_NPL || j.P > 256) return hipErrorInvalidValue;  // a state row in a wave's registers, a row per wave
    MidParams mp;
    mp.zx = (const __bf16*)j.zx;
    mp.ld = j.ld;
    mp.conv_w = j.conv_w;
    mp.conv_b = j.conv_b;
    mp.dt_bias = j.dt_bias;
    mp.A = j.A;
    mp.D = j.D;
    mp.cs_in = (const __bf16*)j.cs_in;
    mp.cs_out = (__bf16*)j.cs_out;
    mp.state = j.state;
    mp.y = (__bf16*)j.y;
    mp.T = j.T;
    mp.H = j.H;
    mp.P = j.P;
    mp.G = j.G;
    mp.N = j.N;
    mp.hpg = j.H / j.G;
    mp.d_inner = j.H * j.P;
    mp.conv_dim = mp.d_inner + 2 * j.G * j.N;
    mp.off_xbc = mp.d_inner;
    mp.off_dt = mp.d_inner + mp.conv_dim;
    mp.state_bs = j.state_bs;
    mp.cs_in_bs = j.cs_in_bs;
    mp.cs_out_bs = j.cs_out_bs;
    mp.gate = j.gate;
    mp.pack = (__bf16*)j.pack;
    mp.pack_w = j.pack_w;
    mp.pack_ssq = j.pack_ssq;
    if (j.stepped) {
        if (!step_supported(j) || (j.pack && (!j.gate || !j.pack_w || !j.pack_ssq))) return hipErrorInvalidValue;
        if (j.stream) {
            if (j.N <= 128) launch_step<1, true>(mp, nb, st);
            else launch_step<2, true>(mp, nb, st);
        } else {
            if (j.N <= 128) launch_step<1, false>(mp, nb, st);
            else launch_step<2, false>(mp, nb, st);
        }
        return hipGetLastError();
    }
    if (j.pack) return hipErrorInvalidValue;
    // rows per wave: one where that gives few enough workgroups (every one of them convolves its group's B and C
    // channels), else 4 or 16
    const size_t lds = (size_t)2 * j.N * sizeof(float);
    auto wgs = [&](int rpw) { return (int64_t)j.H * nb * ((j.P + 4 * rpw - 1) / (4 * rpw)); };
    if (wgs(1) <= 8192)
        hipLaunchKernelGGL(k_decode_mid<1>, dim3(j.H, nb, (j.P + 3) / 4), dim3(256), lds, st, mp);
    else if (wgs(4) <= 2048)
        hipLaunchKernelGGL(k_decode_mid<4>, dim3(j.H, nb, (j.P + 15) / 16), dim3(256), lds, st, mp);
    else
        hipLaunchKernelGGL(k_decode_mid<16>, dim3(j.H, nb, (j.P + 63) / 64), dim3(256), lds, st, mp);
    return hipGetLastError();
}

}  // namespace ssdk
