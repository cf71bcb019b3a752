// The two projections of the Mamba-2 block (dense layers without bias, bf16 storage, fp32 accumulation):
//     out[t,o] = sum_i x[t,i] w[o,i];    dx[t,i] = sum_o dout[t,o] w[o,i];    dw[o,i] = sum_t dout[t,o] x[t,i]
// (the input projection in front of the convolution, whose output width is the larger part of the per-token
// grid-cell activations of App. C, Tab. 7, and the output projection behind the gated normalisation).
// These are dense contractions far above the machine's flop/byte ridge: matrix-core bound.
//
// One scheme, C[M,N] = op(A) op(B)^T with fp32 accumulators in v_mfma_f32_16x16x32_bf16 tiles, for the three
// operand layouts the three products need: an operand is either stored with the contraction index
// contiguous ("k-major": rows of x for the forward product) or with it as the row index (x and dout for
// dw, w for dx).  Both kinds are staged in LDS exactly as they lie in memory (16-byte vectors); k-major
// tiles are read back as plain 16-byte operands, the others through the transposing LDS read.
// One scheme of tiles, three widths: 256 x 256, 256 x 192 or 256 x 128 per workgroup (eight waves of 64 x 128 / 96 / 64, one
// workgroup per compute unit, loads straight to LDS two K steps ahead); the two gradient products share a launch, and the
// launch rule below chooses the one, or for the forward product the two, whose tiles fit the machine best.  Workgroup ids are
// remapped so that each XCD works on a compact block of the tile grid (its L2 then holds the A and B panels that block shares).
#include <stdint.h>
#include <string.h>

#include "mfma_common.h"

namespace ssdk {
namespace {

using namespace mf;

constexpr int BKK = 64;            // K step

struct GemmParams {
    const bf16_t* A;
    const bf16_t* B;
    void* C;
    int64_t lda, ldb, ldc;
    int M, N, K;
    int tiles_m, tiles_n;
    int c_f32;       // C is fp32 (else bf16)
    int accumulate;  // fp32 only: C += product
};

// Tile `id` of the product.  Hardware hands consecutive workgroup ids to the eight XCDs in turn; id -> (id % 8,
// id / 8) gives every XCD a contiguous eighth of a walk that goes down groups of eight row tiles column by
// column, so the workgroups resident on one XCD at a time share a few A row panels and B column panels.
__device__ __forceinline__ void tile_of(const GemmParams& gp, int id, int& tm, int& tn) {
    const int nt = gp.tiles_m * gp.tiles_n;
    if (nt % 8 == 0) id = (id & 7) * (nt >> 3) + (id >> 3);
    const int per_group = 8 * gp.tiles_n;
    const int grp = id / per_group, in = id - grp * per_group;
    const int first = grp * 8;
    const int gsz = gp.tiles_m - first < 8 ? gp.tiles_m - first : 8;
    tm = first + in % gsz;
    tn = in / gsz;
}

// Offsets into K steps stay below 2^31 for row strides up to this.
constexpr int64_t MAX_LD = 1 << 22;
constexpr int GTHR = 512;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The MFMAs are issued with the B operand first, so an accumulator tile holds the transposed product: lane
// -> row m = lane % 16 of C, its four registers -> the consecutive columns 4 (lane / 16) + 0..3.
// Every lane thus stores 8 bytes (bf16) or 16 bytes (fp32) at a time (N is a multiple of 8, so a group of four columns is inside C or
// outside as one).
// fp32 results (weight gradients): where they are added to what is there, the old values of AHEAD columns of tiles are asked for
// before the first of them is used, without a branch (what lies outside C is aimed beyond the descriptor's end): where each of them
// stands under a condition, the compiler waits for all in flight.  4096 rows, 2560 <-> 10576 (both gradients) 375 -> 367 us, 2560 <->
// 5120 180 -> 177; three columns ahead the same.  Where nothing is added they are stores alone: with the loads from an empty
// descriptor instead 1024 rows 5120 <-> 2560 took 63.5 us, now 60.8, dw alone 35.7, now 34.0.
template <int WJ>
__device__ __forceinline__ void store_acc_f32(const GemmParams& gp, const f32x4 (&acc)[4][2 * WJ], int row0, int col0, int lane) {
    constexpr int AHEAD = 4;
    const int row_l = lane & 15, col_l = (lane >> 4) * 4;
    float* org = (float*)gp.C + (int64_t)row0 * gp.ldc + col0;
    if (gp.ldc > MAX_LD / 2) {  // beyond offsets of 32 bits
#pragma unroll
        for (int j = 0; j < 2 * WJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4* at = (f32x4*)(org + (int64_t)(i * 16 + row_l) * gp.ldc + j * 16 + col_l);
                if (row0 + i * 16 + row_l < gp.M && col0 + j * 16 + col_l < gp.N) *at = acc[i][j] + (gp.accumulate ? *at : (f32x4)(0.f));
            }
        return;
    }
    const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc((void*)org, 0, 0x3fffffff, 0x00020000);
    uint32_t row[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) row[i] = row0 + i * 16 + row_l < gp.M ? (uint32_t)(i * 16 + row_l) * (uint32_t)(gp.ldc * 4) : 0x80000000u;
    auto col = [&](int j) { return col0 + j * 16 + col_l < gp.N ? (uint32_t)(j * 16 + col_l) * 4 : 0x40000000u; };
    if (!gp.accumulate) {  // uniform
#pragma unroll
        for (int j = 0; j < 2 * WJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j]), to, row[i] + col(j), 0, 0);
        return;
    }
    f32x4 old[AHEAD][4];
    auto ask = [&](int j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) old[j % AHEAD][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(to, row[i] + col(j), 0, 0));
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) ask(j);
#pragma unroll
    for (int j = 0; j < 2 * WJ; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[i][j] + old[j % AHEAD][i]), to, row[i] + col(j), 0, 0);
        if (j + AHEAD < 2 * WJ) ask(j + AHEAD);
    }
}

// One operand tile of a K step in LDS: k-major [ROWS][64 k] (128 bytes a row) or [64 k][ROWS] (2 ROWS bytes a row), filled by
// loads that go from memory straight to LDS: a wave's load puts 64 consecutive 16-byte pieces down, so there is no room for
// padding.  Instead the pieces of a row are permuted -- which piece a lane fetches, not where it lands -- so that the rows
// that one operand read touches fall into distinct banks:
//   k-major: piece s of row r holds piece s ^ (r / 2 & 7) of the row (a read takes one of four pieces of sixteen rows;
//   with r & 7 every read took twice as long),
//   else: piece s of k row k holds piece s ^ 2 h(k), h = k % 4 + 4 (k / 8 % 2) (half a wave's transposing read takes 32 bytes
//   of each of the k rows 0..3 and 8..11).
template <int ROWS, bool KMAJOR>
struct Tile {
    static constexpr int PITCH = KMAJOR ? 2 * BKK : 2 * ROWS;
    static constexpr int BYTES = 2 * BKK * ROWS;
    static constexpr int VPR = PITCH / 16;                 // pieces of a row
    static constexpr int LOADS = BYTES / (16 * GTHR);      // per thread and K step
    static constexpr int RSTEP = GTHR / VPR;               // memory rows between a thread's consecutive pieces
    static __device__ __forceinline__ int row(int tid) { return tid / VPR; }                    // of a thread's first piece
    static __device__ __forceinline__ int piece(int tid) {                                      // in memory
        const int r = tid / VPR;
        return (tid % VPR) ^ (KMAJOR ? r / 2 & 7 : 2 * (r & 3) + (r & 8));
    }
    static_assert(RSTEP % 16 == 0 && VPR >= 8 && (KMAJOR || VPR == 16 || VPR == 32), "the permutation is the same for all of a thread's pieces");

    // Offset of a thread's first piece inside a K step.  Row-index-k tiles: threads outside the columns that exist start
    // beyond the descriptor's span (what they would fetch lands in columns that are not stored).
    static __device__ __forceinline__ uint32_t voff(int64_t ld, int left, int tid) {
        return !KMAJOR && piece(tid) * 8 >= left ? 0x80000000u : (uint32_t)row(tid) * (uint32_t)(ld * 2) + (uint32_t)piece(tid) * 16;
    }
    // The memory rows of a whole K step that exist: whatever lies outside is not fetched, without a branch.
    static __device__ __forceinline__ u32x4 span(const bf16_t* origin, int64_t ld, int left) {
        const int rows = left < ROWS ? left : ROWS;
        const uint32_t bytes = KMAJOR ? (uint32_t)(rows - 1) * (uint32_t)(ld * 2) + 2 * BKK : (BKK - 1) * (uint32_t)(ld * 2) + 2 * ROWS;
        const uint64_t a = (uint64_t)origin;
        u32x4 r;
        r[0] = (uint32_t)a;
        r[1] = (uint32_t)(a >> 32) & 0xffffu;
        r[2] = bytes;
        r[3] = 0x00020000u;
        return r;
    }
    // Piece I of a K step, memory -> LDS.  The wave's 64 pieces land at m0 in lane order.  As assembly because the compiler
    // drains every load in flight to LDS before each LDS read it can see; there is no output register, and the step waits for
    // the loads itself.  m0 is a register the compiler reserves for itself: it warns that it may not keep a value of its own
    // there across this statement.  It has none in these kernels; it would with an array that is indexed at run time in
    // registers, or another access straight to LDS, a message or a global barrier: those must not come in here.
    template <int I>
    static __device__ __forceinline__ void load(u32x4 r, int64_t ld, uint32_t voff, uint32_t lds, int w) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds + (uint32_t)(I * 16 * GTHR + w * 1024)), "v"(voff + (uint32_t)(I * RSTEP) * (uint32_t)(ld * 2)), "s"(r)
                     : "memory", "m0");
    }
    // The last, partial K step through registers: k beyond the contraction's end has to read as zero.
    static __device__ __forceinline__ void load_part(const bf16_t* origin, int64_t ld, int left, int k_left, char* lds, int tid) {
        bf16x8 v[LOADS];
        asm volatile("" : "+v"(tid));  // the addresses are worked out here: ahead of the K steps they take 20 to 30 of their registers
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int r = row(tid) + RSTEP * i, c = piece(tid) * 8;
            const bool in = KMAJOR ? (r < left && c < k_left) : (r < k_left && c < left);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] = (__bf16)0.f;
            if (in) v[i] = *(const bf16x8*)(origin + (int64_t)r * ld + c);
        }
#pragma unroll
        for (int i = 0; i < LOADS; ++i) *(bf16x8*)(lds + i * 16 * GTHR + tid * 16) = v[i];
    }
    // MFMA operand: rows r0 .. r0+15 (r0 a multiple of 16), k = 32 ks .. 32 ks+31; lane -> row lane % 16, k 8 (lane / 16) .. + 7
    static __device__ __forceinline__ bf16x8 operand(const char* lds, int r0, int ks, int lane) {
        const int g = lane >> 4, r = lane & 15;
        if (KMAJOR) return *(const bf16x8*)(lds + (r0 + r) * PITCH + (((g ^ (r >> 1)) << 4) ^ (ks << 6)));
        const char* p = lds + (32 * ks + 8 * g + (r >> 2)) * PITCH + (((r0 * 2) ^ (((r >> 2) + 4 * (g & 1)) << 5)) + 8 * (r & 3));  // see frag_tr
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * PITCH));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
};

// 256 x 64 WJ tile, eight waves of 64 x 32 WJ, one workgroup per compute unit.  Two waves share a SIMD: one reads its
// operands while the other multiplies.  The MFMAs are 16 x 16 x 32: the chip runs at its power limit here, and on random
// operands in registers they sustain 2075 TFLOP/s where 32 x 32 x 16 sustains 1846 (half the accumulator traffic; on zeros
// both reach 2450-2470).  A K step is WJ phases of sixteen: all of the wave's A operands (64 rows, 64 k)
// against 32 columns of B; during a phase the next 32 columns are read, during the last one the A operands of the next step,
// each right behind its last use.  So A's buffer is free from the second phase of its step on and B's from the last, and with
// two buffers for A and three for B (all of the LDS at WJ = 4) a load is issued one and a half to two steps before its data
// are read: the trip through the L2 under load takes longer than a step of MFMAs (0.93 us).  With both loaded one step ahead
// the same loop ran at 0.68 of what it reaches without loads (8192 x 8192 x 8192, zeros: 1562 against 2299 TFLOP/s).
// Measured, random operands, against the four waves of 128 x 128 with operands staged through registers that this replaces:
// 8192 x 8192 x 8192 1269 -> 1498 TFLOP/s, 4096 x 2560 -> 10576 876 -> 1047 (672 tiles in three rounds, power-limited clock).
// Barriers: X in front of the second phase (every wave has its A operands: A(t + 2) may come in), Y in front of the last
// (every wave has its B operands and its loads of step t + 1 have landed: B(t + 3) may come in).  At WJ = 2 the two are one,
// and A has three buffers as well.
struct BigCtx {
    const bf16_t* a_org;  // tile origin at k = 0
    const bf16_t* b_org;
    int64_t lda, ldb, a_kstep, b_kstep;
    uint32_t va, vb;      // offsets of the thread's pieces in a K step
    int rows_a, rows_b, K;  // extents left from the tile origin
    int tid, lane, w, wm, wn;
};

template <int N>
__device__ __forceinline__ void wait_and_meet() {  // at most N loads to LDS still under way; every operand read done
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <bool AK, bool BK, int WJ>
struct Big {
    typedef Tile<256, AK> TA;
    typedef Tile<64 * WJ, BK> TB;
    static constexpr int NA = WJ == 2 ? 3 : 2, NB = 3;     // buffers
    static constexpr int LDS = NA * TA::BYTES + NB * TB::BYTES;
    static constexpr int SETS = WJ == 3 ? 3 : 2;           // of B operands: a step starts with set 0
    static constexpr int AHEAD_A = NA, AHEAD_B = NB;       // steps between a load and its use

    char* lds;
    uint32_t lds0;
    int a0, b0;  // buffers of the current step
    f32x4 acc[4][2 * WJ];
    bf16x8 a[4][2], b[SETS][2][2];

    static __device__ __forceinline__ int next(int buf, int n) { return buf + 1 == n ? 0 : buf + 1; }
    __device__ __forceinline__ void read_a(const BigCtx& cx, int buf, int i, int ks) {
        a[i][ks] = TA::operand(lds + buf * TA::BYTES, cx.wm * 64 + i * 16, ks, cx.lane);
    }
    // operand q of phase j: k half q / 2, columns 16 (q % 2) ..
    __device__ __forceinline__ void read_b(const BigCtx& cx, int buf, int set, int j, int q) {
        b[set][q & 1][q >> 1] = TB::operand(lds + NA * TA::BYTES + buf * TB::BYTES, cx.wn * 32 * WJ + j * 32 + (q & 1) * 16, q >> 1, cx.lane);
    }
    static __device__ __forceinline__ u32x4 span_a(const BigCtx& cx, int k0) {
        return TA::span(cx.a_org + (int64_t)k0 * cx.a_kstep, cx.lda, cx.rows_a);
    }
    static __device__ __forceinline__ u32x4 span_b(const BigCtx& cx, int k0) {
        return TB::span(cx.b_org + (int64_t)k0 * cx.b_kstep, cx.ldb, cx.rows_b);
    }
    template <int I>
    __device__ __forceinline__ void load_a(const BigCtx& cx, u32x4 s, int buf) {
        TA::template load<I>(s, cx.lda, cx.va, lds0 + buf * TA::BYTES, cx.w);
    }
    template <int I>
    __device__ __forceinline__ void load_b(const BigCtx& cx, u32x4 s, int buf) {
        if constexpr (I < TB::LOADS) TB::template load<I>(s, cx.ldb, cx.vb, lds0 + NA * TA::BYTES + buf * TB::BYTES, cx.w);
    }
    // A whole or partial K step at k0, or nothing beyond the end.
    __device__ __forceinline__ void load_step_a(const BigCtx& cx, int k0, int buf, bool direct) {
        if (k0 >= cx.K) return;
        if (direct && k0 + BKK <= cx.K) {
            const u32x4 s = span_a(cx, k0);
            load_a<0>(cx, s, buf); load_a<1>(cx, s, buf); load_a<2>(cx, s, buf); load_a<3>(cx, s, buf);
        } else {
            TA::load_part(cx.a_org + (int64_t)k0 * cx.a_kstep, cx.lda, cx.rows_a, cx.K - k0, lds + buf * TA::BYTES, cx.tid);
        }
    }
    __device__ __forceinline__ void load_step_b(const BigCtx& cx, int k0, int buf, bool direct) {
        if (k0 >= cx.K) return;
        if (direct && k0 + BKK <= cx.K) {
            const u32x4 s = span_b(cx, k0);
            load_b<0>(cx, s, buf); load_b<1>(cx, s, buf); load_b<2>(cx, s, buf); load_b<3>(cx, s, buf);
        } else {
            TB::load_part(cx.b_org + (int64_t)k0 * cx.b_kstep, cx.ldb, cx.rows_b, cx.K - k0, lds + NA * TA::BYTES + buf * TB::BYTES, cx.tid);
        }
    }

    // Fills the buffers and reads the first operands.
    __device__ __forceinline__ void start(const BigCtx& cx, bool direct) {
        a0 = b0 = 0;
        load_step_a(cx, 0, 0, direct);
        load_step_b(cx, 0, 0, direct);
        load_step_a(cx, BKK, 1, direct);
        load_step_b(cx, BKK, 1, direct);
        if (NA == 3) load_step_a(cx, 2 * BKK, 2, direct);
        load_step_b(cx, 2 * BKK, 2, direct);
        if (direct && 3 * BKK <= cx.K) wait_and_meet<(NA - 1) * TA::LOADS + 2 * TB::LOADS>();
        else wait_and_meet<0>();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            read_b(cx, 0, 0, 0, q);
            read_a(cx, 0, q, 0);
            read_a(cx, 0, q, 1);
        }
    }

    // One K step.  STEADY: the steps whose loads it issues exist and are whole; straight-line code.
    template <bool STEADY>
    __device__ __forceinline__ void step(const BigCtx& cx, int k0, bool direct) {
        const bool more = STEADY || k0 + BKK < cx.K;
        const int a1 = next(a0, NA), b1 = next(b0, NB);
        u32x4 sa, sb;
        if (STEADY) {
            sa = span_a(cx, k0 + AHEAD_A * BKK);
            sb = span_b(cx, k0 + AHEAD_B * BKK);
        }
#pragma unroll
        for (int j = 0; j < WJ; ++j) {
            constexpr bool ONE = WJ == 2;
            const bool last = j == WJ - 1, first_free = j == 1;
            if (first_free && !ONE) {  // X
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                if (!STEADY) load_step_a(cx, k0 + AHEAD_A * BKK, a0, direct);
            }
            if (last) {                // Y
                if (STEADY) wait_and_meet<TA::LOADS + TB::LOADS>();
                else wait_and_meet<0>();
                if (!STEADY) {
                    if (ONE) load_step_a(cx, k0 + AHEAD_A * BKK, a0, direct);
                    load_step_b(cx, k0 + AHEAD_B * BKK, b0, direct);
                }
            }
            // the last phase issues the most besides its MFMAs: the wave that is in it goes first (2 % of the product)
            if (j == 0) __builtin_amdgcn_s_setprio(0);
            if (last) __builtin_amdgcn_s_setprio(1);
            const int set = j % SETS, nset = last ? 0 : (j + 1) % SETS;
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const int ks = m >> 3, i = (m >> 1) & 3, jj = m & 1;
                acc[i][2 * j + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[set][jj][ks], a[i][ks], acc[i][2 * j + jj], 0, 0, 0);
                if (m < 8 && (m & 1) == 0 && (!last || more)) read_b(cx, last ? b1 : b0, nset, last ? 0 : j + 1, m >> 1);
                if (last && more && jj == 1) read_a(cx, a1, i, ks);  // its last use is the MFMA above
                if (STEADY && first_free) {
                    if (m == 1) load_a<0>(cx, sa, a0);
                    if (m == 5) load_a<1>(cx, sa, a0);
                    if (m == 9) load_a<2>(cx, sa, a0);
                    if (m == 13) load_a<3>(cx, sa, a0);
                }
                if (STEADY && last) {
                    if (m == 0) load_b<0>(cx, sb, b0);
                    if (m == 4) load_b<1>(cx, sb, b0);
                    if (m == 8) load_b<2>(cx, sb, b0);
                    if (m == 12) load_b<3>(cx, sb, b0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        a0 = a1;
        b0 = b1;
    }
};

extern __shared__ __attribute__((aligned(1024))) char lds[];  // the K steps in flight; at the end the patches of the result

template <bool AK, bool BK, int WJ>
__device__ __forceinline__ void gemm_tile(const GemmParams& gp, int id) {
    constexpr int BM = 256, BN = 64 * WJ;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    tile_of(gp, id, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    typedef Big<AK, BK, WJ> Gemm;
    Gemm G;
    f32x4 (&acc)[4][2 * WJ] = G.acc;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2 * WJ; ++j) acc[i][j] = (f32x4)(0.f);
    G.lds = lds;
    G.lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    const bool interior = m0 + BM <= gp.M && n0 + BN <= gp.N;
    BigCtx cx;
    cx.a_org = AK ? gp.A + (int64_t)m0 * gp.lda : gp.A + m0;
    cx.b_org = BK ? gp.B + (int64_t)n0 * gp.ldb : gp.B + n0;
    cx.lda = gp.lda;
    cx.ldb = gp.ldb;
    cx.a_kstep = AK ? 1 : gp.lda;  // elements per unit of k
    cx.b_kstep = BK ? 1 : gp.ldb;
    cx.rows_a = gp.M - m0;
    cx.rows_b = gp.N - n0;
    cx.va = Gemm::TA::voff(gp.lda, cx.rows_a, tid);
    cx.vb = Gemm::TB::voff(gp.ldb, cx.rows_b, tid);
    cx.K = gp.K;
    cx.tid = tid;
    cx.lane = tid & 63;
    cx.w = w;
    cx.wm = w >> 1;
    cx.wn = w & 1;
    const int lane = cx.lane, wm = cx.wm, wn = cx.wn;
    // strides beyond what 32-bit offsets reach: every step goes through registers
    const bool direct = gp.lda <= MAX_LD && gp.ldb <= MAX_LD;
    G.start(cx, direct);
    int k0 = 0;
    if (direct)
        for (; k0 + (Gemm::AHEAD_B + 1) * BKK <= gp.K; k0 += BKK) G.template step<true>(cx, k0, true);
    for (; k0 < gp.K; k0 += BKK) G.template step<false>(cx, k0, direct);

    if (gp.c_f32) {
        store_acc_f32<WJ>(gp, acc, m0 + wm * 64, n0 + wn * 32 * WJ, lane);
        return;
    }
    // bf16 result: through LDS (every wave has left its last buffer behind the barrier), so that
    // a store instruction writes whole row pieces (256 bytes at WJ = 4) instead of 32 scattered 16-byte ones.  Each wave
    // transposes its own 64 x 32 WJ tile in a private patch: lane -> row lane % 16, four consecutive columns
    // per tile (see store_acc_f32) on the way in, 16-byte vectors of a row on the way out.
    __syncthreads();
    constexpr int VPR = 4 * WJ, EPITCH = 16 * VPR + 16;  // vectors per row
    char* patch = lds + w * (64 * EPITCH);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2 * WJ; ++j)
            *(bf16x4*)(patch + (i * 16 + (lane & 15)) * EPITCH + (j * 16 + (lane >> 4) * 4) * 2) = __builtin_convertvector(acc[i][j], bf16x4);
#pragma unroll
    for (int it = 0; it < VPR; ++it) {
        const int v = it * 64 + lane, r = v / VPR, c = v % VPR, row = m0 + wm * 64 + r, col = n0 + wn * 32 * WJ + c * 8;
        const bf16x8 o = *(const bf16x8*)(patch + r * EPITCH + c * 16);
        if (interior || (row < gp.M && col < gp.N)) *(bf16x8*)((__bf16*)gp.C + (int64_t)row * gp.ldc + col) = o;
    }
}

template <int WJ>
__global__ __launch_bounds__(GTHR, 1) void k_gemm_big(GemmParams gp) {
    gemm_tile<true, true, WJ>(gp, blockIdx.x);
}

// The first columns in tiles of one width, which fill their rounds, the others in tiles of a narrower one: workgroups first .. run these.
template <int W1, int W2>
__global__ __launch_bounds__(GTHR, 1) void k_gemm_mixed(GemmParams p1, GemmParams p2, int first) {
    if ((int)blockIdx.x < first) gemm_tile<true, true, W1>(p1, blockIdx.x);
    else gemm_tile<true, true, W2>(p2, blockIdx.x - first);
}

// The gradient products of a call, of the input (64 WX columns a tile) and of the weights (64 WW), in one launch: workgroups
// first .. run the second.  They are independent (both read dout; they write dx and dw), and one alone often leaves compute
// units idle: a segment of 4096 rows gives the input gradient of the 2.7B block's input projection 160 tiles for 256 units.
// As two launches on two streams they met only behind a fork and a join, some 20 us a pair, and in whatever order the queues
// were served: us at 4096 rows, two launches -> one, 2560 <-> 10576 375 -> 363, 2560 <-> 5120 227 -> 182, 1024 <-> 4384 95 -> 90,
// 1024 <-> 2048 73 -> 49; 600 rows 154 -> 145, 81 -> 50, 61 -> 49, 40 -> 16.
// A tile of each kind in one kernel fits the registers (240; with the addresses of a partial K step worked out ahead of the steps it
// did not, see load_part).
template <int WX, int WW>
__global__ __launch_bounds__(GTHR, 1) void k_gemm_grads(GemmParams px, GemmParams pw, int dw_first, int first) {
    const bool second = (int)blockIdx.x >= first;
    const int id = second ? blockIdx.x - first : blockIdx.x;
    if (second == (dw_first != 0)) gemm_tile<true, false, WX>(px, id);
    else gemm_tile<false, false, WW>(pw, id);
}

bool ok_ptr(const void* p) { return p && ((uintptr_t)p & 15) == 0; }

template <bool AK, bool BK, int WJ>
constexpr int big_lds() {
    constexpr int PATCHES = 8 * 64 * (64 * WJ + 16);
    return Big<AK, BK, WJ>::LDS > PATCHES ? Big<AK, BK, WJ>::LDS : PATCHES;
}

// The kernels use more dynamic LDS than the default limit; `raised`: per device.
hipError_t allow_lds(const void* kernel, int bytes, bool (&raised)[64]) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (raised[dev]) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    raised[dev] = e == hipSuccess;
    return e;
}

int set_tiles(GemmParams& gp, int wj) {
    gp.tiles_m = (gp.M + 255) / 256;
    gp.tiles_n = (gp.N + 64 * wj - 1) / (64 * wj);
    return gp.tiles_m * gp.tiles_n;
}

template <int WJ>
hipError_t launch_big(GemmParams gp, hipStream_t st) {
    constexpr int LDS = big_lds<true, true, WJ>();
    static bool raised[64];
    const hipError_t e = allow_lds((const void*)k_gemm_big<WJ>, LDS, raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_gemm_big<WJ>), dim3(set_tiles(gp, WJ)), dim3(GTHR), LDS, st, gp);
    return hipGetLastError();
}

template <int W1, int W2>
hipError_t launch_mixed(GemmParams gp, int n1, hipStream_t st) {
    constexpr int L1 = big_lds<true, true, W1>(), L2 = big_lds<true, true, W2>(), LDS = L1 > L2 ? L1 : L2;  // (128 columns have three buffers of both)
    static bool raised[64];
    const hipError_t e = allow_lds((const void*)k_gemm_mixed<W1, W2>, LDS, raised);
    if (e != hipSuccess) return e;
    GemmParams p2 = gp;
    gp.N = n1;
    p2.N -= n1;
    p2.B += (int64_t)n1 * gp.ldb;
    p2.C = (bf16_t*)gp.C + n1;
    const int t1 = set_tiles(gp, W1), t2 = set_tiles(p2, W2);
    hipLaunchKernelGGL((k_gemm_mixed<W1, W2>), dim3(t1 + t2), dim3(GTHR), LDS, st, gp, p2, t1);
    return hipGetLastError();
}

// Without dx or dw: the other alone.
template <int WX, int WW>
hipError_t launch_grads(GemmParams px, GemmParams pw, bool dx, bool dw, bool dw_first, hipStream_t st) {
    constexpr int LX = big_lds<true, false, WX>(), LW = big_lds<false, false, WW>(), LDS = LX > LW ? LX : LW;
    static bool raised[64];
    const hipError_t e = allow_lds((const void*)k_gemm_grads<WX, WW>, LDS, raised);
    if (e != hipSuccess) return e;
    const int tx = dx ? set_tiles(px, WX) : 0, tw = dw ? set_tiles(pw, WW) : 0;
    hipLaunchKernelGGL((k_gemm_grads<WX, WW>), dim3(tx + tw), dim3(GTHR), LDS, st, px, pw, dw_first, dw_first ? tw : tx);
    return hipGetLastError();
}

// Which tile width (64 WJ columns).  A compute unit holds one workgroup, so a product takes ceil(tiles / 256) rounds, and
// a round with narrower tiles is cheaper, though by less than its share of the arithmetic (more LDS and cache traffic per
// MFMA).  Cost of a round against 256 columns, measured over 100 ... 16384 rows at widths 768 ... 2560: forward product
// 0.82 at 192 columns and 0.61-0.71 at 128.
// What it gives (us at 128 / 192 / 256 columns): 4096 x 5120 -> 2560: 117 / 84 / 92; 1905 x 2560 -> 10576: 97 / 90 / 105;
// 1905 x 5120 -> 2560: 56 / 72 / 87; 600 x 1024 -> 4384: 16 / 20 / 23.
constexpr int64_t UNITS = 256;
int64_t tile_count(const GemmParams& gp, int wj) { return (int64_t)((gp.M + 255) / 256) * ((gp.N + 64 * wj - 1) / (64 * wj)); }
constexpr int WIDTH_PCT[5] = {0, 0, 68, 83, 100};  // of a K step, by WJ

// Columns up to n1 in tiles of width w, the others (where n1 < N) in tiles of the next narrower one.  One width leaves the last round as
// empty as it falls out: 4096 x 2560 -> 10576 is 2.6 rounds of 256 columns and takes three; two rounds of them and one of 192 columns for
// the rest are full.  The units that the wide tiles leave idle in their last round take a narrow one there.  us with one width -> with two:
// 4096 x 2560 -> 10576 190 -> 187, 8192 x 2560 -> 10576 366 -> 350, 8192 x 5120 -> 2560 182 -> 174, 4096 x 1024 -> 4384 42 -> 38.
struct ForwardPlan {
    int w, n1;
};
ForwardPlan forward_plan(const GemmParams& gp) {
    ForwardPlan best = {4, gp.N};
    int64_t t = INT64_MAX;
    for (int w = 4; w >= 2; --w) {
        const int64_t c = (tile_count(gp, w) + UNITS - 1) / UNITS * WIDTH_PCT[w];
        if (c < t) t = c, best = {w, gp.N};
    }
    if (tile_count(gp, 4) > 50 * UNITS) return best;
    t -= t / 50;  // for less than 2 % (and so in more than 50 rounds) it is not worth a second kind
    const int64_t tm = (gp.M + 255) / 256;
    for (int w1 = 4; w1 > 2; --w1)
        for (int64_t r = (gp.N - 1) / (64 * w1) * tm / UNITS; r > 0; --r) {
            const int64_t n1 = UNITS * r / tm * 64 * w1, spare = UNITS * r - UNITS * r / tm * tm;
            if (n1 <= 0 || n1 >= gp.N) continue;
            const int64_t rest = tm * ((gp.N - n1 + 64 * (w1 - 1) - 1) / (64 * (w1 - 1))) - spare;
            const int64_t c = r * WIDTH_PCT[w1] + (rest > 0 ? (rest + UNITS - 1) / UNITS * WIDTH_PCT[w1 - 1] : 0);
            if (c < t) t = c, best = {w1, (int)n1};
        }
    return best;
}

// Widths of the gradients' products: 4 or 2 (rows of 192 columns do not permute by an exclusive or, see Tile).  A tile takes
// its K steps and what surrounds them: about four steps' time, and twenty where fp32 results are added to (256 x 256 of them:
// 512 KB in and out for every compute unit at once), half of that at 128 columns.  Side by side the two products fill the
// machine together: while all tiles are resident at once the longer chain counts; else the work spread over the machine plus
// two fifths of a chain of ragged end, and no less than a short tile in front of a long one.  Over six pairs of widths from
// 768 to 10576 and 100 ... 16384 rows the rule is 1.5 % off the best of the four combinations (6 % with the K steps alone).
// The product of the longer tiles goes first: the others then fill the units that its last round leaves idle, instead of the
// long ones running on alone.  2560 <-> 10576 (longer: the input's), 4096 rows: 363 us, the other way round 424; 2560 <-> 5120
// (longer: the weights'), 4096 rows 182, the other way round 217.
// Both at 256 columns -> as chosen: 2560 <-> 10576, 200 rows 185 -> 121 us; 1024 <-> 4384, 4096 rows 92 -> 90.
int64_t tile_cost(const GemmParams& gp, int wj) {
    const int64_t around = gp.c_f32 ? (wj == 4 ? 2000 : 1100) : (wj == 4 ? 400 : 200);
    return (int64_t)((gp.K + BKK - 1) / BKK) * (wj == 4 ? 100 : 66) + around;
}
void backward_widths(const GemmParams* dx, const GemmParams* dw, int& wx, int& ww, bool& dw_first) {
    int64_t best = INT64_MAX;
    for (int a = 4; a >= 2; a -= 2)
        for (int b = 4; b >= 2; b -= 2) {
            const int64_t ta = dx ? tile_count(*dx, a) : 0, ca = dx ? tile_cost(*dx, a) : 0;
            const int64_t tb = dw ? tile_count(*dw, b) : 0, cb = dw ? tile_cost(*dw, b) : 0;
            int64_t t;
            if (!dx || !dw) {
                t = (ta + UNITS - 1) / UNITS * ca + (tb + UNITS - 1) / UNITS * cb;
            } else {
                const int64_t longer = ca > cb ? ca : cb, spread = (ta * ca + tb * cb) / UNITS + longer * 2 / 5;
                t = ta + tb <= UNITS ? longer : (spread > ca + cb ? spread : ca + cb);
            }
            if (t < best) best = t, wx = a, ww = b, dw_first = cb > ca;
        }
}

int check(int64_t rows, int32_t in_dim, int32_t out_dim, int64_t ldx, int64_t ldo) {
    if (rows < 0 || rows > 0x7fffffff || in_dim <= 0 || out_dim <= 0) return SSD_ERR_SHAPE;
    if ((in_dim | out_dim) & 7) return SSD_ERR_DIVISIBILITY;  // 16-byte vectors of bf16
    if ((ldx && (ldx < in_dim || (ldx & 7))) || (ldo && (ldo < out_dim || (ldo & 7)))) return SSD_ERR_SHAPE;
    const int64_t tiles = ((rows + 255) / 256) * (((int64_t)out_dim + 127) / 128);
    const int64_t tiles_w = (((int64_t)out_dim + 255) / 256) * (((int64_t)in_dim + 127) / 128);
    if (tiles > 0x7fffffff || tiles_w > 0x7fffffff) return SSD_ERR_SHAPE;
    return SSD_OK;
}

}  // namespace
}  // namespace ssdk

using namespace ssdk;

extern "C" int ssd_linear_fwd(int64_t rows, int32_t in_dim, int32_t out_dim, const void* x, int64_t x_row_stride,
                              const void* w, void* out, int64_t out_row_stride, void* hip_stream) {
    const int rc = check(rows, in_dim, out_dim, x_row_stride, out_row_stride);
    if (rc != SSD_OK) return rc;
    if (rows == 0) return SSD_OK;
    if (!x || !w || !out) return SSD_ERR_NULL;
    if (!ok_ptr(x) || !ok_ptr(w) || !ok_ptr(out)) return SSD_ERR_ARG;
    if (rows <= FEW_ROWS) {  // a token or a few: bound by reading w once, not by the matrix cores
        FewRowsJob j;
        memset(&j, 0, sizeof(j));
        j.rows = (int)rows;
        j.K = in_dim;
        j.N = out_dim;
        j.x = x;
        j.ldx = x_row_stride ? x_row_stride : in_dim;
        j.w = w;
        j.out = out;
        j.ldo = out_row_stride ? out_row_stride : out_dim;
        if (few_rows_supported(j)) return launch_linear_few_rows(j, (hipStream_t)hip_stream) == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
    }
    GemmParams gp;
    memset(&gp, 0, sizeof(gp));
    gp.A = (const bf16_t*)x;   // [rows, in]   k-major
    gp.B = (const bf16_t*)w;   // [out, in]    k-major
    gp.C = out;
    gp.lda = x_row_stride ? x_row_stride : in_dim;
    gp.ldb = in_dim;
    gp.ldc = out_row_stride ? out_row_stride : out_dim;
    gp.M = (int)rows;
    gp.N = out_dim;
    gp.K = in_dim;
    const ForwardPlan f = forward_plan(gp);
    hipStream_t st = (hipStream_t)hip_stream;
    hipError_t e;
    if (f.n1 < gp.N) e = f.w == 4 ? launch_mixed<4, 3>(gp, f.n1, st) : launch_mixed<3, 2>(gp, f.n1, st);
    else e = f.w == 4 ? launch_big<4>(gp, st) : f.w == 3 ? launch_big<3>(gp, st) : launch_big<2>(gp, st);
    return e == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}

extern "C" int ssd_linear_bwd(int64_t rows, int32_t in_dim, int32_t out_dim, const void* x, int64_t x_row_stride,
                              const void* w, const void* dout, int64_t dout_row_stride, void* dx, int64_t dx_row_stride,
                              float* dw, uint32_t flags, void* hip_stream) {
    int rc = check(rows, in_dim, out_dim, x_row_stride, dout_row_stride);
    if (rc != SSD_OK) return rc;
    if (dx_row_stride && (dx_row_stride < in_dim || (dx_row_stride & 7))) return SSD_ERR_SHAPE;
    if (flags & ~(uint32_t)SSD_FLAG_ACCUM_PARAM) return SSD_ERR_ARG;
    hipStream_t st = (hipStream_t)hip_stream;
    const int accumulate = (flags & SSD_FLAG_ACCUM_PARAM) ? 1 : 0;
    if (rows == 0) {
        if (dw && !accumulate && launch_fill_zero(dw, (size_t)out_dim * in_dim, st) != hipSuccess) return SSD_ERR_LAUNCH;
        return SSD_OK;
    }
    if (!dout || (dx && !w) || (dw && !x)) return SSD_ERR_NULL;
    if (!ok_ptr(dout) || (dx && (!ok_ptr(dx) || !ok_ptr(w))) || (dw && (!ok_ptr(x) || !ok_ptr(dw)))) return SSD_ERR_ARG;
    const int64_t ldd = dout_row_stride ? dout_row_stride : out_dim;
    GemmParams px, pw;
    // dx[rows, in] = dout[rows, out] w[out, in]: contraction over out; w holds it as the row index
    memset(&px, 0, sizeof(px));
    px.A = (const bf16_t*)dout;
    px.B = (const bf16_t*)w;
    px.C = dx;
    px.lda = ldd;
    px.ldb = in_dim;
    px.ldc = dx_row_stride ? dx_row_stride : in_dim;
    px.M = (int)rows;
    px.N = in_dim;
    px.K = out_dim;
    // dw[out, in] = dout^T x: contraction over the rows, the row index of both operands
    memset(&pw, 0, sizeof(pw));
    pw.A = (const bf16_t*)dout;
    pw.B = (const bf16_t*)x;
    pw.C = dw;
    pw.lda = ldd;
    pw.ldb = x_row_stride ? x_row_stride : in_dim;
    pw.ldc = in_dim;
    pw.M = out_dim;
    pw.N = in_dim;
    pw.K = (int)rows;
    pw.c_f32 = 1;
    pw.accumulate = accumulate;
    if (!dx && !dw) return SSD_OK;
    int wx, ww;
    bool dw_first;
    backward_widths(dx ? &px : nullptr, dw ? &pw : nullptr, wx, ww, dw_first);
    hipError_t e;
    if (wx == 4) e = ww == 4 ? launch_grads<4, 4>(px, pw, dx, dw, dw_first, st) : launch_grads<4, 2>(px, pw, dx, dw, dw_first, st);
    else e = ww == 4 ? launch_grads<2, 4>(px, pw, dx, dw, dw_first, st) : launch_grads<2, 2>(px, pw, dx, dw, dw_first, st);
    return e == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}

// Calibration: what the matrix cores deliver when nothing else is in the way -- every wave issues
// `iters` rounds of sixteen independent 32 x 32 x 16 bf16 MFMAs on registers (no memory traffic), four
// waves per compute unit over the whole chip.  bench.py times it (--calibrate-mfma) to put the sustained
// clock of the matrix pipes next to the nominal peak.
namespace ssdk {
namespace {
__global__ __launch_bounds__(256, 1) void k_mfma_peak(int iters, float* sink) {
    f32x16 acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = zero16();
    bf16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        a[e] = (__bf16)(float)(threadIdx.x & 3);
        b[e] = (__bf16)(float)(e & 1);
    }
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = mfma(a, b, acc[i]);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += acc[i][0];
    if (s == -1.f) sink[0] = s;  // never true: keeps the products alive
}
}  // namespace
}  // namespace ssdk

extern "C" int ssd_prof_mfma_peak(int32_t iters, int32_t workgroups, float* sink, void* hip_stream) {
    if (iters <= 0 || workgroups <= 0 || !sink) return SSD_ERR_ARG;
    hipLaunchKernelGGL(k_mfma_peak, dim3(workgroups), dim3(256), 0, (hipStream_t)hip_stream, iters, sink);
    return hipGetLastError() == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}

// Clock probe: one wave that sleeps until the constant 100 MHz counter has advanced by `ticks` and reports how
// many shader-clock cycles went by meanwhile.  Launched on a second stream next to a kernel under test it
// shows the clock that kernel really runs at (the power management lowers it under heavy load), which is what
// a cycle count or a fraction of the nominal peak has to be read against.
namespace ssdk {
namespace {
__global__ __launch_bounds__(64) void k_clock_probe(unsigned long long* out, unsigned long long ticks) {
    const unsigned long long w0 = wall_clock64(), c0 = clock64();
    unsigned long long w = w0;
    // an iteration takes about a microsecond (100 ticks): the time limit ends the loop long before the count does
    for (unsigned long long i = 0; i < ticks && w - w0 < ticks; ++i) {
        __builtin_amdgcn_s_sleep(32);
        w = wall_clock64();
    }
    if (threadIdx.x == 0) {
        out[0] = w - w0;
        out[1] = clock64() - c0;
    }
}
}  // namespace
}  // namespace ssdk

extern "C" int ssd_prof_clock_probe(uint64_t ticks, uint64_t* out, void* hip_stream) {
    if (!out || ticks == 0 || ticks > 100000000ull) return SSD_ERR_ARG;  // at most a second
    hipLaunchKernelGGL(k_clock_probe, dim3(1), dim3(64), 0, (hipStream_t)hip_stream, (unsigned long long*)out, (unsigned long long)ticks);
    return hipGetLastError() == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
}
