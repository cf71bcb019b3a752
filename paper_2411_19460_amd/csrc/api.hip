// C-ABI entry points for one SSD layer: argument validation, workspace partitioning and the
// segment loops of the MA-GC sequence axis (paper Sec. 3.2/3.3, Alg. 1 and Alg. 2).
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "ssd_internal.h"

namespace ssdk {

inline size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

int pick_split(int heads_per_group, int64_t base, int target) {
    for (int ns = 1; ns <= heads_per_group; ++ns)
        if (heads_per_group % ns == 0 && base * ns >= target) return ns;
    return heads_per_group;
}

// As above for a launch that has the machine to itself: the slices that end soonest.  A compute unit holds per_unit of the
// workgroups (1 or 2) and a launch goes by in rounds of them; a workgroup takes `prologue` before its first head (both in
// hundredths of a head), and with a unit to itself where two fit it walks a head in two thirds of the time.  Those are figures
// of chunks of 256.  At 64, where a unit holds more and shorter workgroups, counting them so is still the better rule: forward,
// us, as above -> this, 2000 tokens of 80 heads 64 -> 56, 4000 of 80 111 -> 90, 10007 of 24 / 32 / 64 / 80 92 / 112 / 209 / 263 ->
// 79 / 95 / 167 / 210, backward 287 -> 267 and 281 / 345 / 710 / 882 -> 260 / 310 / 628 / 794; no longer, but for
// what the runs of one side differ by, at any of 35 sizes, 500 ... 60000 tokens.
// The slices need not divide the heads (only those that do -> any, forward + backward: 3333 tokens of 64 heads 185 -> 163 us;
// prefill of 10007 tokens of 80 heads 132.3 -> 127.7).
int pick_rounds(int heads_per_group, int64_t base, int per_unit, int prologue) {
    constexpr int64_t UNITS = 256;
    int best = 1;
    int64_t least = INT64_MAX;
    for (int ns = 1; ns <= heads_per_group; ++ns) {
        const int64_t n = base * ns, hps = (heads_per_group + ns - 1) / ns;  // of the longer slices
        const int64_t t = n <= UNITS && per_unit == 2 ? 65 * hps + prologue : (n + UNITS * per_unit - 1) / (UNITS * per_unit) * (100 * hps + prologue);
        if (t < least) least = t, best = ns;
    }
    return best;
}

// Returns SSD_OK and fills d, or the validation error.
int check_shape(const ssd_shape_t* sh, Dims* d) {
    if (!sh) return SSD_ERR_NULL;
    if (sh->dtype != SSD_F32 && sh->dtype != SSD_BF16) return SSD_ERR_DTYPE;
    if (sh->batch <= 0 || sh->seqlen < 0 || sh->nheads <= 0 || sh->headdim <= 0 || sh->ngroups <= 0 ||
        sh->dstate <= 0 || sh->chunk <= 0)
        return SSD_ERR_SHAPE;
    if (sh->chunk > 1024 || sh->headdim > 256 || sh->dstate > 256) return SSD_ERR_SHAPE;
    if (sh->batch > 65535 || sh->nheads > 65535) return SSD_ERR_SHAPE;
    if (sh->nheads % sh->ngroups != 0) return SSD_ERR_DIVISIBILITY;
    if (sh->seqlen > 0) {
        if (sh->segment <= 0) return SSD_ERR_SHAPE;
        if (sh->segment % sh->chunk != 0) return SSD_ERR_DIVISIBILITY;
    }
    d->Bt = sh->batch;
    d->L = sh->seqlen;
    d->s = sh->seqlen > 0 ? sh->segment : 0;
    d->H = sh->nheads;
    d->P = sh->headdim;
    d->G = sh->ngroups;
    d->N = sh->dstate;
    d->Q = sh->chunk;
    d->hpg = d->H / d->G;
    d->nc = d->nc_seg = sh->seqlen > 0 ? (int)(sh->segment / sh->chunk) : 0;
    d->nseg = sh->seqlen > 0 ? (sh->seqlen + sh->segment - 1) / sh->segment : 0;
    d->F = d->nl = 1;
    d->dg_f32 = false;
    d->nspan = d->nseg;
    d->nct = (sh->seqlen + sh->chunk - 1) / sh->chunk;
    d->bf16 = sh->dtype == SSD_BF16;
    d->esz = d->bf16 ? 2 : 4;
    d->xs_b = sh->x_batch_stride ? sh->x_batch_stride : d->L * d->H * d->P;
    d->dts_b = sh->dt_batch_stride ? sh->dt_batch_stride : d->L * d->H;
    d->bcs_b = sh->bc_batch_stride ? sh->bc_batch_stride : d->L * d->G * d->N;
    d->reset = sh->seq_reset;
    if (d->xs_b < d->L * d->H * d->P || d->dts_b < d->L * d->H || d->bcs_b < d->L * d->G * d->N) return SSD_ERR_SHAPE;
    // every launch keeps its largest grid dimension below 2^31
    const int64_t blocks = d->Bt * (int64_t)d->nc * d->H * 2;
    if (blocks >= ((int64_t)1 << 31) || (int64_t)sh->segment / sh->chunk >= ((int64_t)1 << 24)) return SSD_ERR_SHAPE;
    return SSD_OK;
}

namespace {
// Into how many slices the heads of a group are cut for the partial sums of a span of nc chunks: enough workgroups for the
// machine, in the place a span of whole segments takes.  That place is what the workspace holds (slots), or less for a span
// too short to fill it even with a slice per head: it never shrinks as a sequence gets longer.
struct HeadSlices {
    int hpg, most, target;
    int64_t per;   // workgroups per chunk and slice
    int64_t room;  // (chunk, slice) pairs of a span of whole segments
    HeadSlices(const Dims& d, int most, int64_t per, int target) : hpg(d.hpg), most(most < d.hpg ? most : d.hpg), target(target), per(per), room(INT64_MAX) {
        const int64_t full = (int64_t)d.F * d.nc_seg;
        room = full * split(full);
    }
    int split(int64_t nc) const {
        if (nc <= 0) return 1;
        const int64_t fits = room / nc;
        int ns = pick_split(hpg, nc * per, target);
        ns = ns < most ? ns : most;
        ns = ns < fits ? ns : (int)fits;
        while (hpg % ns) --ns;
        return ns;
    }
    int64_t slots(int64_t nc) const { return nc * most < room ? nc * most : room; }
};
// shape-generic kernels: 64 x 64 tiles, several workgroups per compute unit; the last pass adds the slices up in registers
HeadSlices dg_slices(const Dims& d, bool mfma, int wg_target) {
    const int64_t nt = (d.Q + 63) / 64, bg = d.Bt * d.G;
    return mfma ? HeadSlices(d, d.hpg, bg, wg_target) : HeadSlices(d, GENERIC_SLICES, bg * (nt * (nt + 1) / 2), 256);
}
HeadSlices part_slices(const Dims& d, bool mfma, int wg_target) {
    const int64_t nt = (d.Q + 63) / 64, nn = (d.N + 63) / 64, bg = d.Bt * d.G;
    return mfma ? HeadSlices(d, d.hpg, bg * 2, wg_target) : HeadSlices(d, GENERIC_SLICES, bg * 2 * nt * nn, 256);
}
// Room for the partial sums of dG of a span, in bf16 chunks of scores: one per head slice, two where they are fp32 (generic
// kernels, and fit_splits: of at most half a round of slices, at chunks of 256 mostly no more than the general rule's bf16 ones;
// at chunks of 128, where a round is twice as many, there is room for those of any one round).
int64_t dg_places(const Dims& d, bool mfma, int wg_target) {
    const int64_t bg = d.Bt * d.G, all = 2 * bg * d.nc * d.hpg;
    const int64_t n = bg * dg_slices(d, mfma, wg_target).slots(d.nc) * (mfma && !d.dg_f32 ? 1 : 2);
    if (!mfma || d.Q != 128 || wg_target < 256 || n >= 512) return n;
    return all < 512 ? (n > all ? n : all) : 512;
}
}  // namespace

// Slices of the three head-walking passes of the backward sweep (one launch, chunks of 128 and 256) for sp's span of the sequence.
// A compute unit holds one of their workgroups, two at chunks of 128.  With the machine to itself such a launch ends soonest
// when all its workgroups fit in one round, if slices can be found that make them about equally long: what a workgroup pays
// around its heads (fetching the scores, storing the partial sums) is paid once, and there are fewer partial sums to write
// and add up.  Otherwise every pass gets a workgroup per compute unit and the three alternate.  Slices (dx, dG, head sums) by
// this rule, 32 chunks of 24 heads: (8, 8, 4) -> (3, 3, 1): 75.2 -> 63.6 us, and the finalisation 19.0 -> 13.6; 16 chunks of
// 80 heads, (16, 16, 8) -> (5, 5, 2): 114 -> 103 and 19.1 -> 14.2.
// The slices' partial sums of dG are bf16 in the general rule, and rounded once more when they have been added up.  Sums of two
// to seven such numbers often lie halfway between two others, so that fewer slices alone take dB and dC further from 64 bits
// (eight -> three of 24 heads: 2.90e-3 -> 2.93e-3).  In one round they are therefore fp32 wherever there is room, 2.41e-3, at 2 us
// of 118 for 8192 tokens of 24 heads (chunks of 128: 1.5 of 67-79, 1920 tokens of 24 heads and 2944 of 8), and of two choices that
// end together the one with fp32 sums is taken (31 chunks of 48 heads, forward and backward: 284 -> 271); bf16 only for as many
// slices as the general rule's.  Likewise fp32 in a span that lanes would cut into more slices (plan_dims).
void fit_splits(SegParams& sp, const Dims& d, bool mfma, int wg_target) {
    const int64_t nc = sp.nc;
    const int a0 = dg_slices(d, mfma, wg_target).split(nc), p0 = part_slices(d, mfma, wg_target).split(nc);
    sp.dual_split = 0;
    sp.dg_split = a0;
    sp.part_split = p0;
    sp.dg_f32 = mfma && d.dg_f32;
    if (!mfma || d.Q < 128 || wg_target < 256 || nc <= 0) return;
    // hundreds of cycles of a workgroup around its heads and for each of them: dx, dG, head sums
    struct Cost { int64_t around[3], head[3]; };
    const Cost c = d.Q == 256 ? Cost{{80, 110, 130}, {93, 106, 47}} : Cost{{60, 80, 90}, {110, 80, 50}};
    const int64_t base = d.Bt * nc * d.G, units = d.Q == 256 ? 256 : 512, places = dg_places(d, mfma, wg_target);
    auto one = [&](int pass, int64_t slices) { return c.around[pass] + c.head[pass] * ((d.hpg + slices - 1) / slices); };
    auto longest = [&](int64_t a, int64_t p) {
        int64_t t = one(0, a);
        t = one(1, a) > t ? one(1, a) : t;
        return one(2, p) > t ? one(2, p) : t;
    };
    // what the general rule takes: the work spread over the machine, and half a workgroup of ragged end
    const int64_t work = a0 * (one(0, a0) + one(1, a0)) + 2 * p0 * one(2, p0);
    int64_t least = base * work / units + longest(a0, p0) / 2;
    for (int a = 1; a <= a0 && base * 2 * (a + 1) <= units; ++a) {
        const bool f32 = d.dg_f32 || (a > 1 && base * a * 2 <= places);
        if (!f32 && ((a > 1 && a < a0) || base * a > places)) continue;
        for (int p = 1; p <= p0 && base * 2 * (a + p) <= units; ++p)
            if (longest(a, p) < least || (longest(a, p) == least && f32 && !sp.dg_f32))
                least = longest(a, p), sp.dual_split = sp.dg_split = a, sp.part_split = p, sp.dg_f32 = f32;
    }
}

WsLayout ws_layout(const Dims& d, bool bwd, bool mfma, int wg_target, bool fp32cs) {
    WsLayout w;
    memset(&w, 0, sizeof(w));
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += align_up(bytes);
        return o;
    };
    const size_t tok = (size_t)d.Bt * d.H * d.nc * d.Q * 4;
    const size_t PN = (size_t)d.P * d.N;
    w.nslice = (int)((PN + 255) / 256) * 4;  // partial sums of a reverse scan: one per wave
    w.tok = tok;
    w.cum = take(tok);
    w.dtf = take(tok);
    w.states = w.states_bf = w.dstates = w.dstates_bf = w.dbc_part = WS_NONE;  // present on one path only
    if (!mfma) w.states = take((size_t)d.Bt * (d.nc + 1) * d.H * PN * 4);
    if (mfma && fp32cs) w.states = take((size_t)d.Bt * d.nc * d.H * PN * 4);  // slot c: chunk state c (scan input)
    w.Gm = take((size_t)d.Bt * d.nc * d.G * d.Q * d.Q * 4);
    w.ein = w.eout = w.gintra = w.erow = w.ecol = WS_NONE;
    if (mfma) w.ein = take(tok);
    if (mfma) w.eout = take(tok);
    if (mfma) w.states_bf = take((size_t)d.Bt * d.nc * d.H * PN * 2);
    const int64_t nt = (d.Q + 63) / 64, nn = (d.N + 63) / 64, np = (d.P + 63) / 64;  // 64 x 64 tiles of the generic kernels
    const HeadSlices part = part_slices(d, mfma, wg_target);
    if (bwd) {
        if (!mfma || fp32cs) w.dstates = take((size_t)d.Bt * d.nc * d.H * PN * 4);
        if (mfma) w.dstates_bf = take((size_t)d.Bt * d.nc * d.H * PN * 2);
        w.dG = take((size_t)dg_places(d, mfma, wg_target) * d.Q * d.Q * 2);
        w.dbc_part = take((size_t)d.Bt * part.slots(d.nc) * d.G * 2 * d.Q * d.N * 4);
        w.gterm = take(tok * (mfma ? 1 : 2 * nn));
        w.sterm = take(tok * (mfma ? 1 : 2 * nn));
        if (mfma) w.gintra = take(tok);
        if (!mfma) w.erow = take(tok * 2 * nt);
        if (!mfma) w.ecol = take(tok * 2 * nt);
        w.fterm = take(tok * (mfma ? 1 : 2 * np));
        w.dDrow = take(tok * (mfma ? 1 : 2 * np));
        w.tail_part = take((size_t)d.Bt * d.H * d.nc * w.nslice * 4);
        w.dA_part = take((size_t)d.Bt * d.nc * d.H * 4);
        w.dD_part = take((size_t)d.Bt * d.nc * d.H * 4);
        w.dcarry = take((size_t)d.Bt * d.H * PN * 4);
    }
    w.total = off;
    return w;
}

void bind_workspace(SegParams& sp, const WsLayout& w, void* workspace, bool bwd) {
    char* base = (char*)workspace;
    auto at = [&](size_t off) { return off == WS_NONE ? nullptr : base + off; };
    sp.cum = (float*)(base + w.cum);
    sp.dtf = (float*)(base + w.dtf);
    sp.states = (float*)at(w.states);
    sp.Gm = (float*)(base + w.Gm);
    sp.nslice = w.nslice;
    sp.ein = (float*)at(w.ein);
    sp.eout = (float*)at(w.eout);
    sp.tok_stride = (int64_t)(w.tok / 4);
    sp.states_bf = (bf16_t*)at(w.states_bf);
    if (bwd) {
        sp.dstates_bf = (bf16_t*)at(w.dstates_bf);
        sp.dbc_part = (float*)at(w.dbc_part);
        sp.dstates = (float*)at(w.dstates);
        sp.dG = (float*)(base + w.dG);
        sp.gterm = (float*)(base + w.gterm);
        sp.sterm = (float*)(base + w.sterm);
        sp.gintra = (float*)at(w.gintra);
        sp.erow = (float*)at(w.erow);
        sp.ecol = (float*)at(w.ecol);
        sp.fterm = (float*)(base + w.fterm);
        sp.dDrow = (float*)(base + w.dDrow);
        sp.tail_part = (float*)(base + w.tail_part);
        sp.dA_part = (float*)(base + w.dA_part);
        sp.dD_part = (float*)(base + w.dD_part);
        sp.dcarry = (float*)(base + w.dcarry);
        sp.dcarry_in = sp.dcarry;
    }
}

void base_params(SegParams& sp, const Dims& d, uint32_t flags) {
    memset(&sp, 0, sizeof(sp));
    sp.Bt = (int)d.Bt;
    sp.H = d.H;
    sp.P = d.P;
    sp.G = d.G;
    sp.N = d.N;
    sp.Q = d.Q;
    sp.nc = d.nc;
    sp.hpg = d.hpg;
    sp.xs_b = sp.ys_b = sp.dys_b = sp.dxs_b = d.xs_b;
    sp.dts_b = d.dts_b;
    sp.bcs_b = d.bcs_b;
    sp.flags = flags;
    sp.nc_total = d.nc;
    sp.ntok = d.nc * d.Q;
    sp.seg_chunks = d.nc;
    sp.wg_target = 256;
#ifdef SSDK_STAMPS
    sp.stamps = g_stamps;
#endif
}

static inline const void* off(const void* p, int64_t elems, size_t esz) { return p ? (const char*)p + elems * (int64_t)esz : nullptr; }
static inline void* off(void* p, int64_t elems, size_t esz) { return p ? (char*)p + elems * (int64_t)esz : nullptr; }

bool use_mfma(const ssd_shape_t& sh, uint32_t flags) {
    return !(flags & SSD_FLAG_GENERIC_KERNELS) && mfma_path_supported(sh);
}

// Points the scan of the span that starts with segment k at its entering state, at the checkpoints between its
// segments and at the places its leaving state goes; ns = its segments.
static void wire_states(SegParams& sp, const Dims& d, int64_t k, int64_t ns, const float* init_state, const float* bnd_ro,
                        float* bnd_rw, float* final_state) {
    const int64_t HPN = (int64_t)d.H * d.P * d.N;
    if (k == 0 || !bnd_ro) {
        sp.state_in = init_state;
        sp.state_in_bs = HPN;
    } else {
        sp.state_in = bnd_ro + k * HPN;
        sp.state_in_bs = d.nseg * HPN;
    }
    sp.bnd_write = nullptr;
    sp.state_out = nullptr;
    sp.state_out2 = nullptr;
    sp.state_in16 = nullptr;
    sp.bnd_write16 = nullptr;
    sp.state_out16 = nullptr;
    sp.ckpt = bnd_rw ? bnd_rw + k * HPN : (bnd_ro ? (float*)bnd_ro + k * HPN : nullptr);
    sp.ckpt16 = nullptr;
    sp.ckpt_bs = d.nseg * HPN;
    if (bnd_rw) {
        if (k == 0) {
            sp.bnd_write = bnd_rw;
            sp.bnd_write_bs = d.nseg * HPN;
        }
        if (k + ns < d.nseg) {
            sp.state_out = bnd_rw + (k + ns) * HPN;
            sp.state_out_bs = d.nseg * HPN;
        }
    }
    if (k + ns == d.nseg && final_state) {
        sp.state_out2 = final_state;
        sp.state_out2_bs = HPN;
    }
}

// ---- several spans in flight ---------------------------------------------------------------
// Consecutive spans depend on each other only through the state scan.  With more than one
// span, span k runs on lane k % nl -- lane 0 is the caller's stream, the others are internal
// streams (default priority) -- each lane with its own scratch; events order the scans.
// This overlaps one span's launch gaps, tails and bandwidth-bound kernels with another's matrix work.
constexpr int NPIPE = 4;  // spans in flight at most (the caller's stream + NPIPE - 1 internal ones)
constexpr int INFLIGHT = 8;  // segments in flight at most
struct Pipe {
    hipStream_t aux[NPIPE] = {};       // aux[0] is unused: lane 0 is the caller's stream
    hipEvent_t fork = nullptr, join[NPIPE] = {}, scan[NPIPE] = {};
    bool ok = false;
};

// Created on the first call that needs them on a device (or by ssd_init), under a lock; a partial failure
// releases what was created and leaves the entry unset, so that a later call tries again.
static std::mutex g_pipe_mu;

static Pipe* pipe_for_current_device() {
    static Pipe pipes[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_pipe_mu);
    Pipe& p = pipes[dev];
    if (p.ok) return &p;
    Pipe q;
    bool good = hipEventCreateWithFlags(&q.fork, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; good && i < NPIPE; ++i) {
        if (i > 0) good = hipStreamCreateWithFlags(&q.aux[i], hipStreamNonBlocking) == hipSuccess;
        good = good && hipEventCreateWithFlags(&q.join[i], hipEventDisableTiming) == hipSuccess;
        good = good && hipEventCreateWithFlags(&q.scan[i], hipEventDisableTiming) == hipSuccess;
    }
    if (!good) {
        if (q.fork) (void)hipEventDestroy(q.fork);
        for (int i = 0; i < NPIPE; ++i) {
            if (q.aux[i]) (void)hipStreamDestroy(q.aux[i]);
            if (q.join[i]) (void)hipEventDestroy(q.join[i]);
            if (q.scan[i]) (void)hipEventDestroy(q.scan[i]);
        }
        return nullptr;
    }
    q.ok = true;
    p = q;
    return &p;
}

// Forward without checkpoints (boundary_states == NULL, several spans): the state leaving one
// span reaches the next through two buffers used alternately (the scans are ordered by events, so
// a buffer is rewritten only after its reader has finished).
static size_t carry_bytes(const Dims& d) { return d.nseg > 1 ? 2 * align_up((size_t)d.Bt * d.H * d.P * d.N * 4) : 0; }

// Bytes of the arrays shared by all scratch blocks: the dA / dD partial sums of every chunk.
static size_t shared_bytes(const Dims& d) { return 2 * align_up((size_t)d.Bt * d.nct * d.H * 4); }

// SSD_MAGC_SERIAL=1 in the environment keeps every segment on the caller's stream (diagnostics: per-kernel
// timings are only meaningful when kernels do not overlap).
static bool g_serial = false;  // ssd_prof_serialize

bool serial_mode() {
    static const bool serial = [] {
        const char* v = getenv("SSD_MAGC_SERIAL");
        return v && v[0] == '1';
    }();
    return serial || g_serial;
}

// SSD_MAGC_LANES=n (1 .. NPIPE) in the environment caps the spans in flight (measurements; the default is NPIPE).
static int lane_cap() {
    static const int cap = [] {
        const char* v = getenv("SSD_MAGC_LANES");
        const int n = v ? atoi(v) : NPIPE;
        return n < 1 ? 1 : (n > NPIPE ? NPIPE : n);
    }();
    return cap;
}

// What a launch works on, from the sizes alone.  Work is counted in units of one chunk of one head.
//  - Chunk length: the caller's.  256 tokens are fastest over long sequences (65536 tokens of 80 heads: 3.2 ms, 4.1 ms at
//    128, with twice the chunk states to move), but shorter chunks keep the sums of dt A, and with them the rounding of
//    every decay, smaller, and the results must depend neither on where the checkpoints fall nor on the entry point.
//  - Segments per span: a launch of fewer than SPAN_UNITS units leaves compute units idle and costs the host as much as
//    a full one (8192 tokens of 24 heads in four segments: 43 launches, bound by enqueuing them), so consecutive
//    segments share their launches until that is reached; the scans put the checkpoints down on the way.  131072 tokens of
//    24 heads: segments of 96 units 3.16 ms (4.48 with two segments a launch), of 192 units 2.67 (4.21 with one), of 384 units
//    2.25 (2.69); 65536 of 64 heads, 512 units: 2.58 (2.99).  Segments of 640 units would gain as well (65536 of 80 heads: 3.12
//    ms instead of 3.55) but four launches of two hold 379 MB instead of 262; from 1280 units on nothing changes (3.11).
//  - Memory: at most four segments' scratch is alive at a time, eight (INFLIGHT) when a segment is below a full launch: eight
//    of those hold less than four full ones do.  With four, 65536 tokens of 24 heads in segments of 1024 take 2410 us
//    instead of 1627, 32768 of 80 heads 2107 instead of 1866, 4096 fp32 tokens of 24 heads in segments of 256 578 instead
//    of 432.
//  - A sequence of few units altogether (ONE_SPAN_UNITS), in at most eight segments of less than SPAN_UNITS each or at most four
//    longer ones, is one span: nothing to order, no events, full launches, and no more scratch than on lanes (fewer partial
//    sums: 337 MB instead of 379 for 16384 tokens of 80 heads).  Matrix-core kernels, us on lanes -> as one span, forward +
//    backward.  Near the line: 16091 tokens of 80 heads in four segments 246 + 607 -> 191 + 637, chunks of 128 301 + 700 -> 234 +
//    720, in two segments 307 + 843 -> 235 + 721; 53211 of 24 heads 257 + 692 -> 233 + 650, chunks of 128 320 + 820 -> 272 + 853.
//    So the backward pass alone goes either way there (in 110 shapes, 8 % longer to 25 % shorter); the two together take 2 %
//    longer in two of the shapes (20187 of 64 in four segments, 2 x 26587 of 24 in chunks of 128) and up to 25 % less in the
//    others.  Beyond the line they go either way too: 24576 of 80 (7680 units) 1222 -> 1200, 40000 of 2 x 24 (7500) 1306 ->
//    1346, 65536 of 32 (8192) 1369 -> 1480.
//  - Fewer than ten heads (over the batch) stay on lanes from LANE_UNITS on: the state scan is serial in the chunks of a span and
//    has eight workgroups a head.  163072 tokens of 8 heads 350 + 948 on lanes, 356 + 996 as one span, 326400 of 4 570 + 1360
//    and 525 + 1558, 1305600 of 1 1778 + 4426 and 1690 + 5222; of 10 heads, 130560 tokens, 333 + 903 and 299 + 906.
// Only the number of segments counts, not where the last one ends: the workspace query goes over these plans.
void plan_dims(Dims* d, bool mfma, bool one_stream) {
    if (d->L == 0) return;
    constexpr int64_t SPAN_UNITS = 640, LANE_UNITS = 3840, ONE_SPAN_UNITS = 5120;
    const int64_t unit = d->Bt * d->H * ((d->Q + 63) / 64);  // quarter units: 64 tokens of a head
    const int64_t seg_units = d->nc_seg * unit / 4, all_units = d->nseg * seg_units;
    const int64_t inflight = seg_units >= SPAN_UNITS ? 4 : INFLIGHT;
    d->F = d->nl = 1;
    if (!one_stream && d->nseg > 1) {
        if (d->nseg <= inflight && (all_units <= SPAN_UNITS || (mfma && all_units <= (d->Bt * d->H < 10 ? LANE_UNITS : ONE_SPAN_UNITS)))) {
            d->F = (int)d->nseg;
            d->dg_f32 = mfma && all_units > LANE_UNITS && d->nseg > 2;  // two segments on two lanes have the same slices
        } else {
            while (d->F < inflight && d->F * seg_units < SPAN_UNITS) d->F *= 2;
            const int64_t spans = (d->nseg + d->F - 1) / d->F;
            int64_t nl = inflight / d->F < spans ? inflight / d->F : spans;
            if (nl > lane_cap()) nl = lane_cap();
            if (mfma && !serial_mode()) d->nl = (int)nl;
        }
    }
    d->nspan = (d->nseg + d->F - 1) / d->F;
    const int64_t span_chunks = (int64_t)d->F * d->nc_seg;
    d->nc = (int)(span_chunks < d->nct ? span_chunks : d->nct);
}

// Workgroups a launch should have at least.  One segment at a time: one per compute unit.  Several
// segments in flight: half as many, twice as long -- launches of the other lanes fill the machine, and
// the per-workgroup prologue (fetching the operands shared by all heads) is paid half as often.
static int wg_target(int nlanes) { return nlanes > 1 ? 128 : 256; }

static bool fork_lanes(Pipe* pp, int n, hipStream_t st) {
    if (n <= 1) return true;
    if (hipEventRecord(pp->fork, st) != hipSuccess) return false;
    for (int i = 1; i < n; ++i)
        if (hipStreamWaitEvent(pp->aux[i], pp->fork, 0) != hipSuccess) return false;
    return true;
}

static bool join_lanes(Pipe* pp, int n, hipStream_t st) {
    for (int i = 1; i < n; ++i)
        if (hipEventRecord(pp->join[i], pp->aux[i]) != hipSuccess || hipStreamWaitEvent(st, pp->join[i], 0) != hipSuccess) return false;
    return true;
}

}  // namespace ssdk

using namespace ssdk;

#ifdef SSDK_STAMPS
namespace ssdk {
unsigned long long* g_stamps = nullptr;
}
extern "C" void ssd_debug_stamps(void* p) { ssdk::g_stamps = (unsigned long long*)p; }
#endif

static size_t workspace_need(Dims d, bool bwd, bool mfma, uint32_t flags) {
    plan_dims(&d, mfma, false);
    const size_t block = align_up(ws_layout(d, bwd, mfma, wg_target(d.nl), (flags & SSD_FLAG_FP32_CHUNK_STATES) != 0).total);
    return d.nl * block + (bwd ? shared_bytes(d) : carry_bytes(d));
}

// What the call itself needs, or any shorter sequence if that is more: scratch sized once for the longest serves all.
extern "C" size_t ssd_workspace_bytes_flags(const ssd_shape_t* shape, int32_t is_backward, uint32_t flags) {
    Dims d;
    if (check_shape(shape, &d) != SSD_OK) return 0;
    const bool mfma = use_mfma(*shape, flags), bwd = is_backward != 0;
    size_t t = workspace_need(d, bwd, mfma, flags);
    for (int64_t k = 1; k < d.nseg && k <= INFLIGHT; ++k) {  // from INFLIGHT + 1 segments on the plan is the same
        Dims e = d;
        e.nseg = k;
        e.L = k * d.s;
        e.nct = k * d.nc_seg;
        const size_t n = workspace_need(e, bwd, mfma, flags);
        t = n > t ? n : t;
    }
    return t ? t : 256;  // never 0 for a valid shape, so that 0 unambiguously means "invalid"
}

extern "C" size_t ssd_workspace_bytes(const ssd_shape_t* shape, int32_t is_backward) {
    return ssd_workspace_bytes_flags(shape, is_backward, 0);
}

// Token range of the span of ns segments that starts with segment k.
static void span_tokens(SegParams& sp, const Dims& d, int64_t k, int64_t ns) {
    const int64_t left = d.L - k * d.s, n = ns * d.s;
    sp.ntok = (int)(left < n ? left : n);
    sp.nc = (int)((sp.ntok + d.Q - 1) / d.Q);
    sp.seg_chunks = d.nc_seg;
    sp.reset_bs = d.L;
}

// one_stream: everything stays on the caller's stream (no library stream or event is touched).
static int fwd_impl(const ssd_shape_t* shape, const void* x, const void* dt, const RawDt& raw, const float* A, const void* B,
                    const void* C, const float* D, const float* init_state, void* y, float* final_state,
                    void* boundary_states, void* workspace, size_t workspace_bytes, uint32_t flags,
                    void* hip_stream, bool one_stream) {
    Dims d;
    int rc = check_shape(shape, &d);
    if (rc != SSD_OK) return rc;
    if (flags & ~(uint32_t)(SSD_FLAG_RESIDUAL | SSD_FLAG_GENERIC_KERNELS | SSD_FLAG_ACCUM_PARAM | SSD_FLAG_BF16_CHECKPOINTS | SSD_FLAG_FP32_CHUNK_STATES))
        return SSD_ERR_ARG;
    const bool ck16 = (flags & SSD_FLAG_BF16_CHECKPOINTS) && boundary_states;
    float* bnd32 = ck16 ? nullptr : (float*)boundary_states;
    bf16_t* bnd16 = ck16 ? (bf16_t*)boundary_states : nullptr;
    hipStream_t st = (hipStream_t)hip_stream;
    const size_t HPN = (size_t)d.H * d.P * d.N;
    if (d.L == 0) {  // empty sequence: the state passes through untouched
        if (final_state) {
            hipError_t e = init_state ? launch_copy_f32(final_state, init_state, (size_t)d.Bt * HPN, st)
                                      : launch_fill_zero(final_state, (size_t)d.Bt * HPN, st);
            if (e != hipSuccess) return SSD_ERR_LAUNCH;
        }
        return SSD_OK;
    }
    if (!x || (!dt && !raw.dt) || !A || !B || !C || !D || !y) return SSD_ERR_NULL;
    if (raw.dt && (d.Bt != 1 || !raw.bias)) return SSD_ERR_ARG;
    const bool mfma = use_mfma(*shape, flags);
    plan_dims(&d, mfma, one_stream);
    const int nl = d.nl;
    const WsLayout w = ws_layout(d, false, mfma, wg_target(nl), (flags & SSD_FLAG_FP32_CHUNK_STATES) != 0);
    const size_t block = align_up(w.total);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < nl * block + carry_bytes(d)) return SSD_ERR_WORKSPACE;
    float* carry[2] = {(float*)((char*)workspace + nl * block), (float*)((char*)workspace + nl * block + carry_bytes(d) / 2)};
    Pipe* pp = nl > 1 ? pipe_for_current_device() : nullptr;
    if (nl > 1 && !pp) return SSD_ERR_LAUNCH;

    SegParams sps[NPIPE];
    for (int i = 0; i < nl; ++i) {
        base_params(sps[i], d, flags);
        sps[i].wg_target = wg_target(nl);
        bind_workspace(sps[i], w, (char*)workspace + i * block, false);
        sps[i].A = A;
        sps[i].D = D;
    }
    if (!fork_lanes(pp, nl, st)) return SSD_ERR_LAUNCH;
    for (int64_t q = 0; q < d.nspan; ++q) {
        const int ln = (int)(q % nl);
        SegParams& sp = sps[ln];
        hipStream_t sk = ln ? pp->aux[ln] : st;
        const int64_t k = q * d.F, ns = k + d.F < d.nseg ? d.F : d.nseg - k;  // its segments
        const int64_t t0 = k * d.s;
        const int HP = d.H * d.P, GN = d.G * d.N;
        span_tokens(sp, d, k, ns);
        sp.x = off(x, t0 * HP, d.esz);
        sp.y = off(y, t0 * HP, d.esz);
        sp.dt = off(dt, t0 * d.H, d.esz);
        sp.raw = RawDt{off(raw.dt, t0 * raw.rs, d.esz), raw.rs, raw.bias};
        sp.Bm = off(B, t0 * GN, d.esz);
        sp.Cm = off(C, t0 * GN, d.esz);
        sp.reset = d.reset ? d.reset + t0 : nullptr;
        wire_states(sp, d, k, ns, init_state, bnd32, bnd32, final_state);
        if (bnd16) {  // bf16 checkpoints: rounded copies; the fp32 state itself travels in registers and through the carry buffers
            sp.ckpt16 = bnd16 + k * (int64_t)HPN;
            if (k == 0) {
                sp.bnd_write16 = bnd16;
                sp.bnd_write_bs = d.nseg * (int64_t)HPN;
            }
            if (k + ns < d.nseg) {
                sp.state_out16 = bnd16 + (k + ns) * (int64_t)HPN;
                sp.state_out16_bs = d.nseg * (int64_t)HPN;
            }
        }
        if (!bnd32 && d.nspan > 1) {  // no fp32 checkpoints: hand the state on through the carry buffers
            if (q > 0) {
                sp.state_in = carry[q & 1];
                sp.state_in_bs = (int64_t)HPN;
            }
            if (q + 1 < d.nspan) {
                sp.state_out = carry[(q + 1) & 1];
                sp.state_out_bs = (int64_t)HPN;
            }
        }
        sp.ev_wait = (nl > 1 && q > 0) ? pp->scan[(q - 1) % nl] : nullptr;
        sp.ev_record = (nl > 1 && q + 1 < d.nspan) ? pp->scan[ln] : nullptr;
        const hipError_t e = mfma ? mfma_forward_segment(sp, true, sk) : generic_forward_segment(sp, d.bf16, true, sk);
        if (e != hipSuccess) {
            (void)join_lanes(pp, nl, st);  // whatever was enqueued on the library's streams still ends before the caller's next work
            return SSD_ERR_LAUNCH;
        }
    }
    if (!join_lanes(pp, nl, st)) return SSD_ERR_LAUNCH;
    return SSD_OK;
}

extern "C" int ssd_fwd(const ssd_shape_t* shape, const void* x, const void* dt, const float* A, const void* B,
                       const void* C, const float* D, const float* init_state, void* y, float* final_state,
                       void* boundary_states, void* workspace, size_t workspace_bytes, uint32_t flags,
                       void* hip_stream) {
    return fwd_impl(shape, x, dt, RawDt{}, A, B, C, D, init_state, y, final_state, boundary_states, workspace, workspace_bytes,
                    flags, hip_stream, false);
}

int ssdk::scan_fwd(const ssd_shape_t* shape, const void* x, const void* dt, const RawDt& raw, const float* A, const void* B, const void* C,
                   const float* D, const float* init_state, void* y, float* final_state, void* boundary_states, void* workspace,
                   size_t workspace_bytes, uint32_t flags, hipStream_t st) {
    return fwd_impl(shape, x, dt, raw, A, B, C, D, init_state, y, final_state, boundary_states, workspace, workspace_bytes, flags, st, false);
}

// ---- forward pass for callers that cannot allocate -------------------------------------------------
// The per-segment scratch lives in a file-scope device array instead of a caller's workspace.  Every
// device the library runs on holds its own copy of the array, at its own address, until the process ends;
// the address is looked up once per device (hipGetSymbolAddress with that device current) and only that
// pointer -- never the array's name, which in host code is a stand-in and not a device address -- is
// handed to the kernels.
namespace ssdk {
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)SSD_STATIC_SCRATCH_MIB << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[64] = {};

// The array's address on the current device (looked up on first use there), or NULL on failure.
static void* static_scratch() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

// Scratch bytes of a forward call that stays on one stream.
static size_t fwd_bytes_one_stream(const ssd_shape_t* shape, uint32_t flags) {
    Dims d;
    if (check_shape(shape, &d) != SSD_OK) return 0;
    const bool mfma = use_mfma(*shape, flags);
    plan_dims(&d, mfma, true);
    const size_t t = align_up(ws_layout(d, false, mfma, wg_target(1), (flags & SSD_FLAG_FP32_CHUNK_STATES) != 0).total) + carry_bytes(d);
    return t ? t : 256;
}
}  // namespace ssdk

extern "C" int ssd_init(void) {
    // everything the library creates lazily on a device: the scratch array's address, the streams and events of
    // the segments in flight, the side stream of the blocks
    const bool a = static_scratch() != nullptr, b = pipe_for_current_device() != nullptr;
    const bool c = serial_mode() || side_stream() != nullptr;
    return a && b && c ? SSD_OK : SSD_ERR_LAUNCH;
}

extern "C" size_t ssd_fwd_static_bytes(const ssd_shape_t* shape, uint32_t flags) { return fwd_bytes_one_stream(shape, flags); }

extern "C" int ssd_fwd_static(const ssd_shape_t* shape, const void* x, const void* dt, const float* A, const void* B,
                              const void* C, const float* D, const float* init_state, void* y, float* final_state,
                              void* boundary_states, uint32_t flags, void* hip_stream) {
    Dims d;
    const int rc = check_shape(shape, &d);
    if (rc != SSD_OK) return rc;
    const size_t need = fwd_bytes_one_stream(shape, flags);
    if (need > STATIC_SCRATCH_BYTES) return SSD_ERR_WORKSPACE;  // beyond the array: use ssd_fwd with a workspace
    void* ws = static_scratch();
    if (!ws) return SSD_ERR_LAUNCH;
    // Nothing in the scratch has to start at zero: every array in it is written by the kernel that
    // precedes its first reader within the same call.
    return fwd_impl(shape, x, dt, RawDt{}, A, B, C, D, init_state, y, final_state, boundary_states, ws, need, flags, hip_stream, true);
}

int ssdk::scan_bwd(const ssd_shape_t* shape, const void* x, const void* dt, const RawDt& raw, const float* A, const void* B, const void* C,
                   const float* D, const float* init_state, const void* dy, const float* dfinal_state, const void* boundary_states,
                   void* dx, void* ddt, float* dA, void* dB, void* dC, float* dD, float* dinit_state, void* workspace,
                   size_t workspace_bytes, uint32_t flags, hipStream_t st) {
    Dims d;
    int rc = check_shape(shape, &d);
    if (rc != SSD_OK) return rc;
    if (flags & ~(uint32_t)(SSD_FLAG_RESIDUAL | SSD_FLAG_GENERIC_KERNELS | SSD_FLAG_ACCUM_PARAM | SSD_FLAG_BF16_CHECKPOINTS | SSD_FLAG_FP32_CHUNK_STATES))
        return SSD_ERR_ARG;
    const bool ck16 = (flags & SSD_FLAG_BF16_CHECKPOINTS) && boundary_states;
    if (!dA || !dD) return SSD_ERR_NULL;
    const size_t HPN = (size_t)d.H * d.P * d.N;
    if (d.L == 0) {  // empty sequence: the state adjoint passes through, parameter gradients are zero
        hipError_t e = hipSuccess;
        if (dinit_state)
            e = dfinal_state ? launch_copy_f32(dinit_state, dfinal_state, (size_t)d.Bt * HPN, st)
                             : launch_fill_zero(dinit_state, (size_t)d.Bt * HPN, st);
        if (e == hipSuccess && !(flags & SSD_FLAG_ACCUM_PARAM)) {
            e = launch_fill_zero(dA, d.H, st);
            if (e == hipSuccess) e = launch_fill_zero(dD, d.H, st);
        }
        return e == hipSuccess ? SSD_OK : SSD_ERR_LAUNCH;
    }
    if (!x || (!dt && !raw.dt) || !A || !B || !C || !D || !dy || !dx || !ddt || !dB || !dC) return SSD_ERR_NULL;
    if (dx == dy || (raw.dt && (d.Bt != 1 || !raw.bias))) return SSD_ERR_ARG;
    if (!boundary_states && d.nseg > 1) return SSD_ERR_NULL;
    const bool mfma = use_mfma(*shape, flags);
    plan_dims(&d, mfma, false);
    const int nl = d.nl;
    const WsLayout w = ws_layout(d, true, mfma, wg_target(nl), (flags & SSD_FLAG_FP32_CHUNK_STATES) != 0);
    const size_t block = align_up(w.total);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < nl * block + shared_bytes(d)) return SSD_ERR_WORKSPACE;
    Pipe* pp = nl > 1 ? pipe_for_current_device() : nullptr;
    if (nl > 1 && !pp) return SSD_ERR_LAUNCH;

    // shared by all scratch blocks: the carried state adjoint and the dA / dD partial sums of every chunk
    float* part_all = (float*)((char*)workspace + nl * block);
    SegParams sps[NPIPE];
    for (int i = 0; i < nl; ++i) {
        SegParams& sp = sps[i];
        base_params(sp, d, flags);
        sp.wg_target = wg_target(nl);
        bind_workspace(sp, w, (char*)workspace + i * block, true);
        sp.A = A;
        sp.D = D;
        sp.dA = dA;
        sp.dD = dD;
        sp.dcarry = sps[0].dcarry;
        sp.param_count = i ? sps[0].param_count : (int*)sp.dA_part;  // the block's own array for one span's partial sums is free
        sp.param_stride = d.Bt * d.nc < 32 ? (int)(d.Bt * d.nc) : 32;  // what fits there, a cache line each at most
        sp.dA_part = part_all;
        sp.dD_part = (float*)((char*)part_all + align_up((size_t)d.Bt * d.nct * d.H * 4));
        sp.nc_total = (int)d.nct;  // every chunk of the sequence writes a dA / dD partial sum
        sp.accumulate = (flags & SSD_FLAG_ACCUM_PARAM) ? 1 : 0;
    }
    if (!fork_lanes(pp, nl, st)) return SSD_ERR_LAUNCH;
    for (int64_t q = d.nspan - 1, it = 0; q >= 0; --q, ++it) {
        const int ln = (int)(it % nl);
        SegParams& sp = sps[ln];
        hipStream_t sk = ln ? pp->aux[ln] : st;
        const int64_t k = q * d.F, ns = k + d.F < d.nseg ? d.F : d.nseg - k;  // its segments
        const int64_t t0 = k * d.s;
        const int HP = d.H * d.P, GN = d.G * d.N;
        span_tokens(sp, d, k, ns);
        fit_splits(sp, d, mfma, wg_target(nl));
        sp.x = off(x, t0 * HP, d.esz);
        sp.dy = off(dy, t0 * HP, d.esz);
        sp.dx = off(dx, t0 * HP, d.esz);
        sp.dt = off(dt, t0 * d.H, d.esz);
        sp.raw = RawDt{off(raw.dt, t0 * raw.rs, d.esz), raw.rs, raw.bias};
        sp.ddt = off(ddt, t0 * d.H, d.esz);
        sp.Bm = off(B, t0 * GN, d.esz);
        sp.Cm = off(C, t0 * GN, d.esz);
        sp.dB = off(dB, t0 * GN, d.esz);
        sp.dC = off(dC, t0 * GN, d.esz);
        sp.reset = d.reset ? d.reset + t0 : nullptr;
        sp.chunk0 = (int)(k * d.nc_seg);
        // restore: per-chunk entering states of the span from its segments' checkpoints
        wire_states(sp, d, k, ns, init_state, ck16 ? nullptr : (const float*)boundary_states, nullptr, nullptr);
        if (ck16) {  // restart from the rounded checkpoints
            sp.ckpt16 = (bf16_t*)boundary_states + k * (int64_t)HPN;
            if (k > 0) {
                sp.state_in = nullptr;
                sp.state_in16 = sp.ckpt16;
                sp.state_in_bs = d.nseg * (int64_t)HPN;
            }
        }
        sp.first_span = it == 0;
        sp.dcarry_in = it == 0 ? dfinal_state : sp.dcarry;
        sp.ev_wait = sp.ev_record = nullptr;
        hipError_t e = mfma ? mfma_forward_segment(sp, false, sk) : generic_forward_segment(sp, d.bf16, false, sk);
        if (e == hipSuccess) {
            sp.dinit_out = (k == 0) ? dinit_state : nullptr;
            sp.ev_wait = (nl > 1 && it > 0) ? pp->scan[(it - 1) % nl] : nullptr;
            sp.ev_record = (nl > 1 && q > 0) ? pp->scan[ln] : nullptr;
            e = mfma ? mfma_backward_segment(sp, sk) : generic_backward_segment(sp, d.bf16, sk);
        }
        if (e != hipSuccess) {
            (void)join_lanes(pp, nl, st);  // whatever was enqueued on the library's streams still ends before the caller's next work
            return SSD_ERR_LAUNCH;
        }
    }
    if (!join_lanes(pp, nl, st)) return SSD_ERR_LAUNCH;
    return SSD_OK;
}

extern "C" int ssd_bwd(const ssd_shape_t* shape, const void* x, const void* dt, const float* A, const void* B,
                       const void* C, const float* D, const float* init_state, const void* dy,
                       const float* dfinal_state, const void* boundary_states, void* dx, void* ddt, float* dA,
                       void* dB, void* dC, float* dD, float* dinit_state, void* workspace, size_t workspace_bytes,
                       uint32_t flags, void* hip_stream) {
    return scan_bwd(shape, x, dt, RawDt{}, A, B, C, D, init_state, dy, dfinal_state, boundary_states, dx, ddt, dA, dB, dC, dD, dinit_state,
                    workspace, workspace_bytes, flags, (hipStream_t)hip_stream);
}

extern "C" int ssd_prof_serialize(int32_t on) {
    g_serial = on != 0;
    return SSD_OK;
}

extern "C" const char* ssd_strerror(int status) {
    switch (status) {
        case SSD_OK: return "ok";
        case SSD_ERR_NULL: return "a required pointer is NULL";
        case SSD_ERR_SHAPE: return "a dimension is non-positive or exceeds a kernel limit";
        case SSD_ERR_DIVISIBILITY: return "nheads % ngroups or segment % chunk is not zero (stack: seqlen % segment)";
        case SSD_ERR_DTYPE: return "unknown dtype";
        case SSD_ERR_WORKSPACE: return "workspace is NULL, not 256-byte aligned, or too small";
        case SSD_ERR_LAUNCH: return "a HIP launch failed";
        case SSD_ERR_BUDGET: return "no admissible checkpoint plan fits the budget";
        case SSD_ERR_ARG: return "invalid argument";
        default: return "unknown status";
    }
}
