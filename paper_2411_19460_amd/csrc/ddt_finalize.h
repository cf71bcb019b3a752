// The last step of the backward pass of one chunk and head, shared by the shape-generic kernels and the
// matrix-core path: da = reverse cumulative sum of the gradient of cum (+ the chunk-end term), ddt = A da + f,
// and the chunk's partial sums of dA and dD; the last chunk of a head to come by sums them.
#pragma once
#include "ssd_internal.h"

namespace ssdk {

constexpr int DDT_E = 4;  // tokens per thread at most

struct DdtLds {  // for four waves a chunk and head
    float tot[4], stot[4], tail[4], pa[4], pd[4];
    int last;
};

// Per token: g = gradient of cum without the state term s (dcum = g - s), f = the direct part of ddt, d = dY . x.
struct DdtIn {
    float g, s, f, d;
};

// W waves per (chunk c, head h, batch b), of one workgroup: 4, for chunks of up to 1024 tokens, or 1 for up to 256 (no barrier
// then: the waves of the workgroup have chunks of their own).  load(offset of the chunk and head + i, i) returns what
// the passes before left for token i; store(index into ddt, value) writes one element of ddt in its storage type.
// Sums run inside the waves (lane exchanges) and then over the four waves: two barriers, where a scan over LDS
// took two per doubling (it was half of the launch it rides in for a few chunks).
template <int W, class Load, class Store>
__device__ __forceinline__ void ddt_finalize_body(const SegParams& sp, DdtLds* lds, int c, int h, int b, Load load, Store store) {
    constexpr int T = 64 * W;
    const int tid = threadIdx.x & (T - 1), lane = tid & 63, w = tid >> 6;
    const int Q = sp.Q, V = chunk_rows(sp, c, Q), E = (Q + T - 1) / T;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
    DdtLds& L = *lds;  // not used by a wave on its own
    // over the waves, in their order; every thread has the sum
    auto over_waves = [&](float v, float (&at)[4]) {
        if constexpr (W == 1) return v;
        float t = 0.f;
#pragma unroll
        for (int q = 0; q < W; ++q) t += at[q];
        return t;
    };
    // The gradient of cum_i arrives as g - s, and the gradient of cum at the chunk end carries + sum_j s_j (the chunk
    // state depends on T - cum_j): the very same s values enter with both signs, so their cancellation in the suffix
    // sums is exact.  Thread t owns tokens Q - 1 - t E - e: a prefix sum over the threads is a suffix sum over tokens.
    float da[DDT_E], f[DDT_E], d[DDT_E], run = 0.f, ssum = 0.f;
#pragma unroll
    for (int e = 0; e < DDT_E; ++e) {
        const int i = Q - 1 - (tid * E + e);
        DdtIn v = {0.f, 0.f, 0.f, 0.f};
        if (e < E && i >= 0 && i < V) v = load(cbase + i, i);
        run += v.g - v.s;
        ssum += v.s;
        da[e] = run;
        f[e] = v.f;
        d[e] = v.d;
    }
    const float incl = wave_prefix(run);
    const float* tp = sp.tail_part + (((int64_t)b * sp.H + h) * sp.nc + c) * sp.nslice;
    float tail = 0.f;
    for (int k = tid; k < sp.nslice; k += T) tail += tp[k];
    tail = wave_total(tail);
    ssum = wave_total(ssum);
    if constexpr (W > 1) {
        if (lane == 63) {
            L.tot[w] = incl;
            L.stot[w] = ssum;
            L.tail[w] = tail;
        }
        __syncthreads();
    }
    float before = incl - run;
#pragma unroll
    for (int q = 0; q < W - 1; ++q) before += q < w ? L.tot[q] : 0.f;
    const float end = over_waves(ssum, L.stot) + over_waves(tail, L.tail);
    float pa = 0.f, pd = 0.f;
    const float A = sp.A[h];
#pragma unroll
    for (int e = 0; e < DDT_E; ++e) {
        const int i = Q - 1 - (tid * E + e);
        if (e < E && i >= 0 && i < V) {
            const float g = before + da[e] + end;
            store((int64_t)b * sp.dts_b + ((int64_t)c * Q + i) * sp.H + h, A * g + f[e]);
            pa += sp.dtf[cbase + i] * g;
            pd += d[e];
        }
    }
    auto param_sums = [&] {
        pa = wave_total(pa);
        pd = wave_total(pd);
        if constexpr (W > 1) {
            if (lane == 0) {
                L.pa[w] = pa;
                L.pd[w] = pd;
            }
            __syncthreads();
            pa = over_waves(pa, L.pa);
            pd = over_waves(pd, L.pd);
        }
    };
    param_sums();
    const int n = sp.Bt * sp.nc_total;
    int last = 0;
    if (tid == 0) {
        const int64_t slot = ((int64_t)b * sp.nc_total + sp.chunk0 + c) * sp.H + h;
        __hip_atomic_store(sp.dA_part + slot, pa, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(sp.dD_part + slot, pd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // both have reached the memory that all compute units see
        last = __hip_atomic_fetch_add(sp.param_count + (int64_t)h * sp.param_stride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == n;
    }
    if constexpr (W > 1) {
        if (tid == 0) L.last = last;
        __syncthreads();
        last = L.last;
    } else {
        last = __builtin_amdgcn_readfirstlane(last);
    }
    if (!last) return;
    // Every chunk of this head has left its partial sums: sum them, in an order that only their number sets.  Nobody waits
    // for anybody, the waves that happen to come last do it.  A launch of its own took 4 us and the gap before it,
    // of 64 us for 512 fp32 tokens of 4 heads and 173 us for 8192 tokens of 24.  Relaxed accesses at the device's scope suffice
    // on this chip: they pass by the caches that are not shared, the wait above orders the stores before the count, and the loads
    // are issued once the count is known.  A release and acquire on the count instead, which writes a whole second-level cache
    // back for every chunk and head: 65536 tokens of 80 heads 2984 -> 3902 us, 8192 of 24 166 -> 194.
    // Eight loads of either array in flight: a trip to memory for every T chunks was 77 us of 18760 for 1048576 tokens of 8 heads in
    // chunks of 64 (16384 of them, 64 a trip), 26 of 7476 for 262144 tokens of 24; the same order, the same bits.
    constexpr int U = 8;
    pa = pd = 0.f;
    for (int b0 = 0; b0 < n; b0 += U * T) {
        float va[U], vd[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int bc = b0 + u * T + tid;
            va[u] = vd[u] = 0.f;
            if (bc < n) {
                va[u] = __hip_atomic_load(sp.dA_part + (int64_t)bc * sp.H + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                vd[u] = __hip_atomic_load(sp.dD_part + (int64_t)bc * sp.H + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            pa += va[u];
            pd += vd[u];
        }
    }
    param_sums();
    if (tid == 0) {
        sp.dA[h] = sp.accumulate ? sp.dA[h] + pa : pa;
        sp.dD[h] = sp.accumulate ? sp.dD[h] + pd : pd;
    }
}

// What the matrix-core passes leave per token.
static __device__ __forceinline__ DdtIn ddt_load_mfma(const SegParams& sp, int64_t o) {
    return {sp.gterm[o] + sp.gintra[o], sp.sterm[o], sp.fterm[o], sp.dDrow[o]};
}

}  // namespace ssdk
