// The last step of the backward pass of one chunk and head, shared by the shape-generic kernels and the
// matrix-core path: da = reverse cumulative sum of the gradient of cum (+ the chunk-end term), ddt = A da + f,
// and the chunk's partial sums of dA and dD.
#pragma once
#include "ssd_internal.h"

namespace ssdk {

constexpr int DDT_THREADS = 256, DDT_E = 4;  // threads per workgroup; tokens per thread at most (chunks of up to 1024)

struct DdtLds {
    float tot[DDT_THREADS / 64], stot[DDT_THREADS / 64], tail[DDT_THREADS / 64], pa[DDT_THREADS / 64], pd[DDT_THREADS / 64];
};

// Per token: g = gradient of cum without the state term s (dcum = g - s), f = the direct part of ddt, d = dY . x.
struct DdtIn {
    float g, s, f, d;
};

static __device__ __forceinline__ float wave_sum(float v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// One workgroup of DDT_THREADS per (chunk c, head h, batch b).  load(offset of the chunk and head + i, i) returns what
// the passes before left for token i; store(index into ddt, value) writes one element of ddt in its storage type.
// Sums run inside the waves (lane exchanges) and then over the four waves: two barriers in all, where a scan over LDS
// took two per doubling (it was half of the launch it rides in for a few chunks).
template <class Load, class Store>
__device__ __forceinline__ void ddt_finalize_body(const SegParams& sp, DdtLds& L, int c, int h, int b, Load load, Store store) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int Q = sp.Q, V = chunk_rows(sp, c, Q), E = (Q + DDT_THREADS - 1) / DDT_THREADS;
    const int64_t cbase = (((int64_t)b * sp.H + h) * sp.nc + c) * Q;
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
    float incl = run;
    for (int off = 1; off < 64; off <<= 1) {
        const float v = __shfl_up(incl, off, 64);
        if (lane >= off) incl += v;
    }
    const float* tp = sp.tail_part + (((int64_t)b * sp.H + h) * sp.nc + c) * sp.nslice;
    float tail = 0.f;
    for (int k = tid; k < sp.nslice; k += DDT_THREADS) tail += tp[k];
    tail = wave_sum(tail);
    ssum = wave_sum(ssum);
    if (lane == 63) {
        L.tot[w] = incl;
        L.stot[w] = ssum;
        L.tail[w] = tail;
    }
    __syncthreads();
    float before = incl - run, end = 0.f;
#pragma unroll
    for (int q = 0; q < DDT_THREADS / 64; ++q) {
        before += q < w ? L.tot[q] : 0.f;
        end += L.stot[q] + L.tail[q];
    }
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
    pa = wave_sum(pa);
    pd = wave_sum(pd);
    if (lane == 0) {
        L.pa[w] = pa;
        L.pd[w] = pd;
    }
    __syncthreads();
    if (tid == 0) {
        float a = 0.f, s = 0.f;
#pragma unroll
        for (int q = 0; q < DDT_THREADS / 64; ++q) {
            a += L.pa[q];
            s += L.pd[q];
        }
        sp.dA_part[((int64_t)b * sp.nc_total + sp.chunk0 + c) * sp.H + h] = a;
        sp.dD_part[((int64_t)b * sp.nc_total + sp.chunk0 + c) * sp.H + h] = s;
    }
}

// What the matrix-core passes leave per token.
static __device__ __forceinline__ DdtIn ddt_load_mfma(const SegParams& sp, int64_t o) {
    return {sp.gterm[o] + sp.gintra[o], sp.sterm[o], sp.fterm[o], sp.dDrow[o]};
}

}  // namespace ssdk
