// Merge of the ranges' partials, in a kernel of its own or by the last workgroup of the item kernel:
//   out[r][h][c] = sum_s acc_s[c] 2^(m_s - M) / sum_s l_s 2^(m_s - M)
#pragma once
#include "apt_device.h"

namespace {

// Four channels from c on.  Bound by latency: the partials of up to eight ranges are asked for at once.
// THROUGH: the partials were written by this launch (put_partial), on any XCD
template <bool THROUGH, typename T> __device__ inline T get_partial(const T* at) {
    if constexpr (!THROUGH) return *at;
    uint64_t w[sizeof(T) / 8];
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 8; ++i) w[i] = __hip_atomic_load((const uint64_t*)at + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(T, w);
}
template <bool THROUGH, typename Params> __device__ __forceinline__ float4 merged4(const Params& p, int r, int h, int c, int HD) {
    constexpr int N = 8;
    const int ns = p.plan[APT_PW_HEADER + APT_PA_SPLIT_COUNT * p.B + r];
    const int64_t base = (int64_t)p.plan[APT_PW_HEADER + APT_PA_WS_OFFSET * p.B + r] * p.H + h;
    float2 ml[N];
    float4 acc[N];
    auto load_ml = [&](int s0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < ns) ml[i] = get_partial<THROUGH>(p.ws_ml + base + (int64_t)(s0 + i) * p.H);
    };
    auto load_acc = [&](int s0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < ns) acc[i] = get_partial<THROUGH>((const float4*)(p.ws_acc + (base + (int64_t)(s0 + i) * p.H) * HD + c));
    };
    load_ml(0);
    load_acc(0);
    float M = kSentinel;
    for (int s0 = 0; s0 < ns; s0 += N) {
        if (s0) load_ml(s0);
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < ns) M = fmaxf(M, ml[i].x);
    }
    if (ns > N) load_ml(0);
    float L = 0.f;
    float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < ns; s0 += N) {
        if (s0) load_ml(s0), load_acc(s0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (s0 + i >= ns) continue;
            const float wgt = fast_exp2(ml[i].x - M);
            L = fmaf(ml[i].y, wgt, L);
            A.x = fmaf(acc[i].x, wgt, A.x);
            A.y = fmaf(acc[i].y, wgt, A.y);
            A.z = fmaf(acc[i].z, wgt, A.z);
            A.w = fmaf(acc[i].w, wgt, A.w);
        }
    }
    return make_float4(A.x / L, A.y / L, A.z / L, A.w / L);
}

// elements i .. i + 3 of the output (i a multiple of four; out may lie at any element)
template <int ODT> __device__ inline void store_out4(char* out, int64_t i, const float4& o) {
    store_out<ODT>(out, i, o.x);
    store_out<ODT>(out, i + 1, o.y);
    store_out<ODT>(out, i + 2, o.z);
    store_out<ODT>(out, i + 3, o.w);
}

// A partial of a launch that may merge by itself: written through to the device, so that it needs no write-back of the L2.
__device__ inline void put_partial(const ItemParams& p, int64_t slot, int c, int HD, float acc) {
    __hip_atomic_store(p.ws_acc + slot * HD + c, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void put_partial_ml(const ItemParams& p, int64_t slot, float m, float l) {
    __hip_atomic_store((uint64_t*)(p.ws_ml + slot), __builtin_bit_cast(uint64_t, make_float2(m, l)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int DT, int HD, int NW = 4>
__device__ __forceinline__ void kv_item_through(const ItemParams& p, int r, int h, int t0, int t1, char* lds) {
    kv_range<DT, HD, NW>(p, r, h, t0, t1, lds, [&](int c, float M, float L, float A) {
        const int64_t slot = ((int64_t)p.plan[APT_PW_HEADER + APT_PA_WS_OFFSET * p.B + r] + t0 / p.kv_chunk) * p.H + h;
        put_partial(p, slot, c, HD, A);
        if (c == 0) put_partial_ml(p, slot, M, L);
    });
}

// At the end of every item of a launch of one workgroup per item (p.out set): the workgroup that is last to get here merges all
// partials, so that a small step is a launch shorter.  The ticket is 0 between launches.  A workgroup takes its ticket when all of
// its partial is written through, and the last one reads them past the caches of its XCD.
template <int DT, int HD> __device__ __forceinline__ void merge_by_last(const ItemParams& p, char* lds) {
    if (!p.out) return;
    wait_vmcnt<0>();
    __syncthreads();
    int* ticket = (int*)lds;
    if (threadIdx.x == 0) *ticket = __hip_atomic_fetch_add(p.kv_ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*ticket != p.n_items - 1) return;
    if (threadIdx.x == 0) *p.kv_ticket = 0;
    const int n = p.B * p.H * (HD / 4);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int pair = i / (HD / 4);
        const float4 o = merged4<true>(p, pair / p.H, pair % p.H, i % (HD / 4) * 4, HD);
        if (DT != 0 && p.out_dtype != APT_F32) store_out4<DT>(p.out, 4 * (int64_t)i, o);
        else store_out4<0>(p.out, 4 * (int64_t)i, o);
    }
}

}  // namespace
