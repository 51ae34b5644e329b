// Merge of the ranges' partials, in a kernel of its own or by the last workgroup of the item kernel:
//   out[r][h][c] = sum_s acc_s[c] 2^(m_s - M) / sum_s l_s 2^(m_s - M)
#pragma once
#include "apt_device.h"

namespace {

// THROUGH: the partials were written by this launch (put_partial), on any XCD
template <bool THROUGH, typename T> __device__ inline T get_partial(const T* at) {
    if constexpr (!THROUGH) return *at;
    uint64_t w[sizeof(T) / 8];
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 8; ++i) w[i] = __hip_atomic_load((const uint64_t*)at + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(T, w);
}
// ranges of a (request, head) pair and its first partial
struct MergeOf {
    int ns;
    int64_t base;
};
template <typename Params> __device__ inline MergeOf merge_of(const Params& p, int pair) {
    const int r = pair / p.H;
    return {p.plan[APT_PW_HEADER + APT_PA_SPLIT_COUNT * p.B + r],
            (int64_t)p.plan[APT_PW_HEADER + APT_PA_WS_OFFSET * p.B + r] * p.H + pair % p.H};
}
// Four channels from c on.  Bound by latency: the partials of up to N ranges are asked for at once.  ALL: there are no more.
template <bool THROUGH, int N, bool ALL, typename Params>
__device__ __forceinline__ float4 merged4(const Params& p, const MergeOf& m, int c, int HD) {
    float2 ml[N];
    float4 acc[N];
    auto load_ml = [&](int s0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < m.ns) ml[i] = get_partial<THROUGH>(p.ws_ml + m.base + (int64_t)(s0 + i) * p.H);
    };
    auto load_acc = [&](int s0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < m.ns) acc[i] = get_partial<THROUGH>((const float4*)(p.ws_acc + (m.base + (int64_t)(s0 + i) * p.H) * HD + c));
    };
    load_ml(0);
    load_acc(0);
    const int end = ALL ? 1 : m.ns;
    float M = kSentinel;
    for (int s0 = 0; s0 < end; s0 += N) {
        if (s0) load_ml(s0);
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (s0 + i < m.ns) M = fmaxf(M, ml[i].x);
    }
    if (end > N) load_ml(0);
    float L = 0.f;
    float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < end; s0 += N) {
        if (s0) load_ml(s0), load_acc(s0);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (s0 + i >= m.ns) continue;
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

// At the end of every item of a launch of one workgroup per item (p.out set): the workgroup that is last to get here merges the
// partials, so that a small step is a launch shorter.  A workgroup takes its ticket when all of its partial is written through, and the
// last one reads them past the caches of its XCD.  KV-kind requests alone: a ticket for every eighth head, in the words where a plan with
// hidden-kind items has its queues, so that up to eight workgroups merge a part each and no more than an eighth of the workgroups wait
// for each other.  The tickets are 0 between launches.
// Bound by the latencies of the store, the ticket, the partials and of the code itself, which such a workgroup runs once: four channels per
// thread and no more (apt_items_merge sees to it), where their partials lie is asked for before the ticket, and N ranges without a loop
// around them.  Attention call in a graph, us, a kernel of its own / eight ranges in a loop, looked up behind the ticket / so: KV-kind,
// fp16, 8 heads of 128, 1100 tokens 11.4 / 11.2 / 10.5, 24 heads, 1324 tokens 12.2 / 12.4 / 11.7, 16 heads, 2 x 900 11.9 / 12.4 / 11.5.
template <int DT, int HD, int N, bool KV_ALONE> __device__ __forceinline__ void merge_by_last(const ItemParams& p, int h, char* lds) {
    if (!p.out) return;
    constexpr int G = KV_ALONE ? APT_MERGE_GROUPS : 1;
    const int g = h % G, heads = (p.H - g + G - 1) / G;  // this workgroup's part: heads g, g + G, ...
    const int n = p.B * heads * (HD / 4), i = threadIdx.x;
    const int at = min(i, n - 1) / (HD / 4), pair = at / heads * p.H + g + G * (at % heads);
    const MergeOf of = merge_of(p, pair);
    wait_vmcnt<0>();
    __syncthreads();
    int32_t* const word = KV_ALONE ? p.kv_ticket - APT_PW_KV_TICKET + APT_PW_QUEUE0 + g : p.kv_ticket;
    int* ticket = (int*)lds;
    if (threadIdx.x == 0) *ticket = __hip_atomic_fetch_add(word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*ticket != p.n_items / p.H * heads - 1) return;
    if (threadIdx.x == 0) *word = 0;
    if (i >= n) return;
    const int c = i % (HD / 4) * 4;
    const float4 o = p.most_ranges <= N ? merged4<true, N, true>(p, of, c, HD) : merged4<true, N, false>(p, of, c, HD);
    if (DT != 0 && p.out_dtype != APT_F32) store_out4<DT>(p.out, (int64_t)pair * HD + c, o);
    else store_out4<0>(p.out, (int64_t)pair * HD + c, o);
}

}  // namespace
