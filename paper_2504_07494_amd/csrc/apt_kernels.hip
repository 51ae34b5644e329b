// HIP kernels (gfx950) of the hybrid-cache decode attention step and their launchers.
//
//   items kernel   one workgroup (4 wavefronts of 64) per work item of the plan:
//                    KV-kind item      streams the K and V rows of one head over a token
//                                      range, online softmax per 16-lane group (HBM bound)
//                    hidden-kind item  projects K_h, V_h of a tile of tokens from the gathered
//                                      hidden rows on the matrix cores (apt_mfma.inc packed
//                                      weights, apt_raw16.hip and apt_raw32.hip raw ones) and
//                                      attends to them from registers
//                  every item writes one partial (m, l, acc[head_dim]) in fp32
//   merge kernel   combines a request's partials per head and normalises; in small calls the last workgroup of the items
//                  kernel does (apt_merge.h)
//   whole kernel   KV-kind requests alone, where takes_whole says so: a workgroup per request and head, no partials
//   apt_absorbed.inc, apt_absorb*.hip: the hidden-kind requests without the projection (opt-in, APT_HIDDEN_ABSORBED)
//   cache append / cache write, weight packing, calibration kernels
//
// Scores are kept in base-2 units: s2 = softmax_scale*log2(e)*<q,k>, weights 2^(s2 - m).
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <mutex>
#include <type_traits>
#include "apt_device.h"
#include "apt_hybrid_bench.h"
#include "apt_launch.h"
#include "apt_merge.h"
#include "apt_absorb_tile.h"
#include "apt_pack.h"

// Workspace of apt_hybrid_decode_attn_static: one copy per device, held until the process ends.  In host code this
// name is only a handle for hipGetSymbolAddress; the device address is looked up once per device (device_setup).
static __device__ __align__(256) unsigned char scratch[APT_STATIC_WORKSPACE_BYTES];

namespace {

// ---------------------------------------------------------------------------------
// KV-kind items alone, one workgroup per item (plans without hidden-kind items; fp32, before the absorbed-weight kernels)
// ---------------------------------------------------------------------------------
template <int DT, int HD, int NW>
__global__ __launch_bounds__(NW * 64) void apt_items_kernel(ItemParams p) {
    extern __shared__ __align__(16) char lds[];
    const int item = blockIdx.x + p.item_base;
    if (item >= p.n_items) return;
    const int4 it = ((const int4*)(p.plan + p.items_off))[item];
    kv_item_through<DT, HD, NW>(p, it.x, it.y, it.z, it.w, lds);
    merge_by_last<DT, HD, NW == 16 ? APT_MERGE_RANGES_MANY : APT_MERGE_RANGES, true>(p, it.y, lds);
}

// Whole contexts, one workgroup per request and head, straight to the output: no partials and no merge (see takes_whole).
// in_items: the plan has one item per request and head (longest first), else they are taken as they come.
template <int DT, int HD, int NW, int ODT>
__global__ __launch_bounds__(NW * 64) void apt_whole_kernel(ItemParams p, char* out, int in_items) {
    extern __shared__ __align__(16) char lds[];
    int r = blockIdx.x / p.H, h = blockIdx.x % p.H;
    if (in_items) {
        const int4 it = ((const int4*)(p.plan + p.items_off))[blockIdx.x];
        r = it.x, h = it.y;
    }
    const int n = p.plan[APT_PW_HEADER + APT_PA_CTX_LEN * p.B + r];
    kv_range<DT, HD, NW>(p, r, h, 0, n, lds, [&](int c, float, float L, float A) { store_out<ODT>(out, ((int64_t)r * p.H + h) * HD + c, A / L); });
}

// ---------------------------------------------------------------------------------
// merge kernel
// ---------------------------------------------------------------------------------
// The merge's own parameters: 56 bytes of kernel arguments, not the 300 of ItemParams (step of the smallest batches 0.2-0.3 us less).
struct MergeParams {
    const int32_t* plan;
    int32_t* kv_ticket;
    const float* ws_acc;
    const float2* ws_ml;
    int32_t B, H;
};

// a thread per four channels
template <int ODT>
__global__ __launch_bounds__(kThreads) void apt_merge_kernel(MergeParams p, char* out, int HD) {
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (gid == 0) *p.kv_ticket = 0;         // the item kernel of this call is done: ready for the next call
    if (4 * gid >= (int64_t)p.B * p.H * HD) return;
    const int64_t pair = 4 * gid / HD;
    store_out4<ODT>(out, 4 * gid, merged4<false, 8, false>(p, merge_of(p, (int)pair), (int)(4 * gid % HD), HD));
}

// ---------------------------------------------------------------------------------
// weight packing for the MFMA kernel (one-off per layer)
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void apt_pack_kernel(const uint16_t* W_K, const uint16_t* W_V, uint4* packed,
                                                            int d, int H) {
    // one thread per 16-byte unit; consecutive threads take consecutive channels so
    // that the strided reads of W coalesce
    const int nkt = d / kBK;
    constexpr int units = kBK / 8;                      // 16-byte units per row
    const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t total = (int64_t)H * nkt * 256 * units;
    if (gid >= total) return;
    const int row = (int)(gid % 256);
    const int c = (int)((gid / 256) % units);
    const int kt = (int)((gid / (256 * units)) % nkt);
    const int h = (int)(gid / (256 * units * (int64_t)nkt));
    const uint16_t* W = row < 128 ? W_K : W_V;
    const int ch = h * 128 + (row & 127);
    const int k0 = kt * kBK + c * 8;
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = W[(int64_t)(k0 + e) * d + ch];
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16);
    o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16);
    o.w = v[6] | ((uint32_t)v[7] << 16);
    packed[((int64_t)h * nkt + kt) * (256 * units) + row * units + (c ^ swz16(row))] = o;
}

// A small plan blob rides in the kernel's arguments: one launch, no copy engine, and the host buffer is free at once.
// The smallest steps are bound by the host: this call takes 3.7 us there, the asynchronous copy 6.0 and the event that has
// to follow it another 5.
struct PlanWords { int32_t w[APT_PLAN_INLINE_BYTES / 4]; };
__global__ __launch_bounds__(kThreads) void apt_plan_store_kernel(int32_t* dst, PlanWords blob, int n) {
    for (int i = threadIdx.x; i < n; i += kThreads) dst[i] = blob.w[i];
}

// A larger blob in page-locked memory is read by a kernel, straight over the bus (past the caches: the host rewrites its buffers
// between steps).  The runtime copies up to 16 KB by a kernel of its own and gives more to a copy engine, which starts and ends with a
// wait between the two queues.  Time on the stream beside a copy by the runtime, us: 4 to 16 KB 2.5 and 2.5, 32 KB 15.4 and 2.9, 128 KB
// 17.7 and 4.7, 512 KB 24.9 and 12.2, 2 MB 53 and 41; the call on the host, from Python, 2.1 and 3.6.
constexpr size_t kPlanCopyBytes = 16384;             // up to this size the runtime's copy takes no longer
__global__ __launch_bounds__(kThreads) void apt_plan_copy_kernel(uint64_t* dst, const uint64_t* src, int64_t n, int words) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
        dst[i] = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if ((words & 1) && blockIdx.x == 0 && threadIdx.x == 0)          // the last word of an odd number
        ((int32_t*)dst)[words - 1] = __hip_atomic_load((const int32_t*)src + words - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Whether apt_plan_copy_kernel can take the blob: all of it lies in one page-locked allocation that the device sees at the same address, its
// destination in one allocation of the device too, and the current device, the stream's and that of plan_dev are one.  Anything
// else, buffers that are too small among them, is for the runtime's copy to serve or to refuse.
static bool copied_by_kernel(const void* host, const void* dev, size_t bytes, hipStream_t st) {
    hipPointerAttribute_t from = {}, to = {};
    int current = -1, streams = -1;
    auto ok = [](hipError_t e) {                          // a query's error is not left for a later call to find
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipSuccess;
    };
    auto in_one_allocation = [&](const void* p) {
        void* start = nullptr;
        size_t size = 0;
        if (!ok(hipPointerGetAttribute(&start, HIP_POINTER_ATTRIBUTE_RANGE_START_ADDR, (hipDeviceptr_t)p)) ||
            !ok(hipPointerGetAttribute(&size, HIP_POINTER_ATTRIBUTE_RANGE_SIZE, (hipDeviceptr_t)p)))
            return false;
        const uintptr_t at = (uintptr_t)p - (uintptr_t)start;
        return at <= size && bytes <= size - at;
    };
    return ok(hipPointerGetAttributes(&from, host)) && from.type == hipMemoryTypeHost && from.devicePointer == host &&
           ok(hipPointerGetAttributes(&to, dev)) && to.type == hipMemoryTypeDevice && in_one_allocation(host) && in_one_allocation(dev) &&
           ok(hipGetDevice(&current)) && ok(hipStreamGetDevice(st, &streams)) && streams == current && to.device == current;
}

// Where the cache calls put a new token's vector: 16-byte unit u of it (row_units in all; a unit never straddles a head, as
// head_dim * element size is a multiple of 16) goes to unit first + (u / head_units) * head_stride + u % head_units of its block.
struct CacheRow {
    char* block;
    uint32_t first, head_stride;
    int log2_head_units;
};
struct CacheParams {
    const char *x_new, *k_new, *v_new;
    char *k_pages, *v_pages, *hidden_pages;
    const int32_t* block_tables;
    const int32_t* ctx_lens;
    const uint8_t* cache_kind;
    int B, d, hd, bs, log2_bs, max_blocks, eb;
};
// mat: 0 = hidden vector or K, 1 = V
__device__ inline CacheRow cache_row(const CacheParams& p, int r, int token, bool hidden, int mat) {
    const int slot = token & (p.bs - 1), head_units = p.hd * p.eb / 16;
    const int64_t block = p.block_tables[((int64_t)r * 2 + mat) * p.max_blocks + (token >> p.log2_bs)];
    char* pages = hidden ? p.hidden_pages : mat ? p.v_pages : p.k_pages;
    return {pages + block * p.bs * p.d * p.eb, (uint32_t)slot * (hidden ? p.d * p.eb / 16 : head_units),
            (uint32_t)(hidden ? head_units : p.bs * head_units), 31 - __builtin_clz(head_units)};
}
__device__ inline void store_unit(const CacheRow& row, uint32_t u, const uint4& v) {
    const uint32_t at = row.first + (u >> row.log2_head_units) * row.head_stride + (u & ((1u << row.log2_head_units) - 1));
    const u32x4_t w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (u32x4_t*)(row.block + (int64_t)at * 16));
}

// Cache append: one workgroup per request.  Bound by its chain of memory latencies (length, map entry, store); the vector itself
// is read beside that chain.
__global__ __launch_bounds__(kThreads) void apt_append_kernel(CacheParams p) {
    constexpr int kUnits = 3;                            // units of K (and of V) a thread has in flight
    const int r = blockIdx.x, row_units = p.d * p.eb / 16;
    const bool hidden = p.cache_kind[r] == APT_KIND_HIDDEN;
    const int j = p.ctx_lens[r] - 1;
    if (j < 0) return;
    const char* src0 = (hidden ? p.x_new : p.k_new) + (int64_t)r * row_units * 16;
    const char* src1 = hidden ? src0 : p.v_new + (int64_t)r * row_units * 16;
    const CacheRow row0 = cache_row(p, r, j, hidden, 0), row1 = hidden ? row0 : cache_row(p, r, j, false, 1);
    for (int u0 = threadIdx.x; u0 < row_units; u0 += kUnits * kThreads) {
        uint4 a[kUnits], b[kUnits];
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = u0 + i * kThreads;
            if (u < row_units) {
                a[i] = load16_stream(src0 + u * 16);
                if (!hidden) b[i] = load16_stream(src1 + u * 16);
            }
        }
#pragma unroll
        for (int i = 0; i < kUnits; ++i) {
            const int u = u0 + i * kThreads;
            if (u < row_units) {
                store_unit(row0, u, a[i]);
                if (!hidden) store_unit(row1, u, b[i]);
            }
        }
    }
}

// Cache write of a run of new tokens per request (prefill, or several decoded tokens at once).  Grid (group of kWriteTokens new
// tokens, request, K or V; a hidden vector is matrix 0 alone): a wave per token and matrix, up to ten units per lane read before
// the first is stored.
// Bound by memory, and by where the workgroups of a moment read and write: with the groups of a request side by side they
// stream through neighbouring rows, with a group of every request in turn (the order before) through as many places as there
// are requests.  16 requests of 61..1021 tokens, half hidden-kind, d_model 5120 fp16 (292 MB read and written, a copy of
// as much 50 us, non-temporal 47): 85 us by request, a store behind each load, cached; 80 non-temporal; 73 with ten units in
// flight and four tokens to a workgroup instead of eight; 58 by group.  Eight tokens by group 60, cached accesses 63; runs of 4
// tokens of one head instead of whole rows 58, of 8 tokens 64, of 16 tokens 74.
// (Those are passes over the same buffers.)  Buffers that no pass of the last gigabytes has touched, as a prefill has them, by request with
// a store behind each load / as it is: this shape 81 / 52, d_model 2048 35 / 22, 7168 114 / 73, 9216 148 / 95 (14 and 18 units a lane, in
// two rounds), a KV-kind request of 500 tokens, d_model 5120 (20 MB) 32 / 5.2, 4 requests at d_model 9216 (38 MB) 48 / 11.
constexpr int kWriteTokens = 4;
constexpr int kWriteUnits = 10;
constexpr int kMaxNewTokens = 524280;                // of a request and call, as the header states
__global__ __launch_bounds__(kWriteTokens * 64) void apt_write_kernel(CacheParams p, const int32_t* new_offsets) {
    const int t = blockIdx.x * kWriteTokens + (threadIdx.x >> 6), lane = threadIdx.x & 63, mat = blockIdx.z;
    const int row_units = p.d * p.eb / 16;
    for (int r = blockIdx.y; r < p.B; r += gridDim.y) {
        const int row0 = new_offsets[r], n_new = new_offsets[r + 1] - row0;
        const int first = p.ctx_lens[r] - n_new;         // position of the first new token
        if (t >= n_new || first < 0) continue;           // first < 0: more new tokens than the request holds, nothing is written
        const bool hidden = p.cache_kind[r] == APT_KIND_HIDDEN;
        if (hidden && mat) continue;
        const CacheRow row = cache_row(p, r, first + t, hidden, mat);
        const char* src = (hidden ? p.x_new : mat ? p.v_new : p.k_new) + (int64_t)(row0 + t) * row_units * 16;
        for (int u0 = lane; u0 < row_units; u0 += kWriteUnits * 64) {
            uint4 v[kWriteUnits];
#pragma unroll
            for (int i = 0; i < kWriteUnits; ++i)
                if (u0 + 64 * i < row_units) v[i] = load16_stream(src + (u0 + 64 * i) * 16);
#pragma unroll
            for (int i = 0; i < kWriteUnits; ++i)
                if (u0 + 64 * i < row_units) store_unit(row, u0 + 64 * i, v[i]);
        }
    }
}

__global__ __launch_bounds__(kThreads) void apt_copy_kernel(uint4* dst, const uint4* src, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (; i < n; i += stride) dst[i] = src[i];
}

// Register-only MFMA loop: 4 waves per workgroup, a 128 x 128 accumulator tile per wave (256 registers), no
// memory traffic.  Measures the rate the matrix pipes sustain.  With random_operands the operand registers
// hold values of magnitude ~1 with random mantissas and signs (what real activations look like to the
// multipliers) instead of constants.  VARIANT 0 / 2: 16 independent 32x32x16 MFMAs per iteration (fp16 /
// bf16); 1 / 3: 64 independent 16x16x32 MFMAs per iteration (fp16 / bf16; twice the flops per iteration).
template <int VARIANT>
__global__ __launch_bounds__(kThreads) void apt_mfma_probe_kernel(float* out, int iters, int random_operands) {
    constexpr bool kSmall = (VARIANT & 1) != 0;          // 16x16x32 tiles
    constexpr int DT = (VARIANT & 2) ? 2 : 1;
    constexpr int NF = kSmall ? 8 : 4;                   // operand fragments per side
    uint4 a[NF], b[NF];
    uint32_t x = (threadIdx.x * 2654435761u) ^ (blockIdx.x * 40503u + 12345u);
    const uint32_t one = DT == 1 ? 0x3c003c00u : 0x3f803f80u, half = DT == 1 ? 0x38003800u : 0x3f003f00u;
    const uint32_t keep = DT == 1 ? 0x83ff83ffu : 0x807f807fu;      // sign and mantissa bits
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        a[i] = make_uint4(one, one, one, one);
        b[i] = make_uint4(half, half, half, half);
        if (random_operands) {
            auto nxt = [&]() { x ^= x << 13; x ^= x >> 17; x ^= x << 5; return (x & keep) | one; };
            a[i] = make_uint4(nxt(), nxt(), nxt(), nxt());
            b[i] = make_uint4(nxt(), nxt(), nxt(), nxt());
        }
    }
    float sum = 0.f;
    if constexpr (!kSmall) {
        f32x16_t acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
        for (int it = 0; it < iters; ++it) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i * 4 + j] = mfma32<DT>(a[i], b[j], acc[i * 4 + j]);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum += acc[i][e];
    } else {
        f32x4_t acc[64];
#pragma unroll
        for (int i = 0; i < 64; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][e] = 0.f;
        for (int it = 0; it < iters; ++it) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if constexpr (DT == 1)
                        acc[i * 8 + j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, a[i]),
                                                                                __builtin_bit_cast(h8_t, b[j]), acc[i * 8 + j], 0, 0, 0);
                    else
                        acc[i * 8 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, a[i]),
                                                                                 __builtin_bit_cast(bf8_t, b[j]), acc[i * 8 + j], 0, 0, 0);
                }
        }
#pragma unroll
        for (int i = 0; i < 64; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += acc[i][e];
    }
    out[(int64_t)blockIdx.x * kThreads + threadIdx.x] = sum;
}

// ---------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------
// A CU holds 16 waves of these kernels.  Up to one workgroup per CU, a workgroup has all of them: the range of a lone 1237-token
// request of 40 heads takes 8.8 us instead of 11.4 (of 1000 tokens, three such requests of 49 heads, 10.5 instead of 12.6).
// Eight waves for up to two workgroups per CU gave nothing (320 to 448 items 16.4 us, with four 15.4).
// most16: workgroups up to which they have 16 waves, the number of CUs; 0 where the caller has fixed kv_chunk, so that a request's sums
// are the same in every batch.
template <int DT, int HD> int launch_items(const ItemParams& p, int most16, hipStream_t st) {
    const int n = p.n_items - p.item_base;
    if (n <= most16) hipLaunchKernelGGL((apt_items_kernel<DT, HD, 16>), dim3(n), dim3(1024), (KvItem<DT, HD, 16>::kLds), st, p);
    else hipLaunchKernelGGL((apt_items_kernel<DT, HD, 4>), dim3(n), dim3(kThreads), (KvItem<DT, HD, 4>::kLds), st, p);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

// Whether the last workgroups of the item kernel merge the partials, by apt_items_merge.  Packed weights and the absorbed-weight path have a
// launch of their own that ends the call.
bool merges_by_itself(const ItemParams& p, int hd, int himpl, int most16) {
    if (p.n_hidden_items > 0 && himpl != APT_HIDDEN_VALU) return false;
    const bool alone = p.n_hidden_items == 0;
    return apt_items_merge(alone, alone && p.n_items <= most16 ? 1024 : kThreads, p.B, p.H, hd, p.n_items, p.most_ranges);
}
// Batches of KV-kind requests that need no partials.  Every context is one range of the plan; or the ranges are the planner's own choice
// (most16 > 0), there are no more (request, head) pairs than CUs, and the contexts alone do not take longer than ranges of them on
// more CUs and the merge would.  GPU time decides, by the times that both took (us; the longest context in KB, all of them in MB):
//   - with a merge kernel, on 296 batches of 1 to 30 requests and 8 to 72 heads, equal and ragged lengths of 250 to 2048 tokens, rows of
//     128, 256 and 512 bytes (up to one range per CU: 16 waves a range, else four).  The choice took 0.4 % longer than the better of the
//     two on average; by the longest context at 57 KB/us alone it was 2.9 %, 36 % at most (attention call, fp16, ranges and merge /
//     whole: 40 heads, 3 requests of up to 1743 tokens 17.7 / 22.8; 72 heads, 3 of 2048 41.4 / 35.2; 32 heads, 8 of 1000 24.0 / 20.9);
//   - with a merge by the last workgroups (merges), on 260 batches of 1 to 12 requests and 1 to 72 heads, in a graph: 0.2 % longer than
//     the better one, 6 % at most; by the line above 2.6 % and 41 % (2 heads of 64, bf16, 6 requests of 739..1269 tokens 7.9 / 11.1; one
//     head of 64, 8 of 789..1282 7.8 / 10.9; 9 heads, bf16, 843 tokens 10.4 / 12.6; 32 heads, 563 tokens 11.1 / 9.8).
bool takes_whole(const ItemParams& p, const int32_t* pw, int row_bytes, int most16, bool merges) {
    if (p.n_hidden_items > 0) return false;
    if (pw[APT_PW_NPARTIALS] == p.B) return true;
    if ((int64_t)p.B * p.H > most16 || p.max_blocks > 16 * APT_KV_MAX_PAGES_PER_WAVE) return false;
    const int32_t* lens = pw + APT_PW_HEADER + APT_PA_CTX_LEN * p.B;
    int64_t longest = 0, tokens = 0;
    for (int r = 0; r < p.B; ++r) {
        longest = std::max<int64_t>(longest, lens[r]);
        tokens += lens[r];
    }
    const double kb = 2e-3 * row_bytes, all = 1e-3 * kb * (double)tokens * p.H;
    const double context = kb * (double)longest, range = kb * (double)std::min<int64_t>(longest, p.kv_chunk);
    if (merges) return 4.2 + context / 58.0 + all / 16.9 <= 5.5 + range / 63.5 + all / 12.3;
    return 3.0 + context / 68.0 + all / 13.4 <= (p.n_items <= most16 ? 6.4 + range / 90.0 + all / 11.0 : 5.5 + all / 6.6);
}
template <int DT, int HD, int NW, int ODT> void launch_whole_nw(const ItemParams& p, char* out, int in_items, hipStream_t st) {
    hipLaunchKernelGGL((apt_whole_kernel<DT, HD, NW, ODT>), dim3(p.B * p.H), dim3(NW * 64), (KvItem<DT, HD, NW>::kLds), st, p, out, in_items);
}
template <int DT, int HD> int launch_whole(const ItemParams& p, const int32_t* pw, char* out, int out_dtype, int most16, hipStream_t st) {
    const int in_items = pw[APT_PW_NPARTIALS] == p.B;
    const bool few = (int64_t)p.B * p.H <= most16;
    if (DT == 0 || out_dtype == APT_F32) few ? launch_whole_nw<DT, HD, 16, 0>(p, out, in_items, st) : launch_whole_nw<DT, HD, 4, 0>(p, out, in_items, st);
    else few ? launch_whole_nw<DT, HD, 16, DT>(p, out, in_items, st) : launch_whole_nw<DT, HD, 4, DT>(p, out, in_items, st);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

#include "apt_absorbed.inc"

template <int DT, int HD>
int launch_items_impl(ItemParams& p, int himpl, int n_wg, int most16, bool dealt, hipStream_t st) {
    if (p.n_hidden_items == 0) return launch_items<DT, HD>(p, most16, st);
    if (himpl == APT_HIDDEN_ABSORBED) {
        if (DT == 0 && p.n_hidden_items < p.n_items) {
            p.item_base = p.n_hidden_items;      // the KV-kind items, one workgroup each (16-bit inputs: with the absorbed queries)
            const int rc = launch_items<DT, HD>(p, most16, st);
            if (rc) return rc;
        }
        return launch_absorbed<DT>(p, HD, n_wg, st);
    }
    if (himpl == APT_HIDDEN_VALU) {
        if constexpr (DT == 0) return apt_launch_raw32(p, HD, st);
        else return apt_launch_raw16(p, DT, HD, st);
    }
    if constexpr (DT != 0 && HD == 128) {
        return dealt ? apt_launch_mfma<DT, true>(p, n_wg, st) : apt_launch_mfma<DT, false>(p, n_wg, st);
    }
    return APT_ESHAPE;
}

// ---------------------------------------------------------------------------------
// per-device set-up: made once per device under a mutex, read-only afterwards
// ---------------------------------------------------------------------------------
struct DeviceState {
    bool ready = false;
    int n_wg = 0;             // workgroups of the persistent MFMA launch
    void* scratch_ptr = nullptr;  // this device's copy of the static workspace
};
constexpr int kMaxDevices = 64;
std::mutex g_setup_mutex;
DeviceState g_devices[kMaxDevices];

int device_setup(const DeviceState** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return APT_EHIP;
    std::lock_guard<std::mutex> lock(g_setup_mutex);
    DeviceState& ds = g_devices[dev];
    if (!ds.ready) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return APT_EHIP;
        ds.n_wg = cus >= 8 ? (cus / 8) * 8 : 8;
        // every kernel that can be launched with more than 64 KB of dynamic LDS
        const bool ok = apt_setup_mfma<1, false>() && apt_setup_mfma<1, true>() && apt_setup_mfma<2, false>() && apt_setup_mfma<2, true>() &&
                        apt_setup_raw16() &&
                        apt_raise_lds_limit(apt_absorb_score_kernel<0>) && apt_raise_lds_limit(apt_absorb_pv_kernel<0>) &&
                        apt_setup_absorb_scores16() &&
                        apt_setup_absorb_pv16() && apt_setup_absorb_out16();
        if (!ok) return APT_EHIP;
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return APT_EHIP;
        ds.scratch_ptr = ptr;
        ds.ready = true;
    }
    if (out) *out = &ds;
    return APT_OK;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

extern "C" int apt_init(void) { return device_setup(nullptr); }

extern "C" int apt_plan_upload(const void* plan_host, void* plan_dev, void* stream) {
    apt_plan_info info;
    int rc = apt_plan_get_info(plan_host, &info);
    if (rc) return rc;
    if (!plan_dev) return APT_EINVAL;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
    const bool small = info.plan_bytes <= APT_PLAN_INLINE_BYTES && ((uintptr_t)plan_dev & 3) == 0;
    const bool large = info.plan_bytes > kPlanCopyBytes && (((uintptr_t)plan_dev | (uintptr_t)plan_host) & 7) == 0;
    if (small || large) {
        if (hipStreamIsCapturing((hipStream_t)stream, &capture) != hipSuccess) {
            (void)hipGetLastError();
            capture = hipStreamCaptureStatusActive;
        }
    }
    if (capture == hipStreamCaptureStatusNone && large) {
        if (copied_by_kernel(plan_host, plan_dev, info.plan_bytes, (hipStream_t)stream)) {
            int words = (int)(info.plan_bytes / 4);
            int64_t n = words / 2;
            const unsigned blocks = (unsigned)std::min<int64_t>((n + kThreads - 1) / kThreads, 256);
            void* args[] = {&plan_dev, &plan_host, &n, &words};
            return hipLaunchKernel((const void*)apt_plan_copy_kernel, dim3(blocks), dim3(kThreads), args, 0, (hipStream_t)stream) == hipSuccess
                       ? APT_OK : APT_EHIP;
        }
    } else if (capture == hipStreamCaptureStatusNone) {
        PlanWords blob;
        memcpy(blob.w, plan_host, info.plan_bytes);
        // the launch's own status: like the copy, this call neither fails for an error an earlier call left nor clears it
        int n = (int)(info.plan_bytes / 4);
        void* args[] = {&plan_dev, &blob, &n};
        return hipLaunchKernel((const void*)apt_plan_store_kernel, dim3(1), dim3(kThreads), args, 0, (hipStream_t)stream) == hipSuccess
                   ? APT_OK : APT_EHIP;
    }
    if (hipMemcpyAsync(plan_dev, plan_host, info.plan_bytes, hipMemcpyHostToDevice, (hipStream_t)stream) != hipSuccess)
        return APT_EHIP;
    return APT_OK;
}

extern "C" int apt_packed_weight_bytes(const apt_shape* s, size_t* bytes) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (!bytes) return APT_EINVAL;
    *bytes = (size_t)2 * rs.s.d_model * rs.s.d_model * rs.elem_bytes;
    return APT_OK;
}

extern "C" int apt_pack_weights(const apt_shape* s, const void* W_K, const void* W_V, void* packed, void* stream) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (!W_K || !W_V || !packed) return APT_EINVAL;
    if (rs.s.hidden_impl != APT_HIDDEN_MFMA) return APT_ESHAPE;
    const int d = rs.s.d_model, H = rs.s.n_heads;
    const int64_t total = (int64_t)H * (d / kBK) * 256 * (kBK / 8);
    const int64_t blocks = (total + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(apt_pack_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, (hipStream_t)stream,
                       (const uint16_t*)W_K, (const uint16_t*)W_V, (uint4*)packed, d, H);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

extern "C" int apt_cache_append(const apt_shape* s, int B, const void* x_new, const void* k_new, const void* v_new,
                                void* k_pages, void* v_pages, void* hidden_pages, const int32_t* block_tables,
                                const int32_t* ctx_lens_dev, const uint8_t* cache_kind_dev, void* stream) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (B < 1 || !block_tables || !ctx_lens_dev || !cache_kind_dev) return APT_EINVAL;
    if (!x_new && !k_new && !v_new) return APT_EINVAL;
    if ((x_new && !hidden_pages) || ((k_new || v_new) && (!k_new || !v_new || !k_pages || !v_pages))) return APT_EINVAL;
    if (!aligned16(x_new) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(k_pages) || !aligned16(v_pages) ||
        !aligned16(hidden_pages))
        return APT_EINVAL;
    int log2_bs = 0;
    while ((1 << log2_bs) < rs.s.block_size) ++log2_bs;
    const CacheParams p = {(const char*)x_new, (const char*)k_new, (const char*)v_new, (char*)k_pages, (char*)v_pages, (char*)hidden_pages,
                           block_tables, ctx_lens_dev, cache_kind_dev, B, rs.s.d_model, rs.s.head_dim, rs.s.block_size, log2_bs,
                           rs.s.max_blocks_per_req, rs.elem_bytes};
    hipLaunchKernelGGL(apt_append_kernel, dim3(B), dim3(kThreads), 0, (hipStream_t)stream, p);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

extern "C" int apt_cache_write(const apt_shape* s, int B, const int32_t* new_offsets_dev, int32_t max_new_tokens,
                               const void* x_new, const void* k_new, const void* v_new, void* k_pages, void* v_pages,
                               void* hidden_pages, const int32_t* block_tables, const int32_t* ctx_lens_dev,
                               const uint8_t* cache_kind_dev, void* stream) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (B < 1 || max_new_tokens < 1 || !new_offsets_dev || !block_tables || !ctx_lens_dev || !cache_kind_dev) return APT_EINVAL;
    if (!x_new && !k_new && !v_new) return APT_EINVAL;
    if ((x_new && !hidden_pages) || ((k_new || v_new) && (!k_new || !v_new || !k_pages || !v_pages))) return APT_EINVAL;
    if (!aligned16(x_new) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(k_pages) || !aligned16(v_pages) ||
        !aligned16(hidden_pages))
        return APT_EINVAL;
    if (max_new_tokens > kMaxNewTokens) return APT_ERANGE;
    int log2_bs = 0;
    while ((1 << log2_bs) < rs.s.block_size) ++log2_bs;
    const CacheParams p = {(const char*)x_new, (const char*)k_new, (const char*)v_new, (char*)k_pages, (char*)v_pages, (char*)hidden_pages,
                           block_tables, ctx_lens_dev, cache_kind_dev, B, rs.s.d_model, rs.s.head_dim, rs.s.block_size, log2_bs,
                           rs.s.max_blocks_per_req, rs.elem_bytes};
    // the second matrix only where there are K and V vectors
    const dim3 grid((unsigned)((max_new_tokens + kWriteTokens - 1) / kWriteTokens), std::min(B, 65535), k_new ? 2 : 1);
    hipLaunchKernelGGL(apt_write_kernel, grid, dim3(kWriteTokens * 64), 0, (hipStream_t)stream, p, new_offsets_dev);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

extern "C" int apt_copy_bytes(void* dst, const void* src, size_t bytes, void* stream) {
    if (!dst || !src || bytes == 0 || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) return APT_EINVAL;
    const int64_t n = (int64_t)(bytes / 16);
    int64_t blocks = (n + kThreads - 1) / kThreads;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(apt_copy_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, (hipStream_t)stream,
                       (uint4*)dst, (const uint4*)src, n);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

extern "C" int apt_probe_mfma(void* out, int n_workgroups, int iters, int random_operands, int variant, void* stream) {
    if (!out || n_workgroups < 1 || iters < 1 || variant < 0 || variant > 3) return APT_EINVAL;
    const dim3 grid(n_workgroups), block(kThreads);
    hipStream_t st = (hipStream_t)stream;
    if (variant == 0) hipLaunchKernelGGL(apt_mfma_probe_kernel<0>, grid, block, 0, st, (float*)out, iters, random_operands);
    else if (variant == 1) hipLaunchKernelGGL(apt_mfma_probe_kernel<1>, grid, block, 0, st, (float*)out, iters, random_operands);
    else if (variant == 2) hipLaunchKernelGGL(apt_mfma_probe_kernel<2>, grid, block, 0, st, (float*)out, iters, random_operands);
    else hipLaunchKernelGGL(apt_mfma_probe_kernel<3>, grid, block, 0, st, (float*)out, iters, random_operands);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

// The attention step behind all three entry points.  static_ws: the partials go to this device's static workspace
// (workspace / workspace_bytes are ignored) and nothing may be allocated.
static int decode_attn(const apt_shape* s, const void* plan_host, void* plan_dev,
                       const void* q, const void* k_pages, const void* v_pages, const void* hidden_pages,
                       const void* W_K, const void* W_V, const void* W_packed,
                       const void* b_K, const void* b_V, const int32_t* block_tables,
                       void* out, void* workspace, size_t workspace_bytes, bool static_ws, void* stream,
                       void* ev_begin, void* ev_end) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (!plan_host || !plan_dev || !q || !block_tables || !out || (!workspace && !static_ws)) return APT_EINVAL;
    if (static_ws && rs.s.hidden_impl == APT_HIDDEN_ABSORBED) return APT_ESHAPE;
    if (static_ws) workspace_bytes = APT_STATIC_WORKSPACE_BYTES;
    const int32_t* pw = (const int32_t*)plan_host;
    if (pw[APT_PW_MAGIC] != APT_PLAN_MAGIC) return APT_EINVAL;
    // the plan must have been made for this shape
    if (pw[APT_PW_HEADS] != rs.s.n_heads || pw[APT_PW_HEAD_DIM] != rs.s.head_dim ||
        pw[APT_PW_HIMPL] != rs.s.hidden_impl || pw[APT_PW_D_MODEL] != rs.s.d_model ||
        pw[APT_PW_BLOCK_SIZE] != rs.s.block_size || pw[APT_PW_MAX_BLOCKS] != rs.s.max_blocks_per_req ||
        pw[APT_PW_DTYPE] != rs.s.dtype)
        return APT_ESHAPE;
    // hidden-kind and KV-kind range lengths: the caller's, or the planner's choice for this batch where the caller left them open
    const int hidden_chunk = pw[APT_PW_HCHUNK], kv_chunk = pw[APT_PW_KCHUNK];
    const int shortest = std::min(APT_RAW_MIN_HIDDEN_CHUNK(rs.s.dtype), APT_RAW_PLAN_HIDDEN_CHUNK);
    if (rs.hidden_auto ? (hidden_chunk < shortest || hidden_chunk > rs.s.hidden_chunk) : hidden_chunk != rs.s.hidden_chunk)
        return APT_ESHAPE;
    if (rs.kv_auto ? (kv_chunk < rs.s.kv_chunk || kv_chunk > APT_MAX_AUTO_KV_CHUNK || !apt_kv_chunk_ok(kv_chunk, rs.s.block_size))
                   : kv_chunk != rs.s.kv_chunk)
        return APT_ESHAPE;
    const int n_items = pw[APT_PW_NITEMS], n_hidden = pw[APT_PW_NHIDDEN];
    const int B = pw[APT_PW_BATCH];
    const int64_t hidden_tokens = ((int64_t)pw[APT_PW_HTOK_HI] << 32) | (uint32_t)pw[APT_PW_HTOK_LO];
    const apt_ws_layout L = apt_ws_sections(pw[APT_PW_NPARTIALS], rs.s.n_heads, rs.s.head_dim, rs.s.hidden_impl,
                                            pw[APT_PW_NHIDREQ], hidden_tokens, n_hidden, rs.s.d_model, rs.s.dtype);
    if (workspace_bytes < L.total) return APT_EWORKSPACE;
    // 16-byte vector loads and stores: every base pointer has to be 16-byte aligned
    if ((!static_ws && !aligned16(workspace)) || !aligned16(q) || !aligned16(k_pages) || !aligned16(v_pages) || !aligned16(hidden_pages) ||
        !aligned16(W_K) || !aligned16(W_V) || !aligned16(W_packed) || !aligned16(b_K) || !aligned16(b_V) || !aligned16(plan_dev))
        return APT_EINVAL;
    if (rs.s.hidden_impl == APT_HIDDEN_ABSORBED && n_hidden > 0 && !pw[APT_PW_TILES_OFF]) return APT_EINVAL;   // a blob without the lists
    if (n_hidden < n_items && (!k_pages || !v_pages)) return APT_EINVAL;
    if (n_hidden > 0) {
        if (!hidden_pages || !b_K || !b_V) return APT_EINVAL;
        if (rs.s.hidden_impl == APT_HIDDEN_MFMA && !W_packed) return APT_EINVAL;
        if (rs.s.hidden_impl != APT_HIDDEN_MFMA && (!W_K || !W_V)) return APT_EINVAL;
    }
    int log2_bs = 0;
    while ((1 << log2_bs) < rs.s.block_size) ++log2_bs;
    // every argument is checked: now the device (first call on a device: its one-off set-up)
    const DeviceState* ds = nullptr;
    rc = device_setup(&ds);
    if (rc) return rc;
    if (static_ws) workspace = ds->scratch_ptr;

    ItemParams p;
    p.plan = (const int32_t*)plan_dev;
    p.kv_ticket = (int32_t*)plan_dev + APT_PW_KV_TICKET;
    p.q = (const char*)q;
    p.k_pages = (const char*)k_pages;
    p.v_pages = (const char*)v_pages;
    p.hidden_pages = (const char*)hidden_pages;
    p.W_K = (const char*)W_K;
    p.W_V = (const char*)W_V;
    p.W_packed = (const char*)W_packed;
    p.b_K = (const char*)b_K;
    p.b_V = (const char*)b_V;
    p.block_tables = block_tables;
    char* const ws = (char*)workspace;
    p.ws_acc = (float*)(ws + L.acc);
    p.ws_ml = (float2*)(ws + L.ml);
    p.ab_qt = (float*)(ws + L.qt);
    p.ab_cb = (float*)(ws + L.cb);
    p.ab_s = (float*)(ws + L.s);
    p.ab_ml = (float2*)(ws + L.stat);
    p.ab_yp = (float*)(ws + L.yp);
    p.ab_op = (float*)(ws + L.op);
    p.ab_pp = ws + L.pp;
    p.ab_tokens = hidden_tokens;
    p.n_hid_req = pw[APT_PW_NHIDREQ];
    p.wide_tiles = apt_pack_wide((uint32_t)pw[APT_PW_SHARED_TILES]);
    p.item_base = 0;
    p.ab_ks = 0;
    p.ab_tiles_off = rs.s.hidden_impl == APT_HIDDEN_ABSORBED ? pw[APT_PW_TILES_OFF] : 0;
    p.ab_tiles = p.ab_units = p.ab_units_off = p.ab_group = p.ab_rows = p.ab_os = p.ab_past = 0;
    if (p.ab_tiles_off) {
        p.ab_tiles = pw[p.ab_tiles_off];
        p.ab_group = pw[p.ab_tiles_off + 1];
        p.ab_tiles_off += 2;
        p.ab_units_off = p.ab_tiles_off + p.ab_tiles;
        p.ab_units = pw[APT_PW_WORDS] - p.ab_units_off;
    }
    p.B = B; p.H = rs.s.n_heads; p.d = rs.s.d_model; p.bs = rs.s.block_size; p.log2_bs = log2_bs;
    p.max_blocks = rs.s.max_blocks_per_req;
    p.n_items = n_items; p.n_hidden_items = n_hidden;
    p.hidden_chunk = hidden_chunk; p.kv_chunk = kv_chunk; p.items_off = pw[APT_PW_ITEMS_OFF];
    p.scale_log2e = rs.s.softmax_scale * 1.4426950408889634f;
    // (an argument of the launcher alone: as a word more in ItemParams it made the six kernels of a short absorbed call begin later, 71 heads,
    // five requests of 20..71 tokens 100.0 -> 100.6 us)
    bool dealt = false;
    if (rs.s.hidden_impl == APT_HIDDEN_MFMA && n_hidden > 0) {
        const int32_t *lens = pw + APT_PW_HEADER + APT_PA_CTX_LEN * B, *kinds = pw + APT_PW_HEADER + APT_PA_KIND * B;
        const bool rows320 = hidden_chunk == APT_MFMA_HIDDEN_CHUNK || p.wide_tiles;
        const int64_t kv_tokens = (((int64_t)pw[APT_PW_TOK_HI] << 32) | (uint32_t)pw[APT_PW_TOK_LO]) - hidden_tokens;
        dealt = (rows320 ? apt_deals<10> : apt_deals<8>)(lens, kinds, B, kv_tokens, p.H, p.d, hidden_chunk, (uint32_t)pw[APT_PW_SHARED_TILES], ds->n_wg);
    }
    hipStream_t st = (hipStream_t)stream;

    const int dt = rs.s.dtype, hd = rs.s.head_dim, hi = rs.s.hidden_impl;
    if (ev_begin && hipEventRecord((hipEvent_t)ev_begin, st) != hipSuccess) return APT_EHIP;
    const int most16 = rs.kv_auto ? ds->n_wg : 0;
    const int32_t* ranges = pw + APT_PW_HEADER + APT_PA_SPLIT_COUNT * B;
    p.most_ranges = *std::max_element(ranges, ranges + std::min(B, 256));       // more requests never merge by themselves
    const bool merges = merges_by_itself(p, hd, hi, most16);
    const bool whole = takes_whole(p, pw, hd * rs.elem_bytes, most16, merges);
    p.out = merges && !whole ? (char*)out : nullptr;
    p.out_dtype = rs.s.out_dtype;
    auto launch = [&](auto dtype, auto head_dim) {
        constexpr int DT = decltype(dtype)::value, HD = decltype(head_dim)::value;
        return whole ? launch_whole<DT, HD>(p, pw, (char*)out, rs.s.out_dtype, most16, st)
                     : launch_items_impl<DT, HD>(p, hi, ds->n_wg, most16, dealt, st);
    };
    auto launch_hd = [&](auto dtype) {
        return hd == 64 ? launch(dtype, std::integral_constant<int, 64>{}) : launch(dtype, std::integral_constant<int, 128>{});
    };
    if (dt == APT_F32) rc = launch_hd(std::integral_constant<int, 0>{});
    else if (dt == APT_F16) rc = launch_hd(std::integral_constant<int, 1>{});
    else rc = launch_hd(std::integral_constant<int, 2>{});
    if (rc) return rc;
    // the last kernel of the absorbed-weight path sums the output partials of its requests: it belongs to the interval
    const bool absorbed = hi == APT_HIDDEN_ABSORBED && n_hidden > 0;
    if (ev_end && !absorbed && hipEventRecord((hipEvent_t)ev_end, st) != hipSuccess) return APT_EHIP;

    if (whole || p.out) return APT_OK;

    const unsigned blocks = (unsigned)(((int64_t)B * rs.s.n_heads * hd / 4 + kThreads - 1) / kThreads);
    auto launch_merge = [&](auto kern, const auto& params) { hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), 0, st, params, (char*)out, hd); };
    if (absorbed) {
        if (rs.s.out_dtype == APT_F32) launch_merge(dt == APT_F32 ? apt_absorb_merge_kernel<0, 0> : dt == APT_F16 ? apt_absorb_merge_kernel<1, 0> : apt_absorb_merge_kernel<2, 0>, p);
        else if (rs.s.out_dtype == APT_F16) launch_merge(apt_absorb_merge_kernel<1, 1>, p);
        else launch_merge(apt_absorb_merge_kernel<2, 2>, p);
    } else {
        const MergeParams mp = {p.plan, p.kv_ticket, p.ws_acc, p.ws_ml, p.B, p.H};
        launch_merge(rs.s.out_dtype == APT_F32 ? apt_merge_kernel<0> : rs.s.out_dtype == APT_F16 ? apt_merge_kernel<1> : apt_merge_kernel<2>, mp);
    }
    if (hipGetLastError() != hipSuccess) return APT_EHIP;
    if (ev_end && absorbed && hipEventRecord((hipEvent_t)ev_end, st) != hipSuccess) return APT_EHIP;
    return APT_OK;
}

extern "C" int apt_hybrid_decode_attn_timed(const apt_shape* s, const void* plan_host, void* plan_dev,
                                            const void* q, const void* k_pages, const void* v_pages, const void* hidden_pages,
                                            const void* W_K, const void* W_V, const void* W_packed,
                                            const void* b_K, const void* b_V, const int32_t* block_tables,
                                            void* out, void* workspace, size_t workspace_bytes, void* stream,
                                            void* ev_begin, void* ev_end) {
    return decode_attn(s, plan_host, plan_dev, q, k_pages, v_pages, hidden_pages, W_K, W_V, W_packed, b_K, b_V,
                       block_tables, out, workspace, workspace_bytes, false, stream, ev_begin, ev_end);
}

extern "C" int apt_hybrid_decode_attn(const apt_shape* s, const void* plan_host, void* plan_dev,
                                      const void* q, const void* k_pages, const void* v_pages, const void* hidden_pages,
                                      const void* W_K, const void* W_V, const void* W_packed,
                                      const void* b_K, const void* b_V, const int32_t* block_tables,
                                      void* out, void* workspace, size_t workspace_bytes, void* stream) {
    return decode_attn(s, plan_host, plan_dev, q, k_pages, v_pages, hidden_pages, W_K, W_V, W_packed, b_K, b_V,
                       block_tables, out, workspace, workspace_bytes, false, stream, nullptr, nullptr);
}

extern "C" int apt_hybrid_decode_attn_static(const apt_shape* s, const void* plan_host, void* plan_dev,
                                             const void* q, const void* k_pages, const void* v_pages, const void* hidden_pages,
                                             const void* W_K, const void* W_V, const void* W_packed,
                                             const void* b_K, const void* b_V, const int32_t* block_tables,
                                             void* out, void* stream) {
    return decode_attn(s, plan_host, plan_dev, q, k_pages, v_pages, hidden_pages, W_K, W_V, W_packed, b_K, b_V,
                       block_tables, out, nullptr, 0, true, stream, nullptr, nullptr);
}
