// Hidden-kind items of fp32 inputs, from the raw weights.
#include <type_traits>
#include "apt_device.h"
#include "apt_launch.h"
#include "apt_merge.h"

namespace {

// One item = one head's K and V of up to 64 tokens (NT fragments of 16), k = d_model, on v_mfma_f32_16x16x4_f32: the
// same fp32 products and sums as the plain ALUs at twice their rate (256 flops per clock and CU; packed fp32 is not
// used).  fp32 layers are small and their batches few, so latency decides: operands go straight from memory into
// registers, PD blocks of 16 k ahead, with no LDS tile and no barrier in the k loop.
//
// A wave owns 64 channels of K (mat 0) or V (mat 1).  head_dim 64: two waves per matrix split k in halves; head_dim 128:
// they split the channels.  Scores and outputs are linear in both, so the halves meet as partial scores and partial
// outputs in LDS.  Both operands are read as 16 bytes per lane: a lane's float4 of X holds k = 16 m + 4 (lane / 16)
// + j of token lane % 16, its float4 of W holds channels 4 (lane % 16) + c of row k, so MFMA (j, c) multiplies k-column j
// with channels 4 * row + c; a fragment's rows are every fourth channel.
//
// The fp32 tiny layer (d_model 256, 4 heads of 64, 4 requests of 16..128 tokens): kernel 75.5 us with the plain-ALU
// version (one dependent fma chain over k per channel, loads not ahead of it), 8.2 us now, most of it the start-up chain
// item -> block id -> row.  At d_model 1024, 64 requests: 488 us, 63 % of what a 4096^3 fp32 product reaches.
template <int NT> constexpr int prefetch_blocks() { return NT == 1 ? 6 : NT == 2 ? 4 : 3; }

template <int HD, int NT>
__device__ __forceinline__ void hidden_item_f32(const ItemParams& p, int r, int h, int t0, int t1, float* lds) {
    constexpr int PD = prefetch_blocks<NT>(), T = 16 * NT;
    float* sp_lds = lds;                    // [2][64] partial scores of the two K waves
    float* p_lds = lds + 128;               // [2][64] softmax weights, a copy per V wave
    float* o_lds = lds + 256;               // [2][64] outputs of the two V waves
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, qd = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), mat = w >> 1, sub = w & 1;
    const int d = p.d, nvalid = t1 - t0;
    const int k_begin = HD == 64 ? sub * (d / 2) : 0, nb = (HD == 64 ? d / 2 : d) / 16;
    const int ch0 = h * HD + (HD == 64 ? 0 : sub * 64);        // first channel of this wave

    const float* wsrc = (const float*)(mat == 0 ? p.W_K : p.W_V) + (int64_t)(k_begin + 4 * qd) * d + ch0 + 4 * l16;
    const float* xsrc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tok = min(t0 + 16 * t + l16, t1 - 1);        // rows past the range repeat its last token (masked later)
        const int64_t blk = p.block_tables[(int64_t)r * 2 * p.max_blocks + (tok >> p.log2_bs)];
        xsrc[t] = (const float*)p.hidden_pages + (blk * p.bs + (tok & (p.bs - 1))) * d + k_begin + 4 * qd;
    }
    f32x4_t wv[PD][4], xv[PD][NT];
    auto load = [&](int b, f32x4_t* wb, f32x4_t* xb) {
        b = min(b, nb - 1);                                    // past the end: repeated, not used
#pragma unroll
        for (int j = 0; j < 4; ++j) wb[j] = *(const f32x4_t*)(wsrc + (int64_t)(16 * b + j) * d);
#pragma unroll
        for (int t = 0; t < NT; ++t) xb[t] = *(const f32x4_t*)(xsrc[t] + 16 * b);
    };
    f32x4_t acc[4][NT];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c][t][e] = 0.f;
    auto k_loop = [&](auto is_v) {
#pragma unroll
        for (int s = 0; s < PD; ++s) load(s, wv[s], xv[s]);
        for (int b0 = 0; b0 < nb; b0 += PD) {
#pragma unroll
            for (int s = 0; s < PD; ++s) {
                if (b0 + s < nb) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                acc[c][t] = is_v ? __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s][t][j], wv[s][j][c], acc[c][t], 0, 0, 0)
                                                 : __builtin_amdgcn_mfma_f32_16x16x4f32(wv[s][j][c], xv[s][t][j], acc[c][t], 0, 0, 0);
                }
                load(b0 + s + PD, wv[s], xv[s]);
            }
        }
    };
    const float* bk = (const float*)p.b_K + h * HD;
    const float* q = (const float*)p.q + ((int64_t)r * p.H + h) * HD;
    if (mat == 0) {
        // rows of fragment c: channels ch0 + 4 * row + c; this lane's rows 4 qd + e: channels 16 qd + 4 e + c
        const int c_lane = (HD == 64 ? 0 : sub * 64) + 16 * qd;
        f32x4_t q4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) q4[e] = *(const f32x4_t*)(q + c_lane + 4 * e) * p.scale_log2e;
        float qb = 0.f;                                        // q . b_K of this wave's channels, once
        if (HD == 128 || sub == 0)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < 4; ++c) qb = fmaf(q4[e][c], bk[c_lane + 4 * e + c], qb);
        k_loop(std::false_type{});
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            float s = qb;
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) s = fmaf(acc[c][t][e], q4[e][c], s);
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (qd == 0) sp_lds[sub * 64 + 16 * t + l16] = s;
        }
    } else {
        k_loop(std::true_type{});
    }
    __syncthreads();
    // every V wave (and wave 0, for the statistics) forms the softmax weights of the range, one token per lane
    const bool ok = lane < nvalid;
    const float s = ok ? sp_lds[lane & (T - 1)] + sp_lds[64 + (lane & (T - 1))] : kSentinel;
    const float m = group_max<64>(s);
    const float pw = ok ? fast_exp2(s - m) : 0.f;
    const float l = group_sum<64>(pw);
    const int32_t* ws_offset = p.plan + APT_PW_HEADER + p.B;
    const int64_t slot = ((int64_t)ws_offset[r] + t0 / p.hidden_chunk) * p.H + h;
    if (tid == 0) put_partial_ml(p, slot, m, l);
    if (mat == 1) {
        p_lds[sub * 64 + lane] = pw;                           // read back by this wave only
        f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 p4 = *(const float4*)(p_lds + sub * 64 + 16 * t + 4 * qd);
            const int rest = nvalid - 16 * t - 4 * qd;         // rows past the range: left out, not multiplied by zero (V may be infinite)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                o[c] = fmaf(rest > 0 ? acc[c][t][0] : 0.f, p4.x, o[c]);
                o[c] = fmaf(rest > 1 ? acc[c][t][1] : 0.f, p4.y, o[c]);
                o[c] = fmaf(rest > 2 ? acc[c][t][2] : 0.f, p4.z, o[c]);
                o[c] = fmaf(rest > 3 ? acc[c][t][3] : 0.f, p4.w, o[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            o[c] += __shfl_xor(o[c], 16);
            o[c] += __shfl_xor(o[c], 32);
        }
        if (qd == 0) *(f32x4_t*)(o_lds + sub * 64 + 4 * l16) = o;
    }
    __syncthreads();
    if (tid < HD) {
        const float bv = ((const float*)p.b_V)[h * HD + tid];
        put_partial(p, slot, tid, HD, fmaf(l, bv, HD == 64 ? o_lds[tid] + o_lds[64 + tid] : o_lds[tid]));
    }
}

// grid as for the 16-bit kernel
template <int HD>
__global__ __launch_bounds__(kThreads) void apt_items_f32_kernel(ItemParams p, int share) {
    extern __shared__ __align__(16) char lds[];
    const int g = blockIdx.x;
    const int4* items = (const int4*)(p.plan + p.items_off);
    if (g < 8 * share) {
        const int i = apt_dealt_item(p.plan + APT_PW_QUEUE0, share, g);
        if (i < 0) return;
        const int4 it = items[i];
        const int n = it.w - it.z;
        if (n <= 16) hidden_item_f32<HD, 1>(p, it.x, it.y, it.z, it.w, (float*)lds);
        else if (n <= 32) hidden_item_f32<HD, 2>(p, it.x, it.y, it.z, it.w, (float*)lds);
        else hidden_item_f32<HD, 4>(p, it.x, it.y, it.z, it.w, (float*)lds);
    } else {
        const int i = p.n_hidden_items + g - 8 * share;
        if (i >= p.n_items) return;
        const int4 it = items[i];
        kv_item_through<0, HD>(p, it.x, it.y, it.z, it.w, lds);
    }
    merge_by_last<0, HD, APT_MERGE_RANGES, false>(p, 0, lds);
}

template <int HD> int launch(const ItemParams& p, hipStream_t st) {
    const int share = (p.n_hidden_items + 7) / 8;
    constexpr int G = 4 * (64 / (HD / 4));                     // lane groups of a KV-kind item
    constexpr size_t kv_lds = (size_t)(2 * G + G * HD) * 4;
    static_assert(kv_lds >= 384 * 4, "LDS of a hidden-kind item");
    const unsigned grid = 8u * share + (unsigned)(p.n_items - p.n_hidden_items);
    hipLaunchKernelGGL(apt_items_f32_kernel<HD>, dim3(grid), dim3(kThreads), kv_lds, st, p, share);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

}  // namespace

int apt_launch_raw32(const ItemParams& p, int head_dim, hipStream_t st) {
    return head_dim == 64 ? launch<64>(p, st) : launch<128>(p, st);
}
