// Device code shared by the translation units of the library: parameters of the attention launch, element and
// cross-lane helpers, MFMA and global->LDS copy wrappers, and the KV-kind item (served by every item kernel).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "apt_internal.h"

struct ItemParams {
    const int32_t* plan;          // device blob
    int32_t* kv_ticket;           // device blob word APT_PW_KV_TICKET: next KV-kind item of the persistent launch, items done of one that merges (merge_by_last)
    char* out;                    // a launch that merges by itself (merge_by_last): the output and its element type, else NULL
    int32_t out_dtype, most_ranges;   // most_ranges: of a request
    const char* q;
    const char* k_pages;
    const char* v_pages;
    const char* hidden_pages;
    const char* W_K;
    const char* W_V;
    const char* W_packed;
    const char* b_K;
    const char* b_V;
    const int32_t* block_tables;
    float* ws_acc;                // [n_slots][HD]
    float2* ws_ml;                // [n_slots]
    int32_t B, H, d, bs, log2_bs, max_blocks;
    int32_t n_items, n_hidden_items, hidden_chunk, kv_chunk, items_off;
    float scale_log2e;
    int32_t wide_tiles;           // packed weights, ranges of 256 tokens: tiles of 320 rows (apt_pack.h)
    int32_t item_base;            // one-workgroup-per-item launch: first item of the grid
    // absorbed-weight hidden path: workspace sections (fp32)
    float* ab_qt;                 // [n_hid_req][H][d], 16-bit inputs: parts in the score kernel's order
    float* ab_cb;                 // [n_hid_req][H]
    float* ab_s;                  // [ab_ks][H][ab_tokens] partial scores over d_model slices; slice 0 ends as the scores
    float2* ab_ml;                // [n_hid_req][H]
    float* ab_yp;                 // [n_hidden_items][H][d], the sum of a unit at its first range
    float* ab_op;                 // [ab_os][n_hid_req][H][HD]
    void* ab_pp;                  // 16-bit inputs: softmax weights as 16-bit parts, [16 n_hidden_items][parts * ab_rows][32]
    int64_t ab_tokens;            // cached tokens of all hidden-kind requests
    int32_t n_hid_req;
    int32_t ab_ks;                // slices of d_model in the score partials
    int32_t ab_tiles, ab_tiles_off;   // 256-token tiles of all hidden-kind requests, their place in the plan
    int32_t ab_units, ab_units_off;   // units of the weighted sums, their place in the plan
    int32_t ab_group;                 // ranges per unit
    int32_t ab_os;                    // slices of d_model in the output partials
    int32_t ab_rows;                  // 16-bit inputs: rows per part of the weights (heads padded to whole fragments)
    int32_t ab_past;                  // 16-bit inputs: what is read past the caches (APT_AB_PAST_*)
};

namespace {

constexpr float kSentinel = -1.0e30f;   // "no score yet": finite, so differences never give NaN
constexpr int kThreads = 256;

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// 16-byte load of data that is read once (streamed past the caches)
__device__ inline uint4 load16_stream(const char* p) {
    const u32x4_t v = __builtin_nontemporal_load((const u32x4_t*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}


// ---------------------------------------------------------------------------------
// element helpers.  DT: 0 = fp32, 1 = fp16, 2 = bf16
// ---------------------------------------------------------------------------------
template <int DT> struct Elt { static constexpr int bytes = DT == 0 ? 4 : 2; static constexpr int per16 = 16 / bytes; };

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

template <int DT> __device__ inline float load_elem(const char* base, int64_t idx) {
    if constexpr (DT == 0) return ((const float*)base)[idx];
    else if constexpr (DT == 1) return (float)((const _Float16*)base)[idx];
    else return bf16_to_f32(((const uint16_t*)base)[idx]);
}

// 16 bytes -> Elt<DT>::per16 floats
template <int DT> __device__ inline void cvt16(const uint4& v, float* out) {
    if constexpr (DT == 0) {
        out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y);
        out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
    } else if constexpr (DT == 1) {
        h8_t h = __builtin_bit_cast(h8_t, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = (float)h[i];
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
}

__device__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------------
// cross-lane helpers
// ---------------------------------------------------------------------------------
template <int CTRL> __device__ inline float dpp_mov(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// Exchange between two registers: the odd 16-lane rows of a with the even rows of b (swap16), the upper half of a with the
// lower half of b (swap32).  With a == b each then holds one of the two values a lane pair is to combine.
__device__ inline void swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
}
__device__ inline void swap32(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
}
// Sums over the four 16-lane rows of four values at once: row i of the result holds the sum of s_i, (row 0 + row 1) + (row 2 +
// row 3).  Three exchanges, where a butterfly for each value takes eight through LDS.
__device__ inline float sum_rows4(float s0, float s1, float s2, float s3) {
    swap16(s0, s1);
    swap16(s2, s3);
    s0 += s1, s2 += s3;
    swap32(s0, s2);
    return s0 + s2;
}
// Sum over the aligned group of LANES lanes a lane belongs to; every lane gets the sum.
template <int LANES> __device__ inline float group_sum(float x) {
    x += dpp_mov<0xB1>(x);                          // quad_perm [1,0,3,2]
    x += dpp_mov<0x4E>(x);                          // quad_perm [2,3,0,1]
    if constexpr (LANES >= 8) x += dpp_mov<0x141>(x);   // row_half_mirror
    if constexpr (LANES >= 16) x += dpp_mov<0x140>(x);  // row_mirror
    if constexpr (LANES >= 32) { float y = x; swap16(x, y); x += y; }
    if constexpr (LANES >= 64) { float y = x; swap32(x, y); x += y; }
    return x;
}
template <int LANES> __device__ inline float group_max(float x) {
    x = fmaxf(x, dpp_mov<0xB1>(x));
    x = fmaxf(x, dpp_mov<0x4E>(x));
    if constexpr (LANES >= 8) x = fmaxf(x, dpp_mov<0x141>(x));
    if constexpr (LANES >= 16) x = fmaxf(x, dpp_mov<0x140>(x));
    if constexpr (LANES >= 32) { float y = x; swap16(x, y); x = fmaxf(x, y); }
    if constexpr (LANES >= 64) { float y = x; swap32(x, y); x = fmaxf(x, y); }
    return x;
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ODT: element type of the output
template <int ODT> __device__ inline void store_out(char* out, int64_t i, float o) {
    if constexpr (ODT == 0) ((float*)out)[i] = o;
    else if constexpr (ODT == 1) ((_Float16*)out)[i] = (_Float16)o;
    else ((uint16_t*)out)[i] = f32_to_bf16_rne(o);
}

// ---------------------------------------------------------------------------------
// KV-kind item
// ---------------------------------------------------------------------------------
// K/V block layout [head][slot][HD]: the rows of one (block, head) are one contiguous run
// of bs*HD elements, read as 1 KB wave loads (64 lanes x 16 B).  LPR lanes share a row,
// 64/LPR rows per load.  A lane group keeps its own online-softmax state for the rows it
// sees; the groups are combined through LDS at the end.
constexpr int kKvUnits = 4;   // 1 KB loads of K (and of V) per pipeline stage

// NW waves share an item.  The lane groups are combined in up to two rounds: with more than four waves, every HD threads
// combine the groups of four waves, or fewer, and the first HD then those sums.
template <int DT, int HD, int NW> struct KvItem {
    static constexpr int kGroups = NW * (64 / (HD * Elt<DT>::bytes / 16));
    static constexpr int kParts = NW > 4 ? NW * 64 / HD : 1;
    static constexpr int kLds = (kGroups + (kParts > 1 ? kParts : 0)) * (2 + HD) * 4;
};

// done(c, M, L, A): thread c < HD has the sums of channel c over the range
template <int DT, int HD, int NW, typename Done>
__device__ __forceinline__ void kv_range(const ItemParams& p, int r, int h, int t0, int t1, char* lds, Done done) {
    constexpr int EB = Elt<DT>::bytes;
    constexpr int EPL = Elt<DT>::per16;          // elements per lane per load
    constexpr int LPR = HD * EB / 16;            // lanes per row
    constexpr int RPL = 64 / LPR;                // rows per 1 KB load
    constexpr int G = NW * RPL;                  // lane groups in the workgroup

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int bs = p.bs;
    const int log2_nl = p.log2_bs - __builtin_ctz(RPL);     // loads per page per matrix = bs/RPL
    const int nl_mask = (1 << log2_nl) - 1;
    const int64_t blk_bytes = (int64_t)bs * p.d * EB;
    const int64_t head_off = (int64_t)h * bs * HD * EB;

    const int p0 = t0 >> p.log2_bs;
    const int p1 = (t1 + bs - 1) >> p.log2_bs;
    // pages of this wave: p0 + w, p0 + w + NW, ...
    const int npg = (p1 - p0 - w + NW - 1) / NW;
    const int nunits = npg > 0 ? (npg << log2_nl) : 0;

    // lane i holds the block ids of the wave's i-th page
    int32_t kid = 0, vid = 0;
    if (lane < npg) {
        const int64_t e = (int64_t)r * 2 * p.max_blocks + p0 + w + NW * lane;
        kid = p.block_tables[e];
        vid = p.block_tables[e + p.max_blocks];
    }

    // q for the lane's channels, pre-scaled
    const int c0 = (lane % LPR) * EPL;
    float qf[EPL];
    cvt16<DT>(*(const uint4*)(p.q + (((int64_t)r * p.H + h) * HD + c0) * EB), qf);
#pragma unroll
    for (int i = 0; i < EPL; ++i) qf[i] *= p.scale_log2e;

    float m = kSentinel, l = 0.f, acc[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) acc[i] = 0.f;

    uint4 kb[2][kKvUnits], vb[2][kKvUnits];
    auto issue = [&](int g, uint4* kbuf, uint4* vbuf) {
#pragma unroll
        for (int i = 0; i < kKvUnits; ++i) {
            const int u = g * kKvUnits + i;
            if (u < nunits) {
                const int pg = u >> log2_nl;
                const int64_t kblk = __builtin_amdgcn_readlane(kid, pg);
                const int64_t vblk = __builtin_amdgcn_readlane(vid, pg);
                const int64_t off = head_off + (int64_t)(u & nl_mask) * 1024 + lane * 16;
                kbuf[i] = load16_stream(p.k_pages + kblk * blk_bytes + off);
                vbuf[i] = load16_stream(p.v_pages + vblk * blk_bytes + off);
            }
        }
    };
    auto consume = [&](int g, const uint4* kbuf, const uint4* vbuf) {
        float s[kKvUnits];
        bool ok[kKvUnits];
        float mn = m;
#pragma unroll
        for (int i = 0; i < kKvUnits; ++i) {
            const int u = g * kKvUnits + i;
            const int pg = u >> log2_nl;
            const int tok = ((p0 + w + NW * pg) << p.log2_bs) + (u & nl_mask) * RPL + lane / LPR;
            ok[i] = (u < nunits) && (tok < t1);
            float kf[EPL];
            cvt16<DT>(kbuf[i], kf);
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) part = fmaf(kf[e], qf[e], part);
            part = group_sum<LPR>(part);
            s[i] = ok[i] ? part : kSentinel;
            mn = fmaxf(mn, s[i]);
        }
        const float alpha = fast_exp2(m - mn);
        l *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
#pragma unroll
        for (int i = 0; i < kKvUnits; ++i) {
            const float pw = ok[i] ? fast_exp2(s[i] - mn) : 0.f;
            l += pw;
            float vf[EPL];
            cvt16<DT>(vbuf[i], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(pw, ok[i] ? vf[e] : 0.f, acc[e]);
        }
        m = mn;
    };

    const int ngroups = (nunits + kKvUnits - 1) / kKvUnits;
    if (ngroups > 0) issue(0, kb[0], vb[0]);
    for (int g = 0; g < ngroups; g += 2) {
        if (g + 1 < ngroups) issue(g + 1, kb[1], vb[1]);
        consume(g, kb[0], vb[0]);
        if (g + 2 < ngroups) issue(g + 2, kb[0], vb[0]);
        if (g + 1 < ngroups) consume(g + 1, kb[1], vb[1]);
    }

    // combine the lane groups: LDS [G] m, [G] l, [G][HD] acc
    float* gm = (float*)lds;
    float* gl = gm + G;
    float* ga = gl + G;
    const int grp = w * RPL + lane / LPR;
    if (lane % LPR == 0) { gm[grp] = m; gl[grp] = l; }
#pragma unroll
    for (int e = 0; e < EPL; ++e) ga[grp * HD + c0 + e] = acc[e];
    __syncthreads();
    constexpr int P = KvItem<DT, HD, NW>::kParts;
    auto combine = [&](const float* sm, const float* sl, const float* sa, int n, int c, float& M, float& L, float& A) {
        M = kSentinel;
        for (int g = 0; g < n; ++g) M = fmaxf(M, sm[g]);
        L = A = 0.f;
        for (int g = 0; g < n; ++g) {
            const float wgt = fast_exp2(sm[g] - M);
            L = fmaf(sl[g], wgt, L);
            A = fmaf(sa[g * HD + c], wgt, A);
        }
    };
    float M, L, A;
    if constexpr (P > 1) {
        static_assert(G % P == 0, "groups of a part");
        float* pm = ga + G * HD;
        float* pl = pm + P;
        float* pa = pl + P;
        const int part = tid / HD, g = part * (G / P), c = tid % HD;
        combine(gm + g, gl + g, ga + g * HD, G / P, c, M, L, A);
        if (c == 0) { pm[part] = M; pl[part] = L; }
        pa[tid] = A;
        __syncthreads();
        gm = pm, gl = pl, ga = pa;
    }
    if (tid < HD) {
        combine(gm, gl, ga, P > 1 ? P : G, tid, M, L, A);
        done(tid, M, L, A);
    }
}

// A range of the plan: its partial goes to the workspace
template <int DT, int HD, int NW = 4>
__device__ __forceinline__ void kv_item(const ItemParams& p, int r, int h, int t0, int t1, char* lds) {
    kv_range<DT, HD, NW>(p, r, h, t0, t1, lds, [&](int c, float M, float L, float A) {
        const int32_t* ws_offset = p.plan + APT_PW_HEADER + APT_PA_WS_OFFSET * p.B;
        const int64_t slot = ((int64_t)ws_offset[r] + t0 / p.kv_chunk) * p.H + h;
        p.ws_acc[slot * HD + c] = A;
        if (c == 0) p.ws_ml[slot] = make_float2(M, L);
    });
}

// ---------------------------------------------------------------------------------
// matrix cores and global -> LDS copies
// ---------------------------------------------------------------------------------
constexpr int kBK = 32;                                // k extent of one LDS tile of the matrix kernels

// Position swizzle of the 16-byte units of 64-byte LDS rows, measured free of bank conflicts (SQ_LDS_BANK_CONFLICT = 0,
// 4 cycles per ds_read_b128) for the operand reads of 16x16x32 MFMAs (16 consecutive rows, all four units).
__host__ __device__ inline int swz16(int row) { return (row >> 1) & 3; }

template <int DT> __device__ inline f32x16_t mfma32(const uint4& a, const uint4& b, f32x16_t c) {
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8_t, a), __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b), c, 0, 0, 0);
}
// A: lane l holds row l % 16, k = 8 (l / 16) .. +7; B: column l % 16, the same k; D: column l % 16, rows 4 (l / 16) + e
template <int DT> __device__ inline f32x4_t mfma16(const uint4& a, const uint4& b, f32x4_t c) {
    if constexpr (DT == 1)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, a), __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b), c, 0, 0, 0);
}

// 16-byte global -> LDS copy without a register stage: lane i's 16 bytes land at
// lds_addr + 16 i.  The LDS address goes through M0 and must be wave-uniform.
__device__ inline void gload_lds16(const void* g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(g) : "memory", "m0");
}
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
// 16-byte LDS read at an absolute LDS address (the dynamic LDS base is folded into the operand addresses once)
__device__ inline uint4 lds_read16(uint32_t addr) {
    const u32x4_t v = *(const lds_u32x4_t*)(uintptr_t)addr;
    return make_uint4(v.x, v.y, v.z, v.w);
}
// Transposing LDS read of an MFMA operand whose k runs over LDS rows: 16 consecutive lanes cover 4 rows x 32 bytes, lane i
// reads 8 bytes at its address and receives the 4 k of column i.  Unit u (32 bytes) of row k sits at u ^ wswz(k) where the
// rows are a multiple of 256 bytes apart, so that the rows of a read fall on different banks.
__device__ inline int wswz(int k) { return (k & 3) | ((k >> 1) & 4); }

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
__device__ inline uint2 lds_read_tr(uint32_t addr) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(uintptr_t)addr));
}
template <int N> __device__ inline void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// waits until the copies of no more than `tiles` k-tiles are in flight, COPIES each; MOST: of no more than these
template <int MOST, int COPIES> __device__ __forceinline__ void wait_tiles(int tiles) {
    if constexpr (MOST > 0) {
        if (tiles < MOST) return wait_tiles<MOST - 1, COPIES>(tiles);
    }
    wait_vmcnt<MOST * COPIES>();
}

}  // namespace
