// Hidden-kind items straight from the raw weights (fp16 / bf16, head_dim 64 or 128): no packed copy is needed.
#include <type_traits>
#include "apt_device.h"
#include "apt_launch.h"
#include "apt_merge.h"

namespace {

// One item = one head's K and V of a tile of T tokens: D[2 HD channels][T tokens] with k = d_model on
// v_mfma_f32_16x16x32.  The four waves are (mat, th) as in the packed-weight kernel: mat 0 = K channels, 1 = V
// channels; th = token blocks of 32 (2 b + th), so a wave owns HD channels x T / 2 tokens.
//
// The raw W is [d_in][d_out]: eight consecutive k of one channel, which is what an MFMA operand wants, are d_model
// elements apart.  The k-tile is therefore copied as it lies in memory (32 rows of 2 HD channels, global -> LDS
// without registers) and read with the transposing LDS read ds_read_b64_tr_b16: 16 lanes read 4 k-rows x 16 channels
// and each lane receives the 4 k of one channel.  The 32-byte units of a row sit at u ^ wswz(k), so that the four
// rows of such a read fall on different banks (rows are 256 or 512 bytes apart, the same bank otherwise).
//
// Tiles: at most 256 tokens x 128 channels (HD 64) or 128 x 256 (HD 128), 128 accumulator registers per wave, 24 KB
// per k-tile and three stages, so that two workgroups share a CU and one's barriers and epilogue are covered by the
// other's MFMAs.  Short ranges take the 192-, 128- or 64-token variant: less padding, and in the two smaller ones
// with the LDS this frees more stages in flight.  (Ranges of 129 to 192 tokens in 192 instead of 256 rows, whole step: 25 heads, 25 requests of 64..562 tokens 139.5 ->
// 132 us, 27 heads, 27 of 145..1024 162 -> 153, 32 heads, 24 of 123..1006 beside as many KV-kind ones 248 -> 242.)
//
// 48 requests of 32..1024 tokens at d_model 2048, head_dim 64 (13 k hidden-kind tokens) take 0.225 ms for the whole step (0.224 to 0.229
// over machines), 950 TFLOP/s on 4 d^2 per token; the plain-ALU kernel that served these shapes before took 13.58 ms (16 TFLOP/s).
// No one unit is at its limit there (counters): matrix pipes 0.51 of the cycles, LDS about 0.57 by its bytes (72 KB of reads and copies per
// k-tile and workgroup at 128 a clock), L2 0.63 of a request per clock and channel (four in five ask for half a line: 32 k of a token's row),
// 1790 of 2048 waves resident, which wait for an instruction's turn 45 % of their time and for copies and barriers 25 %.
template <int HD, int T> struct RawTile {
    static constexpr int kChan = 2 * HD;
    static constexpr int kWRow = kChan * 2;                    // bytes of a k-row of the W image
    static constexpr int kWBytes = kBK * kWRow;
    static constexpr int kXBytes = T * kBK * 2;
    static constexpr int kStage = kWBytes + kXBytes;
    static constexpr int kStages = 73728 / kStage < 6 ? 73728 / kStage : 6;
    static constexpr int kWCopies = kWBytes / 4096;            // 1 KB copies per wave and k-tile
    static constexpr int kXCopies = kXBytes / 4096;
    static constexpr int kCopies = kWCopies + kXCopies;
    static constexpr int kScratch = (T + 5 * HD + 8) * 4;
    static constexpr int kLds = kStages * kStage + kScratch;
    static_assert(T % 64 == 0 && kStages >= 3 && kLds <= 80 * 1024, "two workgroups per CU");
};
constexpr int kAhead = 2;                                       // token fragments read ahead of the products
template <int HD> constexpr int raw_max_tile() { return 16384 / HD; }      // 256 or 128 tokens
template <int HD> constexpr int raw_lds_bytes() {
    int m = 0;
    if constexpr (HD == 64) m = RawTile<HD, 256>::kLds > RawTile<HD, 192>::kLds ? RawTile<HD, 256>::kLds : RawTile<HD, 192>::kLds;
    m = m > RawTile<HD, 128>::kLds ? m : RawTile<HD, 128>::kLds;
    return m > RawTile<HD, 64>::kLds ? m : RawTile<HD, 64>::kLds;
}

template <int DT, int HD, int T>
__device__ __forceinline__ void hidden_item_raw(const ItemParams& p, int r, int h, int t0, int t1, char* lds) {
    using C = RawTile<HD, T>;
    constexpr int CF = HD / 16, XF = T / 32;                   // channel and token fragments of a wave
    constexpr int S = C::kStages;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, qd = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), mat = w >> 1, th = w & 1;
    const int d = p.d, nkt = d / kBK, nvalid = t1 - t0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // ---- copy sources of this lane.  W chunk n (1 KB, n = w + 4 i): rows of kWRow bytes; X chunk n: 16 token rows
    const char* wsrc[C::kWCopies];
    const char* xsrc[C::kXCopies];
#pragma unroll
    for (int i = 0; i < C::kWCopies; ++i) {
        const int byte = (w + 4 * i) * 1024 + lane * 16;
        const int k = byte / C::kWRow, u16 = (byte % C::kWRow) >> 4;
        const int ch = ((u16 >> 1) ^ wswz(k)) * 16 + (u16 & 1) * 8;
        wsrc[i] = (ch < HD ? p.W_K + ((int64_t)k * d + h * HD + ch) * 2 : p.W_V + ((int64_t)k * d + h * HD + ch - HD) * 2);
    }
#pragma unroll
    for (int i = 0; i < C::kXCopies; ++i) {
        const int row = 16 * (w + 4 * i) + (lane >> 2);
        const int tok = min(t0 + row, t1 - 1);                 // rows past the range repeat its last token (masked later)
        const int64_t blk = p.block_tables[(int64_t)r * 2 * p.max_blocks + (tok >> p.log2_bs)];
        xsrc[i] = p.hidden_pages + ((blk * p.bs + (tok & (p.bs - 1))) * d) * 2 + (((lane & 3) ^ swz16(row)) << 4);
    }
    const int64_t wstep = (int64_t)kBK * d * 2;
    auto copy = [&](int kt, int i) {                           // copy i of k-tile kt
        const uint32_t st = lds0 + (kt % S) * C::kStage + w * 1024;
        if (i < C::kWCopies) gload_lds16(wsrc[i] + kt * wstep, st + i * 4096);
        else gload_lds16(xsrc[i - C::kWCopies] + kt * (kBK * 2), st + C::kWBytes + (i - C::kWCopies) * 4096);
    };
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        if (s >= nkt) continue;
#pragma unroll
        for (int i = 0; i < C::kCopies; ++i) copy(s, i);
    }

    // ---- per-item constants of the epilogue
    float* scr = (float*)(lds + S * C::kStage);
    float* p_lds = scr;                     // [T] softmax weights (per token half, relative to its maximum)
    float* qs_lds = scr + T;                // [HD] q * scale * log2(e)
    float* bk_lds = qs_lds + HD;            // [HD]
    float* bv_lds = bk_lds + HD;            // [HD]
    float* o_lds = bv_lds + HD;             // [2][HD]
    float* ml_lds = o_lds + 2 * HD;         // [2][2]
    if (tid < HD) {
        qs_lds[tid] = load_elem<DT>(p.q, ((int64_t)r * p.H + h) * HD + tid) * p.scale_log2e;
        bk_lds[tid] = load_elem<DT>(p.b_K, (int64_t)h * HD + tid);
        bv_lds[tid] = load_elem<DT>(p.b_V, (int64_t)h * HD + tid);
    }

    // ---- operand addresses: W fragment c (channels 16 c .. of this wave), X fragment t; further stages are a constant away
    uint32_t waddr[CF];
#pragma unroll
    for (int c = 0; c < CF; ++c) {
        const int k = 8 * qd + (l16 >> 2);
        waddr[c] = lds0 + k * C::kWRow + (((mat * CF + c) ^ wswz(k)) << 5) + (l16 & 3) * 8;
    }
    const uint32_t xaddr = lds0 + C::kWBytes + (th * 32 + l16) * (kBK * 2) + ((qd ^ swz16(l16)) << 4);

    f32x4_t acc[CF][XF];
#pragma unroll
    for (int c = 0; c < CF; ++c)
#pragma unroll
        for (int t = 0; t < XF; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c][t][e] = 0.f;

    // The copies of the k-tile S - 1 ahead go out one by one between the products (asked for in one go, a wave is held until the copy path
    // has taken all of the workgroup's), and a token fragment is read two ahead of its products.  Whole step, copies in one go and all operands
    // read first / so: 39 heads, 8 requests of 16..105 tokens 35.5 / 30.4 us, 22 heads, 19 of 148..762 69.9 / 62.3, 35 heads, 36 of 64..222
    // 124.6 / 113.5, 32 heads, 48 of 32..1024 231.7 / 226.3.  Attention call of 30 drawn batches 0.94 of the time, of 40 more whose
    // hidden-kind items fill the chip about once beside KV-kind ones 0.93 to 0.94 (0.81 to 1.04, four of them above 1: there two runs of
    // one side differ by as much).  Copies in one go, operands read ahead 0.97; in the first quarter of the products 0.95; all operands read
    // first and copies spread 0.93 to 0.96.
    auto k_loop = [&](auto is_v) {
        int stage = 0;
        auto step = [&](int kt, auto refill) {
            __syncthreads();        // k-tile kt has landed for every wave; nobody still reads the stage refilled next
            const uint32_t so = stage * C::kStage;
            uint4 wf[CF], xf[kAhead + 1];
            auto read = [&](int t) { xf[t % (kAhead + 1)] = lds_read16(xaddr + so + (64 * (t >> 1) + 16 * (t & 1)) * (kBK * 2)); };
#pragma unroll
            for (int c = 0; c < CF; ++c) {
                const uint2 lo = lds_read_tr(waddr[c] + so), hi = lds_read_tr(waddr[c] + so + 4 * C::kWRow);
                wf[c] = make_uint4(lo.x, lo.y, hi.x, hi.y);
            }
#pragma unroll
            for (int t = 0; t < kAhead && t < XF; ++t) read(t);
#pragma unroll
            for (int t = 0; t < XF; ++t) {
                if (t + kAhead < XF) read(t + kAhead);
                if constexpr (refill)
#pragma unroll
                    for (int i = t * C::kCopies / XF; i < (t + 1) * C::kCopies / XF; ++i) copy(kt + S - 1, i);
#pragma unroll
                for (int c = 0; c < CF; ++c) {
                    const uint4& x = xf[t % (kAhead + 1)];
                    acc[c][t] = is_v ? mfma16<DT>(x, wf[c], acc[c][t]) : mfma16<DT>(wf[c], x, acc[c][t]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            stage = stage == S - 1 ? 0 : stage + 1;
        };
        int kt = 0;
        for (; kt + S - 1 < nkt; ++kt) {
            wait_vmcnt<(S - 2) * C::kCopies>();
            step(kt, std::true_type{});
        }
        for (; kt < nkt; ++kt) {
            wait_tiles<S - 2, C::kCopies>(nkt - 1 - kt);
            step(kt, std::false_type{});
        }
    };
    if (mat == 0) k_loop(std::false_type{});
    else k_loop(std::true_type{});

    auto tok_row = [&](int t) { return th * 32 + 64 * (t >> 1) + 16 * (t & 1); };
    if (mat == 0) {
        // K wave: rows = channels 16 c + 4 qd + e, columns = tokens of fragment t
        float sp[XF];
#pragma unroll
        for (int t = 0; t < XF; ++t) sp[t] = 0.f;
        float qb = 0.f;
#pragma unroll
        for (int c = 0; c < CF; ++c) {
            const float4 q4 = *(const float4*)(qs_lds + 16 * c + 4 * qd), b4 = *(const float4*)(bk_lds + 16 * c + 4 * qd);
            qb = fmaf(q4.x, b4.x, fmaf(q4.y, b4.y, fmaf(q4.z, b4.z, fmaf(q4.w, b4.w, qb))));
#pragma unroll
            for (int t = 0; t < XF; ++t) {
                sp[t] = fmaf(acc[c][t][0], q4.x, sp[t]);
                sp[t] = fmaf(acc[c][t][1], q4.y, sp[t]);
                sp[t] = fmaf(acc[c][t][2], q4.z, sp[t]);
                sp[t] = fmaf(acc[c][t][3], q4.w, sp[t]);
            }
        }
        float m = kSentinel;
        bool ok[XF];
#pragma unroll
        for (int t = 0; t < XF; ++t) {
            sp[t] += qb;                     // the lane group's share of q . b_K
            sp[t] += __shfl_xor(sp[t], 16);
            sp[t] += __shfl_xor(sp[t], 32);
            ok[t] = tok_row(t) + l16 < nvalid;
            sp[t] = ok[t] ? sp[t] : kSentinel;
            m = fmaxf(m, sp[t]);
        }
        m = group_max<16>(m);                // the four lane groups hold the same scores
        float l = 0.f;
#pragma unroll
        for (int t = 0; t < XF; ++t) {
            const float pw = ok[t] ? fast_exp2(sp[t] - m) : 0.f;
            l += pw;
            if (qd == 0) p_lds[tok_row(t) + l16] = pw;
        }
        l = group_sum<16>(l);
        if (lane == 0) { ml_lds[th * 2] = m; ml_lds[th * 2 + 1] = l; }
    }
    __syncthreads();
    if (mat == 1) {
        // V wave: rows = tokens 4 qd + e of fragment t, columns = channels 16 c + l16
        float o[CF];
#pragma unroll
        for (int c = 0; c < CF; ++c) o[c] = 0.f;
#pragma unroll
        for (int t = 0; t < XF; ++t) {
            const float4 p4 = *(const float4*)(p_lds + tok_row(t) + 4 * qd);
            const int rest = nvalid - tok_row(t) - 4 * qd;     // rows past the range: left out, not multiplied by zero (V may be infinite)
#pragma unroll
            for (int c = 0; c < CF; ++c) {
                o[c] = fmaf(rest > 0 ? acc[c][t][0] : 0.f, p4.x, o[c]);
                o[c] = fmaf(rest > 1 ? acc[c][t][1] : 0.f, p4.y, o[c]);
                o[c] = fmaf(rest > 2 ? acc[c][t][2] : 0.f, p4.z, o[c]);
                o[c] = fmaf(rest > 3 ? acc[c][t][3] : 0.f, p4.w, o[c]);
            }
        }
        const float l = ml_lds[th * 2 + 1];
#pragma unroll
        for (int c = 0; c < CF; ++c) {
            o[c] += __shfl_xor(o[c], 16);
            o[c] += __shfl_xor(o[c], 32);
            if (qd == 0) o_lds[th * HD + 16 * c + l16] = l > 0.f ? fmaf(l, bv_lds[16 * c + l16], o[c]) : o[c];
        }
    }
    __syncthreads();
    if (tid < HD) {
        const float m0 = ml_lds[0], l0 = ml_lds[1], m1 = ml_lds[2], l1 = ml_lds[3];
        const float M = fmaxf(m0, m1);
        const float w0 = fast_exp2(m0 - M), w1 = fast_exp2(m1 - M);
        const int32_t* ws_offset = p.plan + APT_PW_HEADER + p.B;
        const int64_t slot = ((int64_t)ws_offset[r] + t0 / p.hidden_chunk) * p.H + h;
        put_partial(p, slot, tid, HD, o_lds[tid] * w0 + o_lds[HD + tid] * w1);
        if (tid == 0) put_partial_ml(p, slot, M, l0 * w0 + l1 * w1);
    }
}

// One workgroup per item: the hidden-kind items as dealt to the XCDs (apt_dealt_item), then the KV-kind items.
template <int DT, int HD>
__global__ __launch_bounds__(kThreads, 2) void apt_items_raw_kernel(ItemParams p, int share) {
    extern __shared__ __align__(16) char lds[];
    const int g = blockIdx.x;
    const int4* items = (const int4*)(p.plan + p.items_off);
    if (g < 8 * share) {
        const int i = apt_dealt_item(p.plan + APT_PW_QUEUE0, share, g);
        if (i < 0) return;
        const int4 it = items[i];
        const int n = it.w - it.z;
        if (n <= 64) hidden_item_raw<DT, HD, 64>(p, it.x, it.y, it.z, it.w, lds);
        else if (HD == 128 || n <= 128) hidden_item_raw<DT, HD, 128>(p, it.x, it.y, it.z, it.w, lds);
        else if constexpr (HD == 64) {
            if (n <= 192) hidden_item_raw<DT, HD, 192>(p, it.x, it.y, it.z, it.w, lds);
            else hidden_item_raw<DT, HD, 256>(p, it.x, it.y, it.z, it.w, lds);
        }
    } else {
        const int i = p.n_hidden_items + g - 8 * share;
        if (i >= p.n_items) return;
        const int4 it = items[i];
        kv_item_through<DT, HD>(p, it.x, it.y, it.z, it.w, lds);
    }
    merge_by_last<DT, HD, APT_MERGE_RANGES, false>(p, 0, lds);
}

template <int DT, int HD> int launch(const ItemParams& p, hipStream_t st) {
    const int share = (p.n_hidden_items + 7) / 8;
    const unsigned grid = 8u * share + (unsigned)(p.n_items - p.n_hidden_items);
    hipLaunchKernelGGL((apt_items_raw_kernel<DT, HD>), dim3(grid), dim3(kThreads), raw_lds_bytes<HD>(), st, p, share);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

}  // namespace

int apt_launch_raw16(const ItemParams& p, int dtype, int head_dim, hipStream_t st) {
    if (dtype == APT_F16) return head_dim == 64 ? launch<1, 64>(p, st) : launch<1, 128>(p, st);
    return head_dim == 64 ? launch<2, 64>(p, st) : launch<2, 128>(p, st);
}

bool apt_setup_raw16() {
    return apt_raise_lds_limit(apt_items_raw_kernel<1, 64>) && apt_raise_lds_limit(apt_items_raw_kernel<1, 128>) &&
           apt_raise_lds_limit(apt_items_raw_kernel<2, 64>) && apt_raise_lds_limit(apt_items_raw_kernel<2, 128>);
}
