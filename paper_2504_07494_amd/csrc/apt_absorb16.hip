// Absorbed-weight hidden path, 16-bit inputs: the kernels that build the absorbed queries and the scores.
#include <algorithm>
#include <type_traits>
#include "apt_device.h"
#include "apt_launch.h"
#include "apt_absorb_tile.h"

namespace {

// ---- absorbed queries: QT[hr][h][k] = scale * log2(e) * W_K[k, h] . q, as 16-bit parts in the order the score kernel
// copies: [hr][k-tile][part * R + head][unit c at c ^ swizzle(head)], rows of KT values.
// One wave per (head, 32 rows of W_K), the requests of its z-slice in turn; both operands are 16-bit, so the products are exact.
// D rows are k, columns are requests; the rows of the two W fragments are dealt so that a lane ends with 8 consecutive k of
// one request: one 16-byte store per part, 64 contiguous bytes per request.  Eight neighbouring heads of the same rows run
// together on one XCD (workgroup g runs on XCD g % 8), as their stores lie in the same lines.  The queries of all the
// requests are put into LDS first: loads between the stores would wait for them, the two share a counter.
// Bound by the write of QT, R * parts * 2 bytes per k and request (a fill of its size takes 62 us), and by each workgroup's
// start, W_K and the queries behind their indexes.  72 heads, bf16, 96 requests at d_model 9216 (382 MB, 441 counted at
// memory): 195 us with queries from memory, 187 in this order, 155 through LDS, 131 with 128 requests to a workgroup.
//
// 128 requests where that leaves two workgroups per CU (short contexts, 64 / 128, the whole call: 24 heads, 128 requests 113.1 /
// 110.4 us, 32 heads, 100 requests 142.5 / 135.5; 16 heads, 100 requests 64.4 / 66.1, not taken).
__host__ __device__ inline int ab_q_reqs(const ItemParams& p) { return (p.d / 32 + 3) / 4 * p.H >= 512 ? 128 : 64; }
__host__ __device__ inline int ab_q_z_blocks(const ItemParams& p) { return (p.n_hid_req + ab_q_reqs(p) - 1) / ab_q_reqs(p); }
inline int ab_q_groups(const ItemParams& p) { return (p.d / 32 + 3) / 4 * ((p.H + 7) / 8) * ab_q_z_blocks(p); }

template <int HD> __device__ inline int ab_q_swz(int row) { return HD == 128 ? row & 15 : (row >> 1) & 7; }

template <int DT, int HD, int NF>
__device__ __forceinline__ void absorb_q16(const ItemParams& p, int block, char* lds) {
    using C = AbTile<DT, NF>;
    constexpr int NS = C::NS, KS = HD / 32, UPR = HD / 8;
    const int lane = threadIdx.x & 63, l16 = lane & 15, qd = lane >> 4;
    const int slot = block >> 3, group = (slot >> 3) * 8 + (block & 7);
    const int head_groups = (p.H + 7) / 8, z_blocks = ab_q_z_blocks(p);
    const int h = group % head_groups * 8 + (slot & 7), z = group / head_groups % z_blocks;
    const int kb = group / head_groups / z_blocks * 4 + (threadIdx.x >> 6);   // 32-row block of W_K
    if (h >= p.H) return;
    uint4 wf[2][KS];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        const int k = min(kb * 32 + 8 * (l16 >> 2) + 4 * f + (l16 & 3), p.d - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) wf[f][s] = *(const uint4*)(p.W_K + ((int64_t)k * p.d + h * HD + 32 * s + 8 * qd) * 2);
    }
    // the queries of this head: 16-byte unit u of a row at u ^ ab_q_swz(row), free of bank conflicts; rows past the last request repeat it
    const int hr_begin = z * ab_q_reqs(p), n = min(p.n_hid_req - hr_begin, ab_q_reqs(p));
    const int32_t* hid_req = plan_array(p, APT_PA_HID_REQ);
    for (int i = threadIdx.x; i < (n + 15) / 16 * 16 * UPR; i += kThreads) {
        const int row = i / UPR, u = i % UPR, r = hid_req[hr_begin + min(row, n - 1)];
        *(uint4*)(lds + (row * UPR + (u ^ ab_q_swz<HD>(row))) * 16) = *(const uint4*)(p.q + (((int64_t)r * p.H + h) * HD + u * 8) * 2);
    }
    __syncthreads();
    if (kb * 32 >= p.d) return;
    const int k8 = kb * 4 + qd;                          // this lane's unit of 8 k
    const int kt = k8 / (C::KT / 8), c = (k8 % (C::KT / 8)) ^ ab_swz<C::KT>(h);
    for (int row0 = 0; row0 < n; row0 += 16) {
        const int row = row0 + l16, hr = hr_begin + row;
        uint4 qf[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = *(const uint4*)(lds + (row * UPR + ((4 * s + qd) ^ ab_q_swz<HD>(row))) * 16);
        f32x4_t acc[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[f][e] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) acc[f] = mfma16<DT>(wf[f][s], qf[s], acc[f]);
        }
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = acc[e >> 2][e & 3] * p.scale_log2e;
        uint4 part[NS];
        AbSplit<DT>::split8(v, part);
        if (row < n) {
            char* base = (char*)p.ab_qt + ((int64_t)hr * (p.d / C::KT) + kt) * C::kABytes + c * 16;
#pragma unroll
            for (int sp = 0; sp < NS; ++sp) *(uint4*)(base + (sp * C::R + h) * C::kRow) = part[sp];
        }
        if (kb == 0) {                                   // CB = scale * log2(e) * q . b_K
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                float qv[8], bv[8];
                cvt16<DT>(qf[i], qv);
                cvt16<DT>(*(const uint4*)(p.b_K + (h * HD + 32 * i + 8 * qd) * 2), bv);
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(qv[e], bv[e], s);
            }
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (qd == 0 && row < n) p.ab_cb[(int64_t)hr * p.H + h] = s * p.scale_log2e;
        }
    }
}

// The KV-kind items of the batch and the absorbed queries in one launch: neither needs the other, the items (longest first) keep
// memory busy, and the queries fill the CUs that the last items leave.  The step, items in a launch of their own at its end / here:
// 40 heads, 32 + 32 requests of 128..2048 tokens 371 / 363 us; 57
// heads, 7 requests of 158..617 tokens 110 / 101 us (1.4 us of either from the two last kernels in one).
template <int DT, int HD, int NF>
__global__ __launch_bounds__(kThreads) void apt_absorb_q16_kernel(ItemParams p) {
    extern __shared__ __align__(16) char lds[];
    const int n_kv = p.n_items - p.n_hidden_items;
    if ((int)blockIdx.x < n_kv) {
        const int4 it = ((const int4*)(p.plan + p.items_off))[p.n_hidden_items + blockIdx.x];
        kv_item<DT, HD>(p, it.x, it.y, it.z, it.w, lds);
    } else {
        absorb_q16<DT, HD, NF>(p, blockIdx.x - n_kv, lds);
    }
}

// ---- score partials: SP[slice][h][token] = <x_token, QT> over one slice of d_model
// Workgroup = 256 tokens x one slice x all heads, eight waves: wave w takes tokens 64 (w % 4) .. + 63 and the first
// (w < 4) or the second half of the head fragments, so that each SIMD has two waves, one of either half, and one's LDS
// reads are covered by the other's MFMAs.  D rows are heads, columns tokens; the parts of a head are summed in one
// accumulator.  k-tiles of X rows and of QT go global -> LDS without registers, as many stages as LDS holds (one
// workgroup per CU).
//
// X is read past the caches or not by apt_absorbed_past.  A k-tile's copies go out between its products (72 heads, bf16, 96 requests: the
// kernel 620 -> 580 us, 549 without the products).
// Bound by how memory serves the X rows, one 128-byte line per row and 64 k (rows lie 2 d_model apart): 64-wide k-tiles
// in three stages take 87 us for 40 heads, fp16, 33.6 k tokens at d_model 5120 (344 MB of X; 0.40 GB of 128-byte line reads, 4.5
// TB/s), 32-wide ones in seven stages, with more bytes in flight, 99 us.  Where both do not fit 64 wide, X is 64 wide in three
// stages beside four 32-wide ones of the queries (kWideX; two k-tiles share an X tile and its copies): 2.70 GB of memory reads
// instead of 2.80 for 72 heads, bf16, 102 k tokens at d_model 9216 (X is 1.885 GB; the rest are the queries, 0.4 GB, read by each
// of the groups that a request's tiles fall into).  Whole call there 1405 / 1373 us (32 / 64 wide), 49 heads, 64 requests of
// 64..1024 tokens 386 / 374, 65 heads, 16 requests of 20..500 150 / 147.  A start of the k loop that differs between the groups,
// so that they read other memory channels, changed nothing.  The version
// with heads padded to 64, an accumulator per part and 512-wide slices took 117 us for the 40 heads, and 1193 us for the 72.
template <int DT, int NF, int F0, int FN, typename Copy, typename Issue>
__device__ __forceinline__ void score_loop(f32x4_t (*acc)[4], f32x4_t (*sum)[4], f32x4_t (*total)[4], uint32_t lds0, int tg, int nkt, Copy copy, Issue issue) {
    using C = AbTile<DT, NF>;
    constexpr int NS = C::NS, KT = C::KT, S = C::S, XPT = C::XPT;
    constexpr int G = KT / 32 * FN * NS;                 // operand fragments of a k-tile, each for four products
    constexpr int kAhead = G > 2 ? 2 : 1;                // read ahead of the products
    const int lane = threadIdx.x & 63, l16 = lane & 15, qd = lane >> 4;
    int stage = 0, xstage = 0;
    // refill: the copies that iteration kt asks for go out one by one between the products (asked for in one go, a wave is held until
    // the copy path has taken all of the workgroup's); else they have been asked for, or there are none.  odd: kt is
    auto step = [&](int kt, auto odd, auto refill) {
        const uint32_t xst = lds0 + xstage * C::kXBytes, ast = lds0 + C::SX * C::kXBytes + stage * C::kABytes;
        uint4 x[KT / 32][4], a[kAhead + 1];
        auto read = [&](int g) {
            const int ks = g / (FN * NS), f = g / NS % FN, s = g % NS;
            const uint32_t off = (((4 * ks + qd) ^ ab_swz<KT>(l16)) << 4) + l16 * C::kRow;
            a[g % (kAhead + 1)] = lds_read16(ast + (s * C::R + 16 * (F0 + f)) * C::kRow + off);
        };
#pragma unroll
        for (int ks = 0; ks < KT / 32; ++ks) {
            const uint32_t xoff = (((4 * ks + qd + (XPT == 2 && odd ? 4 : 0)) ^ ab_swz<KT * XPT>(l16)) << 4) + l16 * C::kXRow;
#pragma unroll
            for (int t = 0; t < 4; ++t) x[ks][t] = lds_read16(xst + (64 * tg + 16 * t) * C::kXRow + xoff);
        }
#pragma unroll
        for (int g = 0; g < kAhead; ++g) read(g);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g + kAhead < G) read(g + kAhead);
            if constexpr (refill)
#pragma unroll
                for (int i = g * C::kCopies / G; i < (g + 1) * C::kCopies / G; ++i) copy(kt, i, odd);
            const int ks = g / (FN * NS), f = g / NS % FN;
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[f][t] = mfma16<DT>(a[g % (kAhead + 1)], x[ks][t], acc[f][t]);
        }
        stage = stage == S - 1 ? 0 : stage + 1;
        if (XPT == 1 || odd) xstage = xstage == C::SX - 1 ? 0 : xstage + 1;
        if ((kt + 1) % (kAbFold / KT) == 0) ab_fold<4>(acc, sum, FN);
        if ((kt + 1) % (kAbFoldSums / KT) == 0) ab_fold<4>(sum, total, FN);
    };
    // k-tile kt has landed for every wave behind the barrier, and nobody still reads the stages refilled next
    int kt = 0;
    auto full = [&](auto odd) {
        wait_vmcnt<(S - 2) * C::kCopies>();
        __syncthreads();
        step(kt++, odd, std::true_type{});
    };
    // iterations with all their copies
    for (const int end = nkt - XPT * (C::SX - 1); kt < end;) {
        full(std::false_type{});
        if constexpr (XPT == 2) full(std::true_type{});
    }
    auto last = [&](auto odd) {
        // the copies of this k-tile were issued S - 1 of them ago; the last X tile's go out a k-tile before the last queries'
        if (kt + S - 3 + XPT < nkt) wait_vmcnt<(S - 2) * C::kCopies>();
        else wait_vmcnt<0>();
        __syncthreads();
        issue(kt);
        step(kt++, odd, std::false_type{});
    };
    while (kt < nkt) {
        last(std::false_type{});
        if constexpr (XPT == 2) last(std::true_type{});
    }
    ab_fold<4>(acc, sum, FN);
    ab_fold<4>(sum, total, FN);
}

// PAST: X is read past the caches
template <int DT, int NF, bool PAST>
__global__ __launch_bounds__(kAbWaves * 64) void apt_absorb_score16_kernel(ItemParams p) {
    using C = AbTile<DT, NF>;
    constexpr int KT = C::KT, S = C::S, SX = C::SX, XPT = C::XPT, NF0 = C::NF0;
    constexpr int RPC = 1024 / C::kXRow;                 // rows per 1 KB copy
    constexpr int UPR = C::kXRow / 16;                   // 16-byte units per row
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x & 63, l16 = lane & 15, qd = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tg = w & 3, second = w >> 2;
    // A group = eight neighbouring tiles, one slice: they share that slice of their requests' absorbed queries, so a
    // group stays on one XCD (workgroup g runs on XCD g % 8); groups are dealt to the XCDs in turn
    const int slot = blockIdx.x >> 3, group = (slot >> 3) * 8 + (blockIdx.x & 7);
    const int ti = (group / p.ab_ks) * 8 + (slot & 7), slice = group % p.ab_ks;
    if (ti >= p.ab_tiles) return;
    const int tile = p.plan[p.ab_tiles_off + ti], range = tile >> 1;
    const int4 it = ((const int4*)(p.plan + p.items_off))[range];
    const int r = it.x, t1 = it.w, tb = it.z + kAbMT * (tile & 1);
    const int hr = plan_array(p, APT_PA_HID_INDEX)[r];
    const int64_t tok0 = (int64_t)plan_array(p, APT_PA_HID_TOK_OFF)[r] + tb;
    const int n_xt = p.d / (KT * XPT), xt0 = slice * n_xt / p.ab_ks, nxt = (slice + 1) * n_xt / p.ab_ks - xt0;
    const int n_kt = n_xt * XPT, kt0 = xt0 * XPT, nkt = nxt * XPT, k_begin = kt0 * KT;

    const char* xsrc[C::kXCopies];
#pragma unroll
    for (int i = 0; i < C::kXCopies; ++i) {
        const int row = RPC * (C::kXCopies * w + i) + lane / UPR;   // rows past the range repeat its last token (scores not stored)
        xsrc[i] = hidden_row(p, r, min(tb + row, t1 - 1), 2) + (int64_t)k_begin * 2 + (((lane % UPR) ^ ab_swz<KT * XPT>(row)) << 4);
    }
    const char* asrc = (const char*)p.ab_qt + ((int64_t)hr * n_kt + kt0) * C::kABytes + lane * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    auto copy_x = [&](int xt, int i) {
        const char* src = xsrc[i] + xt * C::kXRow;
        const uint32_t dst = lds0 + (xt % SX) * C::kXBytes + (C::kXCopies * w + i) * 1024;
        if constexpr (PAST) gload_lds16_stream(src, dst);
        else gload_lds16(src, dst);
    };
    auto copy_a = [&](int at, int i) {                   // some waves copy the last chunk again (same bytes)
        const int n = min(w + kAbWaves * i, C::kABytes / 1024 - 1);
        gload_lds16(asrc + (int64_t)at * C::kABytes + n * 1024, lds0 + SX * C::kXBytes + (at % S) * C::kABytes + n * 1024);
    };
    // k-tile kt: the queries S - 1 k-tiles ahead, and the X tile SX - 1 ahead (two k-tiles share a wide one's copies)
    auto issue = [&](int kt) {
        const int xt = (kt + XPT * SX) / XPT - 1, at = kt + S - 1;
        if (xt >= 0 && xt < nxt) {
            if (XPT == 1 || (kt & 1) == 0)
#pragma unroll
                for (int i = 0; i < C::kXCopies / XPT; ++i) copy_x(xt, i);
            else
#pragma unroll
                for (int i = C::kXCopies / XPT; i < C::kXCopies; ++i) copy_x(xt, i);
        }
        if (at >= 0 && at < nkt)
#pragma unroll
            for (int i = 0; i < C::kACopies; ++i) copy_a(at, i);
    };
    // copy i of those of iteration kt, which has them all
    auto copy = [&](int kt, int i, auto odd) {
        constexpr int kX = C::kXCopies / XPT;
        if (i < kX) copy_x(kt / XPT + SX - 1, i + (XPT == 2 && odd ? kX : 0));
        else copy_a(kt + S - 1, i - kX);
    };
    f32x4_t acc[NF0][4], sum[NF0][4], total[NF0][4];
#pragma unroll
    for (int f = 0; f < NF0; ++f)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[f][t][e] = sum[f][t][e] = total[f][t][e] = 0.f;
#pragma unroll
    for (int kt = -XPT * (SX - 1); kt < 0; ++kt) issue(kt);
    if (!second) score_loop<DT, NF, 0, NF0>(acc, sum, total, lds0, tg, nkt, copy, issue);
    else score_loop<DT, NF, NF0, NF - NF0>(acc, sum, total, lds0, tg, nkt, copy, issue);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int token = 64 * tg + 16 * t + l16;
        if (tb + token >= t1) continue;
#pragma unroll
        for (int f = 0; f < NF0; ++f)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int h = 16 * (second * NF0 + f) + 4 * qd + e;
                if ((f < NF - NF0 || !second) && h < p.H)
                    p.ab_s[((int64_t)slice * p.H + h) * p.ab_tokens + tok0 + token] = total[f][t][e];
            }
    }
}

template <int DT, int NF> int launch_scores(const ItemParams& p, int head_dim, hipStream_t st) {
    using C = AbTile<DT, NF>;
    const unsigned first = (unsigned)(p.n_items - p.n_hidden_items) +
                           (unsigned)((ab_q_groups(p) + 7) / 8 * 64);
    const int q_lds = (std::min(p.n_hid_req, ab_q_reqs(p)) + 15) / 16 * 16 * head_dim * 2;
    if (head_dim == 128) hipLaunchKernelGGL((apt_absorb_q16_kernel<DT, 128, NF>), dim3(first), dim3(kThreads), std::max(q_lds, KvItem<DT, 128, 4>::kLds), st, p);
    else hipLaunchKernelGGL((apt_absorb_q16_kernel<DT, 64, NF>), dim3(first), dim3(kThreads), std::max(q_lds, KvItem<DT, 64, 4>::kLds), st, p);
    const unsigned groups = (unsigned)((p.ab_tiles + 7) / 8 * p.ab_ks);
    const dim3 grid((groups + 7) / 8 * 64), block(kAbWaves * 64);
    if (p.ab_past & APT_AB_PAST_SCORES) hipLaunchKernelGGL((apt_absorb_score16_kernel<DT, NF, true>), grid, block, C::kLds, st, p);
    else hipLaunchKernelGGL((apt_absorb_score16_kernel<DT, NF, false>), grid, block, C::kLds, st, p);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}

template <int DT> int launch_scores_nf(const ItemParams& p, int head_dim, hipStream_t st) {
    switch (ab_head_frags(p.H)) {
    case 2: return launch_scores<DT, 2>(p, head_dim, st);
    case 3: return launch_scores<DT, 3>(p, head_dim, st);
    case 4: return launch_scores<DT, 4>(p, head_dim, st);
    case 5: return launch_scores<DT, 5>(p, head_dim, st);
    case 6: return launch_scores<DT, 6>(p, head_dim, st);
    default: return launch_scores<DT, 8>(p, head_dim, st);
    }
}

template <int DT, int NF> bool setup_nf() {
    return apt_raise_lds_limit(apt_absorb_score16_kernel<DT, NF, false>) && apt_raise_lds_limit(apt_absorb_score16_kernel<DT, NF, true>);
}
template <int DT> bool setup() {
    return setup_nf<DT, 2>() && setup_nf<DT, 3>() && setup_nf<DT, 4>() && setup_nf<DT, 5>() && setup_nf<DT, 6>() && setup_nf<DT, 8>();
}

}  // namespace

// the KV-kind items, the absorbed queries, the scores
int apt_launch_absorb_scores16(const ItemParams& p, int dtype, int head_dim, hipStream_t st) {
    return dtype == APT_F16 ? launch_scores_nf<1>(p, head_dim, st) : launch_scores_nf<2>(p, head_dim, st);
}

bool apt_setup_absorb_scores16() { return setup<1>() && setup<2>(); }
