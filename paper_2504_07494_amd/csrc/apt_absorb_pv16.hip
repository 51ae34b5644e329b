// Absorbed-weight hidden path, 16-bit inputs: the weighted sums of the cached rows.
#include <type_traits>
#include "apt_device.h"
#include "apt_launch.h"
#include "apt_absorb_tile.h"

namespace {

// YP[range][h][:] = sum_j 2^(s_j - m) x_j over the ranges of one unit (one to four 512-token ranges of a request, listed
// in the plan; the result lies at the unit's first range).
//
// Workgroup = one unit x CW columns x all heads, eight waves, a wave owns CW / 8 columns.  D rows are columns of x, D
// columns are heads, k = tokens on v_mfma_f32_16x16x32; the 16-bit parts of a weight are summed in one accumulator.
// k-tiles of 32 tokens go global -> LDS without registers, as many stages as LDS holds: X rows as they lie (1 KB or 512
// contiguous bytes of a row; read with the transposing LDS read, which gives a lane the four tokens of one column, the
// 32-byte units of a row at u ^ wswz(token) so that its four rows fall on different banks) and the weight parts in the
// order the statistics kernel wrote them.
//
// Bound by memory and the matrix pipes together (X once, and NS parts of every head per column).  512 columns halve the
// weight bytes an X byte brings along.  256 are taken where three stages then fit in half of LDS (fp16 up to 80 heads, bf16 up
// to 48), so that one workgroup's start-up and stores are covered by the other's loop, where the stages or accumulators of 512 do
// not fit at all, and in batches that would leave CUs without a unit.
//
// 72 heads, bf16, 96 requests with 102 k tokens at d_model 9216 (1.9 GB of X): 450-480 us (whole call, copies of a k-tile in one go / between
// the products / and X past the caches, by apt_absorbed_past, 1350 / 1325 / 1304; the kernel without its products 393, with X from the caches 457), 1200 us with heads padded to 128
// in two passes over X, a 16-bit gather per operand and sums per 512-token range.  40 heads, fp16, 33.6 k tokens at
// d_model 5120 (344 MB): 80 us with 256 columns and two workgroups per CU, 87 us with 512 and one, 86 us before.
template <int DT, int NF, int CW> struct PvTile {
    static constexpr int NS = AbSplit<DT>::parts;
    static constexpr int R = 16 * NF;
    static constexpr int kRow = CW * 2;
    static constexpr int kXBytes = 32 * kRow;
    static constexpr int kPBytes = R * NS * 64;
    static constexpr int kStage = kXBytes + kPBytes;
    // three stages of a 256-column tile in half of LDS: two workgroups share a CU
    static constexpr bool kTwo = CW == 256 && 3 * kStage <= 78 * 1024;
    static constexpr int kLdsMost = (kTwo ? 78 : 156) * 1024;
    static constexpr int S = kLdsMost / kStage < 6 ? kLdsMost / kStage : 6;
    static constexpr int kXCopies = kXBytes / 1024 / kAbWaves;     // 1 KB copies per wave and k-tile
    static constexpr int kPCopies = (kPBytes / 1024 + kAbWaves - 1) / kAbWaves;
    static constexpr int kCopies = kXCopies + kPCopies;
    static constexpr int CF = CW / kAbWaves / 16;                  // column fragments of a wave
    // stages in LDS, and both accumulator sets in the 256 registers of a wave (two per SIMD) with room for the rest: 8 head
    // fragments x 512 columns would need all 256 (103 spilled; fp16, 112 heads of 128, 48 requests 1366 us, 1066 with 256 columns)
    static constexpr bool kFits = S >= 3 && 2 * NF * CF * 4 <= 192;
    static_assert((S - 2) * kCopies <= 63, "vmcnt range");
};
constexpr int kAhead = 2;                                 // weight operands read ahead of the products
constexpr int kPvBlkBytes = APT_ABSORBED_MAX_GROUP * APT_ABSORBED_CHUNK / 4 * 4;      // block ids of a unit, blocks of 4 tokens at least

// PAST: X is read past the caches
template <int DT, int NF, int CW, bool PAST>
__global__ __launch_bounds__(kAbWaves * 64) void apt_absorb_pv16_kernel(ItemParams p, int n_cslices) {
    using C = PvTile<DT, NF, CW>;
    constexpr int NS = C::NS, S = C::S, CF = C::CF;
    constexpr int RPC = 1024 / C::kRow;                  // rows per 1 KB copy
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, qd = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // longest units first, the column slices of a unit side by side (dealt over the XCDs, which balances them; each XCD
    // then reads the weights of every unit once, a small part of what it reads of X)
    const int c0 = (int)(blockIdx.x % n_cslices) * CW;
    const int range = p.plan[p.ab_units_off + blockIdx.x / n_cslices];
    const int4 it = ((const int4*)(p.plan + p.items_off))[range];
    const int r = it.x, t0 = it.z;
    const int len = min(plan_array(p, APT_PA_CTX_LEN)[r] - t0, p.ab_group * kAbTok);
    const int nkt = (len + 31) >> 5;
    int32_t* blk = (int32_t*)(lds + S * C::kStage);
    const int nblk = (len + p.bs - 1) >> p.log2_bs;
    for (int i = tid; i < nblk; i += kAbWaves * 64)
        blk[i] = p.block_tables[(int64_t)r * 2 * p.max_blocks + (t0 >> p.log2_bs) + i];
    __syncthreads();

    const char* psrc = (const char*)p.ab_pp + ((int64_t)plan_array(p, APT_PA_HID_CHUNK_OFF)[r] * (kAbTok / 32) + (t0 >> 5)) * C::kPBytes + lane * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    int row_of[C::kXCopies], col_of[C::kXCopies];        // row of the k-tile and byte offset in a token row this lane copies
#pragma unroll
    for (int i = 0; i < C::kXCopies; ++i) {
        const int at = lane * 16 % C::kRow;
        row_of[i] = RPC * (C::kXCopies * w + i) + lane * 16 / C::kRow;
        // columns past d_model repeat the last eight (never stored)
        col_of[i] = min(c0 + ((at >> 5) ^ wswz(row_of[i])) * 16 + ((at >> 4) & 1) * 8, p.d - 8) * 2;
    }
    // copy i of k-tile kt, its X rows from xsrc as row_sources left them
    const char* xsrc[C::kXCopies];
    auto row_sources = [&](int kt) {
#pragma unroll
        for (int i = 0; i < C::kXCopies; ++i) {
            const int rel = min(kt * 32 + row_of[i], len - 1);     // rows past the range repeat its last token (their weights are zero)
            xsrc[i] = p.hidden_pages + ((int64_t)blk[rel >> p.log2_bs] * p.bs + (rel & (p.bs - 1))) * p.d * 2 + col_of[i];
        }
    };
    auto copy = [&](int kt, int i) {
        const uint32_t st = lds0 + (kt % S) * C::kStage;
        if (i < C::kXCopies) {
            if constexpr (PAST) gload_lds16_stream(xsrc[i], st + (C::kXCopies * w + i) * 1024);
            else gload_lds16(xsrc[i], st + (C::kXCopies * w + i) * 1024);
        } else {                                         // some waves copy the last chunk again (same bytes)
            const int n = min(w + kAbWaves * (i - C::kXCopies), C::kPBytes / 1024 - 1);
            gload_lds16(psrc + (int64_t)kt * C::kPBytes + n * 1024, st + C::kXBytes + n * 1024);
        }
    };
    uint32_t xaddr[CF];
#pragma unroll
    for (int c = 0; c < CF; ++c) {
        const int k = 8 * qd + (l16 >> 2);
        xaddr[c] = lds0 + k * C::kRow + (((w * CF + c) ^ wswz(k)) << 5) + (l16 & 3) * 8;
    }
    const uint32_t paddr = lds0 + C::kXBytes + l16 * 64 + ((qd ^ ab_swz<32>(l16)) << 4);
    f32x4_t acc[NF][CF], sum[NF][CF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int c = 0; c < CF; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[f][c][e] = sum[f][c][e] = 0.f;
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        if (s >= nkt) continue;
        row_sources(s);
#pragma unroll
        for (int i = 0; i < C::kCopies; ++i) copy(s, i);
    }
    row_sources(S - 1);
    int stage = 0;
    // The copies of the k-tile S - 1 ahead go out one by one between the products: asked for in one go, a wave would be held until
    // the copy path has taken all of the workgroup's.  Their row addresses are worked out an iteration ahead.
    auto step = [&](int kt, auto refill) {
        __syncthreads();            // k-tile kt has landed for every wave; nobody still reads the stage refilled next
        const uint32_t so = stage * C::kStage;
        uint4 xf[CF], pf[kAhead + 1];
#pragma unroll
        for (int c = 0; c < CF; ++c) {
            const uint2 lo = lds_read_tr(xaddr[c] + so), hi = lds_read_tr(xaddr[c] + so + 4 * C::kRow);
            xf[c] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        constexpr int G = NS * NF;
        auto read = [&](int g) { pf[g % (kAhead + 1)] = lds_read16(paddr + so + (g / NF * C::R + 16 * (g % NF)) * 64); };
#pragma unroll
        for (int g = 0; g < kAhead; ++g) read(g);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g + kAhead < G) read(g + kAhead);
            if constexpr (refill)
#pragma unroll
                for (int i = g * C::kCopies / G; i < (g + 1) * C::kCopies / G; ++i) copy(kt + S - 1, i);
#pragma unroll
            for (int c = 0; c < CF; ++c) acc[g % NF][c] = mfma16<DT>(xf[c], pf[g % (kAhead + 1)], acc[g % NF][c]);
        }
        if constexpr (refill) row_sources(kt + S);
        stage = stage == S - 1 ? 0 : stage + 1;
        if ((kt + 1) % (kAbFold / 32) == 0) ab_fold<CF>(acc, sum, NF);
    };
    int kt = 0;
    for (; kt + S - 1 < nkt; ++kt) {
        wait_vmcnt<(S - 2) * C::kCopies>();
        step(kt, std::true_type{});
    }
    for (; kt < nkt; ++kt) {
        // for this k-tile, not for all that are in flight: attention call in a graph, all / this one, 40 heads, fp16, a request of 1500
        // tokens 65.4 -> 65.0 us, 25 heads, 82 requests of 55..181, half hidden-kind 73.3 -> 72.8
        wait_tiles<S - 2, C::kCopies>(nkt - 1 - kt);
        step(kt, std::false_type{});
    }
    ab_fold<CF>(acc, sum, NF);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int h = 16 * f + l16;
        if (h >= p.H) continue;
        float* y = p.ab_yp + ((int64_t)range * p.H + h) * p.d;
#pragma unroll
        for (int c = 0; c < CF; ++c) {
            const int col = c0 + 16 * (w * CF + c) + 4 * qd;
            if (col < p.d) *(f32x4_t*)(y + col) = sum[f][c];
        }
    }
}

template <int DT, int NF, int CW> int launch_cw(const ItemParams& p, hipStream_t st) {
    using C = PvTile<DT, NF, CW>;
    const int n_cslices = (p.d + CW - 1) / CW;
    const dim3 grid((unsigned)(p.ab_units * n_cslices)), block(kAbWaves * 64);
    constexpr int kLds = C::S * C::kStage + kPvBlkBytes;
    if (p.ab_past & APT_AB_PAST_SUMS) hipLaunchKernelGGL((apt_absorb_pv16_kernel<DT, NF, CW, true>), grid, block, kLds, st, p, n_cslices);
    else hipLaunchKernelGGL((apt_absorb_pv16_kernel<DT, NF, CW, false>), grid, block, kLds, st, p, n_cslices);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}
template <int DT, int NF> int launch_nf(const ItemParams& p, int n_cus, hipStream_t st) {
    if constexpr (PvTile<DT, NF, 512>::kFits && !PvTile<DT, NF, 256>::kTwo)
        if ((int64_t)p.ab_units * ((p.d + 511) / 512) >= n_cus) return launch_cw<DT, NF, 512>(p, st);
    return launch_cw<DT, NF, 256>(p, st);
}
template <int DT> int launch(const ItemParams& p, int n_cus, hipStream_t st) {
    switch (ab_head_frags(p.H)) {
    case 2: return launch_nf<DT, 2>(p, n_cus, st);
    case 3: return launch_nf<DT, 3>(p, n_cus, st);
    case 4: return launch_nf<DT, 4>(p, n_cus, st);
    case 5: return launch_nf<DT, 5>(p, n_cus, st);
    case 6: return launch_nf<DT, 6>(p, n_cus, st);
    default: return launch_nf<DT, 8>(p, n_cus, st);
    }
}
template <int DT, int NF, int CW> bool setup_cw() {
    return apt_raise_lds_limit(apt_absorb_pv16_kernel<DT, NF, CW, false>) && apt_raise_lds_limit(apt_absorb_pv16_kernel<DT, NF, CW, true>);
}
template <int DT, int NF> bool setup_nf() {
    if constexpr (PvTile<DT, NF, 512>::kFits && !PvTile<DT, NF, 256>::kTwo)
        if (!setup_cw<DT, NF, 512>()) return false;
    return setup_cw<DT, NF, 256>();
}
template <int DT> bool setup() {
    return setup_nf<DT, 2>() && setup_nf<DT, 3>() && setup_nf<DT, 4>() && setup_nf<DT, 5>() && setup_nf<DT, 6>() && setup_nf<DT, 8>();
}

}  // namespace

int apt_launch_absorb_pv16(const ItemParams& p, int dtype, int n_cus, hipStream_t st) {
    return dtype == APT_F16 ? launch<1>(p, n_cus, st) : launch<2>(p, n_cus, st);
}

bool apt_setup_absorb_pv16() { return setup<1>() && setup<2>(); }
