// Absorbed-weight hidden path, 16-bit inputs: the output projection of the weighted sums.
#include "apt_device.h"
#include "apt_launch.h"
#include "apt_absorb_tile.h"

namespace {

// OP[slice][hr][h][:] = (sum of the request's units of YP)[rows of the slice] W_V[rows of the slice, h]
//
// Workgroup = one head, 16 RF requests, one slice of d_model; its four waves take every fourth step of 32 rows and run
// without barriers, each with its own two LDS stages: the 32 rows of W_V as they lie (read with the transposing LDS read)
// and 32 fp32 values of YP per request.  YP is split into 16-bit parts in registers and multiplied on v_mfma_f32_16x16x32
// (D rows = channels, columns = requests).  fp16 parts: a request's sums are scaled by a power of two that puts the largest
// of the wave's first step at 4 to 8, so that they keep their bits whatever their magnitude; the low part is kept 2^11 times
// larger, so that it is not subnormal, in accumulators of its own.  Where a later sum passes 2^15 (4096 times the first ones)
// the wave does its steps again with the scale of the largest: rescaling the accumulators on the way takes registers that
// three request fragments do not have.  Error of the outputs against 64 bits, hidden vectors of magnitude 1 / 1e-3 / 1e-4 / 1e-5, 32 heads:
// 6.0e-7 / 1.7e-7 / 1.7e-7 / 1.5e-7 (fp32 products on the plain ALUs 6.4e-7 / 2.2e-7 / 2.3e-7 / 1.7e-7; scaled by the softmax
// denominator only 6.0e-7 / 3.7e-7 / 3.3e-6 / 2.7e-5), at the same time.
//
// Bound by the reads of YP (fp32, H d_model values per unit) and of W_V, once per group of 16 RF requests: 114-125 us for
// 72 heads, bf16, 96 requests at d_model 9216 (255 MB of YP, W_V twice; 108 us without folding the sums, 480 us on the plain
// ALUs, whose output partials per 256 rows took the last kernel another 30 us), 28 us for 40 heads, fp16, 32 requests (70 us).
template <int DT, int HD, int RF> struct OutTile {
    static constexpr int NS = AbSplit<DT>::parts;
    static constexpr int NA = DT == 1 ? 2 : 1;              // accumulator sets
    static constexpr bool kFolded = DT == 2;                // long sums folded (kAbFold); the two fp16 sets leave no registers for it
    static constexpr int CF = HD / 16;
    static constexpr int kWRow = HD * 2;
    static constexpr int kWBytes = 32 * kWRow;
    static constexpr int kYBytes = RF * 2048;
    static constexpr int kWCopies = kWBytes / 1024, kYCopies = kYBytes / 1024;
    static constexpr int kWave = 2 * (kWBytes + kYBytes);   // LDS of a wave
    static_assert(CF * RF * 1024 <= kWave, "accumulators of the waves meet in the stages");
};
template <int HD> __device__ inline int out_swz(int k) {     // 32-byte units of the W_V rows; rows of 128 bytes hold four
    return HD == 128 ? wswz(k) : ((k >> 1) & 1) | ((k >> 2) & 2);
}
constexpr float kLoScale = 2048.f;
constexpr int kTopBits = 3, kRangeBits = 15;                 // scaled sums: largest at first, most

template <int DT, int HD, int RF>
__global__ __launch_bounds__(kThreads, HD == 64 ? 2 : 1) void apt_absorb_out16_kernel(ItemParams p) {
    using C = OutTile<DT, HD, RF>;
    constexpr int NS = C::NS, CF = C::CF;
    extern __shared__ __align__(16) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, qd = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.x, hr0 = blockIdx.y * 16 * RF;
    const int n_steps = p.d / 32, z = blockIdx.z, n_slices = gridDim.z;
    const int s_begin = (int)((int64_t)z * n_steps / n_slices) + w, s_end = (int)((int64_t)(z + 1) * n_steps / n_slices);
    const int32_t* hid_req = plan_array(p, APT_PA_HID_REQ);
    auto units_of = [&](int hr) { return (plan_array(p, APT_PA_SPLIT_COUNT)[hid_req[hr]] + p.ab_group - 1) / p.ab_group; };
    auto slot_of = [&](int i) { return min(hr0 + i, p.n_hid_req - 1); };      // requests past the last repeat it (not stored)

    // copy sources: YP chunk n holds requests 8 n .. + 7 (unit c of a row at c ^ row), W_V chunk n rows of kWRow bytes
    const char* ysrc[C::kYCopies];
    int ylast[C::kYCopies];
#pragma unroll
    for (int n = 0; n < C::kYCopies; ++n) {
        const int hr = slot_of(8 * n + (lane >> 3));
        ysrc[n] = (const char*)(p.ab_yp + ((int64_t)plan_array(p, APT_PA_HID_CHUNK_OFF)[hid_req[hr]] * p.H + h) * p.d) + (((lane & 7) ^ (lane >> 3)) << 4);
        ylast[n] = units_of(hr) - 1;
    }
    const int64_t ystep = (int64_t)p.ab_group * p.H * p.d * 4;                // from one unit to the next
    const char* wsrc[C::kWCopies];
#pragma unroll
    for (int n = 0; n < C::kWCopies; ++n) {
        const int at = n * 1024 + lane * 16, k = at / C::kWRow, b = at % C::kWRow;
        wsrc[n] = p.W_V + ((int64_t)k * p.d + h * HD) * 2 + (((b >> 5) ^ out_swz<HD>(k)) << 5) + (b & 16);
    }
    // this lane's requests as columns of D
    int count[RF], most = 1;
    int ex[RF];                                              // fp16: exponent of the largest sum the scale was chosen for
#pragma unroll
    for (int f = 0; f < RF; ++f) {
        const int hr = slot_of(16 * f + l16);
        count[f] = units_of(hr);
        ex[f] = -100;
        most = max(most, count[f]);
    }
#pragma unroll
    for (int i = 1; i < 16; i *= 2) most = max(most, __shfl_xor(most, i));
    most = __builtin_amdgcn_readfirstlane(most);

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + w * C::kWave;
    const uint32_t yst = lds0 + 2 * C::kWBytes;
    // the stages alternate by themselves: W_V per step, YP per (step, unit)
    auto issue_w = [&](int step, int stage) {
#pragma unroll
        for (int n = 0; n < C::kWCopies; ++n) gload_lds16(wsrc[n] + (int64_t)step * 32 * p.d * 2, lds0 + stage * C::kWBytes + n * 1024);
    };
    auto issue_y = [&](int step, int u, int stage) {
#pragma unroll
        for (int n = 0; n < C::kYCopies; ++n) gload_lds16_stream(ysrc[n] + min(u, ylast[n]) * ystep + step * 128, yst + stage * C::kYBytes + n * 1024);
    };
    uint32_t waddr[CF];
#pragma unroll
    for (int c = 0; c < CF; ++c) {
        const int k = 8 * qd + (l16 >> 2);
        waddr[c] = lds0 + k * C::kWRow + ((c ^ out_swz<HD>(k)) << 5) + (l16 & 3) * 8;
    }
    const uint32_t yaddr[2] = {yst + l16 * 128 + (((2 * qd) ^ (l16 & 7)) << 4), yst + l16 * 128 + (((2 * qd + 1) ^ (l16 & 7)) << 4)};

    f32x4_t acc[C::NA][CF][RF], sum[C::kFolded ? CF : 1][RF];
    float y[RF][8];
    float top[RF];                                            // fp16: largest sum of this lane
#pragma unroll
    for (int f = 0; f < RF; ++f) top[f] = 0.f;
    // whether a sum seen so far is too large for the scale; if so, the exponents of the largest ones are taken
    auto outgrown = [&]() {
        bool over = false;
#pragma unroll
        for (int f = 0; f < RF; ++f) over |= top[f] >= __builtin_amdgcn_ldexpf(1.f, ex[f] + kRangeBits - kTopBits);
        if (!__any(over)) return false;
        bool grown = false;
#pragma unroll
        for (int f = 0; f < RF; ++f) {
            // the four lane groups hold a request's 32 sums of a step (an infinite one has exponent 0 here)
            top[f] = fmaxf(top[f], __shfl_xor(top[f], 16));
            top[f] = fmaxf(top[f], __shfl_xor(top[f], 32));
            const int now = top[f] > 0.f ? __builtin_amdgcn_frexp_expf(top[f]) : ex[f];
            grown |= now > ex[f];
            ex[f] = max(ex[f], now);
        }
        return (bool)__any(grown);
    };
    do {
#pragma unroll
        for (int a = 0; a < C::NA; ++a)
#pragma unroll
            for (int c = 0; c < CF; ++c)
#pragma unroll
                for (int f = 0; f < RF; ++f)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[a][c][f][e] = 0.f;
        if constexpr (C::kFolded)
#pragma unroll
            for (int c = 0; c < CF; ++c)
#pragma unroll
                for (int f = 0; f < RF; ++f)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[c][f][e] = 0.f;
        int ys = 0, ws = 0;
        if (s_begin < s_end) {
            issue_w(s_begin, 0);
            issue_y(s_begin, 0, 0);
        }
        for (int step = s_begin; step < s_end; step += 4) {
            for (int u = 0; u < most; ++u) {
                // the next (step, unit) is on its way while this one is used; this wave's LDS reads of the stages it refills are done
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (u + 1 < most) {
                    issue_y(step, u + 1, ys ^ 1);
                    wait_vmcnt<C::kYCopies>();
                } else if (step + 4 < s_end) {
                    issue_w(step + 4, ws ^ 1);
                    issue_y(step + 4, 0, ys ^ 1);
                    wait_vmcnt<C::kWCopies + C::kYCopies>();
                } else {
                    wait_vmcnt<0>();
                }
#pragma unroll
                for (int f = 0; f < RF; ++f)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        float v[4];
                        cvt16<0>(lds_read16(yaddr[i] + ys * C::kYBytes + f * 2048), v);
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[f][4 * i + e] = (u == 0 ? 0.f : y[f][4 * i + e]) + (u < count[f] ? v[e] : 0.f);
                    }
                ys ^= 1;
            }
            if constexpr (DT == 1) {
#pragma unroll
                for (int f = 0; f < RF; ++f)
#pragma unroll
                    for (int e = 0; e < 8; ++e) top[f] = fmaxf(top[f], fabsf(y[f][e]));
                if (step == s_begin) outgrown();
            }
            uint4 wf[CF];
#pragma unroll
            for (int c = 0; c < CF; ++c) {
                const uint2 lo = lds_read_tr(waddr[c] + ws * C::kWBytes), hi = lds_read_tr(waddr[c] + ws * C::kWBytes + 4 * C::kWRow);
                wf[c] = make_uint4(lo.x, lo.y, hi.x, hi.y);
            }
#pragma unroll
            for (int f = 0; f < RF; ++f) {
                uint4 part[NS];
                if constexpr (DT == 1) {
                    const float scale = __builtin_amdgcn_ldexpf(1.f, kTopBits - ex[f]);
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = y[f][e] * scale;
                    AbSplit<DT>::split8(v, part, kLoScale);
                } else {
                    AbSplit<DT>::split8(y[f], part);
                }
#pragma unroll
                for (int s = 0; s < NS; ++s) {
#pragma unroll
                    for (int c = 0; c < CF; ++c) acc[C::NA == 2 ? s : 0][c][f] = mfma16<DT>(wf[c], part[s], acc[C::NA == 2 ? s : 0][c][f]);
                }
            }
            ws ^= 1;
            if constexpr (C::kFolded)
                if ((step - s_begin) % (4 * kAbFold / 32) == 4 * (kAbFold / 32 - 1)) ab_fold<RF>(acc[0], sum, CF);
        }
    } while (DT == 1 && outgrown());
    // the waves' sums meet in LDS, each in the wave's own stages
#pragma unroll
    for (int c = 0; c < CF; ++c)
#pragma unroll
        for (int f = 0; f < RF; ++f) {
            f32x4_t v = acc[0][c][f];
            if constexpr (C::kFolded) v += sum[c][f];
            if constexpr (C::NA == 2)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = fmaf(acc[1][c][f][e], 1.f / kLoScale, v[e]) * __builtin_amdgcn_ldexpf(1.f, ex[f] - kTopBits);
            *(f32x4_t*)(lds + w * C::kWave + ((c * RF + f) * 64 + lane) * 16) = v;
        }
    __syncthreads();
    for (int i = tid; i < CF * RF * 64; i += kThreads) {
        const int c = i / 64 / RF, f = i / 64 % RF;           // lane = i % 64 of the wave that wrote it
        const int hr = hr0 + 16 * f + l16;
        f32x4_t v = *(const f32x4_t*)(lds + i * 16);
#pragma unroll
        for (int k = 1; k < 4; ++k) v += *(const f32x4_t*)(lds + k * C::kWave + i * 16);
        if (hr < p.n_hid_req) *(f32x4_t*)(p.ab_op + (((int64_t)z * p.n_hid_req + hr) * p.H + h) * HD + 16 * c + 4 * qd) = v;
    }
}

template <int DT, int HD, int RF> int launch(const ItemParams& p, hipStream_t st) {
    constexpr int kLds = 4 * OutTile<DT, HD, RF>::kWave;
    const dim3 grid(p.H, (p.n_hid_req + 16 * RF - 1) / (16 * RF), p.ab_os);
    hipLaunchKernelGGL((apt_absorb_out16_kernel<DT, HD, RF>), grid, dim3(kThreads), kLds, st, p);
    return hipGetLastError() == hipSuccess ? APT_OK : APT_EHIP;
}
template <int DT, int HD> int launch_rf(const ItemParams& p, int rf, hipStream_t st) {
    switch (rf) {
    case 1: return launch<DT, HD, 1>(p, st);
    case 2: return launch<DT, HD, 2>(p, st);
    default: return launch<DT, HD, 3>(p, st);
    }
}
template <int DT, int HD> bool setup() {
    return apt_raise_lds_limit(apt_absorb_out16_kernel<DT, HD, 1>) && apt_raise_lds_limit(apt_absorb_out16_kernel<DT, HD, 2>) &&
           apt_raise_lds_limit(apt_absorb_out16_kernel<DT, HD, 3>);
}

}  // namespace

// Requests of a workgroup: all of them up to 48 (64 spill in fp16), else equal groups.  Slices of d_model: workgroups run in rounds of one per
// CU, a slice costs a wave its steps and a start-up of about four; at most the slices the workspace has room for.
int apt_absorb_out16_groups(int n_hid_req, int* rf) {
    const int frags = (n_hid_req + 15) / 16, groups = (frags + 2) / 3;
    *rf = (frags + groups - 1) / groups;
    return (n_hid_req + 16 * *rf - 1) / (16 * *rf);
}
int apt_absorb_out16_slices(const ItemParams& p, int n_cus, int most) {
    int rf = 1;
    const int64_t per_slice = (int64_t)p.H * apt_absorb_out16_groups(p.n_hid_req, &rf);
    const int n_steps = p.d / 32;
    int best = 1;
    int64_t best_cost = 0;
    for (int z = 1; z <= most && 4 * z <= n_steps; ++z) {
        const int64_t cost = (per_slice * z + n_cus - 1) / n_cus * ((n_steps + 4 * z - 1) / (4 * z) + 4);
        if (z == 1 || cost < best_cost) { best = z; best_cost = cost; }
    }
    return best;
}

int apt_launch_absorb_out16(const ItemParams& p, int dtype, int head_dim, hipStream_t st) {
    int rf = 1;
    apt_absorb_out16_groups(p.n_hid_req, &rf);
    if (dtype == APT_F16) return head_dim == 128 ? launch_rf<1, 128>(p, rf, st) : launch_rf<1, 64>(p, rf, st);
    return head_dim == 128 ? launch_rf<2, 128>(p, rf, st) : launch_rf<2, 64>(p, rf, st);
}

bool apt_setup_absorb_out16() { return setup<1, 128>() && setup<1, 64>() && setup<2, 128>() && setup<2, 64>(); }
