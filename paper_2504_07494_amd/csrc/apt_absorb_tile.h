// What the kernels of the absorbed-weight hidden path share: plan lookups, the split of fp32 operands into 16-bit parts,
// and (16-bit inputs) the tiles of the score and weighted-sum kernels.
#pragma once
#include "apt_device.h"

namespace {

__device__ inline const int32_t* plan_array(const ItemParams& p, int which) {
    return p.plan + APT_PW_HEADER + (int64_t)which * p.B;
}

// address of the cached hidden row of a token
__device__ inline const char* hidden_row(const ItemParams& p, int r, int token, int eb) {
    const int32_t blk = p.block_tables[(int64_t)r * 2 * p.max_blocks + (token >> p.log2_bs)];
    return p.hidden_pages + ((int64_t)blk * p.bs + (token & (p.bs - 1))) * p.d * eb;
}

// Eight fp32 values -> 16-bit parts for the matrix cores, a 16-byte unit per part: fp16 hi + lo (22 bits), bf16 hi + mid + lo
// (24 bits).  The products of the parts with 16-bit inputs are exact in the fp32 accumulator.  Pairs of values go through the
// packed conversions (round to nearest even).
template <int DT> struct AbSplit;
template <> struct AbSplit<1> {
    static constexpr int parts = 2;
    typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
    // the low part times lo_scale (a power of two)
    __device__ static inline void split8(const float* v, uint4* out, float lo_scale = 1.f) {
        uint32_t w[2][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a = v[2 * i], b = v[2 * i + 1];
            // rounded to fp32 here: contracted with the product behind them, the two uses of hi below could round differently
            asm("" : "+v"(a), "+v"(b));
            const h2_t hi = {(_Float16)a, (_Float16)b};
            const h2_t lo = {(_Float16)((a - (float)hi.x) * lo_scale), (_Float16)((b - (float)hi.y) * lo_scale)};
            w[0][i] = __builtin_bit_cast(uint32_t, hi);
            w[1][i] = __builtin_bit_cast(uint32_t, lo);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) out[s] = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
    }
};
template <> struct AbSplit<2> {
    static constexpr int parts = 3;
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    __device__ static inline void split8(const float* v, uint4* out) {
        uint32_t w[3][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a = v[2 * i], b = v[2 * i + 1];
            asm("" : "+v"(a), "+v"(b));
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const b2_t r = {(__bf16)a, (__bf16)b};
                w[s][i] = __builtin_bit_cast(uint32_t, r);
                a -= __uint_as_float(w[s][i] << 16);
                b -= __uint_as_float(w[s][i] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) out[s] = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
    }
};

// gload_lds16 of data that is read once (streamed past the caches)
__device__ inline void gload_lds16_stream(const void* g, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds_addr), "v"(g) : "memory", "m0");
}

// waits until the copies of no more than `tiles` k-tiles are in flight, COPIES each; MOST: of no more than these
template <int MOST, int COPIES> __device__ __forceinline__ void wait_tiles(int tiles) {
    if constexpr (MOST > 0) {
        if (tiles < MOST) return wait_tiles<MOST - 1, COPIES>(tiles);
    }
    wait_vmcnt<MOST * COPIES>();
}

constexpr int kAbTok = APT_ABSORBED_CHUNK;                // tokens per range
constexpr int kAbMT = 256;                                // tokens per workgroup of the score kernel

constexpr int kAbWaves = 8;                               // waves of such a workgroup

// Operand fragments of 16 heads the kernels are built for; heads are padded to 16 * this many rows per part (padded
// rows hold anything: they only reach outputs that are not stored).  An instantiation per count keeps padding and
// registers small: 72 heads are 5 fragments, not the 8 of a multiple of 64.
static inline int ab_head_frags(int H) {
    const int nf = (H + 15) / 16;
    return nf < 2 ? 2 : nf == 7 ? 8 : nf;
}

// Long fp32 sums on the matrix cores round at the size of the running sum, once per part and 32 k: every kAbFold k the
// accumulators are added to a second set and cleared, so that the sum is one of short sums.  Scores of large batches run over
// all of d_model in one slice: their second set goes into a third every kAbFoldSums k.  Error of the hidden-kind outputs
// against 64 bits: an accumulator per part over 512 k, those added in fp32, projection on the plain ALUs / two sets in the scores,
// none in the bf16 projection / as it is:
//     72 heads, 96 requests of 64..2048 tokens, bf16    5.1e-7  / 7.7e-7  / 4.9e-7      fp16  1.15e-6 / 1.26e-6 / 1.15e-6
//     55 heads, 169 requests of 15..79, bf16            3.5e-7  / 5.3e-7  / 3.0e-7
//     40 heads, 32 requests of 128..2048, bf16          4.0e-7  / 3.75e-7 / 3.4e-7      fp16  9.2e-7  / 9.0e-7  / 8.9e-7
//     geometric mean of 53 batches, bf16                3.9e-7  / 3.8e-7  / 3.4e-7
// The third set costs no time; the folded projection 10 us of 1420 (first line; 64 instead of 128 everywhere: another 30).
constexpr int kAbFold = 128;
constexpr int kAbFoldSums = 512;

template <int N> __device__ inline void ab_fold(f32x4_t (*acc)[N], f32x4_t (*sum)[N], int rows) {
#pragma unroll
    for (int i = 0; i < rows; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sum[i][j][e] += acc[i][j][e];
                acc[i][j][e] = 0.f;
            }
}

// LDS tile of KT values of k per row: the fp32 operand as NS parts of R = 16 NF rows, and 256 rows of X.  KT = 64 (whole
// 128-byte lines of X per row) where three stages fit, else 32, with X 64 wide all the same where that fits (kWideX).
template <int DT, int NF> struct AbTile {
    static constexpr int NS = AbSplit<DT>::parts;
    static constexpr int R = 16 * NF;
    static constexpr int kLdsMost = 158 * 1024;
    static constexpr int KT = 3 * (kAbMT + R * NS) * 128 <= kLdsMost ? 64 : 32;
    static constexpr int kRow = KT * 2;
    static constexpr int kABytes = R * NS * kRow;
    // 64-wide X tiles, three stages, beside four of 32-wide operand tiles: a k-tile's copies of either were issued three k-tiles ago
    static constexpr bool kWideX = KT == 32 && 4 * kABytes + 3 * kAbMT * 128 <= kLdsMost;
    static constexpr int XPT = kWideX ? 2 : 1;                    // k-tiles per X tile
    static constexpr int kXRow = kRow * XPT;
    static constexpr int kXBytes = kAbMT * kXRow;
    static constexpr int S = kWideX ? 4 : kLdsMost / (kABytes + kXBytes) < 7 ? kLdsMost / (kABytes + kXBytes) : 7;
    static constexpr int SX = kWideX ? 3 : S;
    static constexpr int kLds = SX * kXBytes + S * kABytes;
    static constexpr int kXCopies = kXBytes / 1024 / kAbWaves;    // 1 KB copies per wave and X tile
    static constexpr int kACopies = (kABytes / 1024 + kAbWaves - 1) / kAbWaves;
    static constexpr int NF0 = (NF + 1) / 2;                    // head fragments of waves 0..3; waves 4..7 take the rest
    static constexpr int kCopies = kXCopies / XPT + kACopies;     // per wave and k-tile
    static_assert(S >= 3 && (S - 2) * kCopies <= 63, "stages / vmcnt range");
};
// unit c of a row sits at c ^ ab_swz(row): the 16-row operand reads are free of bank conflicts
template <int KT> __host__ __device__ inline int ab_swz(int row) { return (row >> 1) & (KT / 8 - 1); }

}  // namespace
