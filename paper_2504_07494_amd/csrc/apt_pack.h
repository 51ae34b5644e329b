// Tiles of the projection kernel on packed weights that hold the last, shorter ranges of several requests.
//
// The ranges of a head are projected with the same weights, so one tile of token rows can take the short ranges of
// several requests; only scores, softmax and output are per range.  A tile is cut into blocks of 32 rows and a range
// starts at a block.  The planner decides per head queue how many blocks a shared tile may fill (its word
// APT_PW_SHARED_TILES, four bits a queue, 0 = every range gets a tile of its own); which ranges share a tile follows
// from that and from the lengths alone, by the rule below, so the list of items stays as it is.
//
// Tiles of 320 rows can also serve ranges of 256 tokens: then the full ranges share
// tiles as well (a cap of 9 or 10 blocks).
//
// Attention call with a tile per range / shared tiles, us, fp16, one run: 40 heads, 256 requests of 128 tokens 3461 / 2513, 512 of 32
// tokens 5328 / 1300, three of 415, 513 and 619 tokens 176 / 157; 72 heads, 256 of 160 tokens 14 130 / 10 710; half of the requests on
// the hidden cache: 40 heads, 64 of 128..2048 tokens 2812 / 2694; 72 heads, 256 of 64..2048 39 320 / 38 020.
//
// A queue's short ranges are sorted by decreasing length, hence by decreasing class (number of blocks).  A pattern
// names how many ranges of each class a tile takes, the largest classes first, and is used as often as the ranges
// last; then the next pattern is formed from what is left.
#pragma once
#include <stdint.h>
#include "apt_internal.h"

#ifdef __HIPCC__
#define APT_HOST_DEVICE __host__ __device__
#else
#define APT_HOST_DEVICE
#endif

#define APT_PACK_BLOCK 32
#define APT_PACK_MAX_BLOCKS (APT_MFMA_HIDDEN_CHUNK / APT_PACK_BLOCK)
// A pattern that ends leaves fewer ranges of one class than a tile could take of it, so class c ends at most
// blocks / c patterns: at most 27 for tiles of 10 blocks, 20 for 8.
#define APT_PACK_MAX_PATTERNS 32

// Whether a plan with ranges of 256 tokens asks for tiles of 320 rows: a cap beyond 8 in one of its queues.
APT_HOST_DEVICE static inline bool apt_pack_wide(uint32_t word) {
    bool wide = false;
    for (int x = 0; x < APT_N_QUEUES; ++x) wide |= ((word >> (4 * x)) & 15) > APT_MFMA_HIDDEN_CHUNK_SMALL / APT_PACK_BLOCK;
    return wide;
}

// NC: blocks of a tile.  Ranges that may share a tile: bounded by the LDS next to the stages of the k loop.
template <int NC> struct apt_pack_tile { static constexpr int max_ranges = NC == 10 ? 6 : 8; };

// left[c], c = 1 .. NC: ranges of class c; used up.  emit(reps, take): a pattern of take[c] ranges of class c, reps tiles.
template <int NC, class Emit>
APT_HOST_DEVICE static inline void apt_pack_patterns(int32_t* left, int cap, Emit emit) {
    for (int i = 0; i < APT_PACK_MAX_PATTERNS; ++i) {
        int32_t take[NC + 1], reps = 0x7fffffff;
        int room = cap, n = 0;
        take[0] = 0;
#pragma unroll
        for (int c = NC; c >= 1; --c) {
            int t = room / c;
            if (n == 0 && t == 0 && left[c] > 0) t = 1;          // a range longer than the cap: alone
            if (t > apt_pack_tile<NC>::max_ranges - n) t = apt_pack_tile<NC>::max_ranges - n;
            if (t > left[c]) t = left[c];
            take[c] = t;
            n += t;
            room -= t * c;
            if (room < 0) room = 0;
            if (t > 0 && (int64_t)reps * t > left[c]) reps = t == 1 ? left[c] : left[c] / t;
        }
        if (n == 0) return;
#pragma unroll
        for (int c = 1; c <= NC; ++c) left[c] -= reps * take[c];
        emit(reps, take);
    }
}
