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

// Time of a tile of NC blocks of which `blocks` hold tokens of `ranges` ranges, ns, all workgroups busy: prologue and epilogue, then the
// k loop, whose copies do not shrink with the rows that hold tokens.  Measured, us a tile of 2, 4, 6, 8 (and 10) blocks: NC 8, d_model 1024:
// 18, 22, 28, 32; 3072: 35, 47, 61, 76; 5120: 53, 74, 97, 122.  NC 10, 1024: 22, 27, 33, 38, 47; 5120: 59, 81, 102, 126, 156; 9216:
// 140, 186, 218, 242, 282 (there the weights of an XCD's heads no longer come from its L2).  A further range in a tile takes 0.5 to 1.5 us more.
static inline int64_t apt_tile_ns(int NC, int d, int blocks, int ranges) {
    const int64_t b = blocks > 2 ? blocks : 2;
    if (NC == 8) return 10000 + d * (20000 + 11100 * b) / 5120 + 800 * (ranges - 1);
    return 11000 + 800 * b + d * (d < APT_MFMA_LARGE_TILE_D_MODEL ? 4300 + 2280 * b : 11100 + 1880 * b) / 1024 + 1100 * (ranges - 1);
}

// Time of the KV-kind items of a launch with packed weights on the whole chip, ns: 4 d bytes a token at 5.5 TB/s.
static inline int64_t apt_kv_ns(int64_t kv_tokens, int d) { return kv_tokens * d / 1375; }

// Heads dealt to all XCDs.  Queue x holds the heads h with h % 8 == x and runs on XCD x; with a head count that is no multiple of eight the
// first H % 8 queues have a head more than the others.  The tiles of these heads can be dealt to all XCDs in turn: XCD x takes its own
// other heads as always, and tile t of the dealt head of queue q where (t + q) % 8 == x.  Dealt launches share tiles by one cap for all
// queues, that of the queues with the nearer number of heads (the other one where that is 0); below eight heads all are dealt.
APT_HOST_DEVICE static inline int apt_dealt_cap(uint32_t word, int H) {
    const int more = H & 7, cap_long = word & 15, cap_short = H < 8 ? cap_long : (int)(word >> (4 * more)) & 15;
    const int nearer = more >= 4 ? cap_long : cap_short;
    return nearer ? nearer : cap_long > cap_short ? cap_long : cap_short;
}

// The i-th tile of XCD x: the number of the tile among its head's (returned; from the number of a head's tiles on: none, nor are the later
// ones), the queue of the head and its place among that queue's heads.  nh = H / 8 heads of the XCD's own, more = H % 8 dealt ones.
APT_HOST_DEVICE static inline int apt_dealt_tile(int i, int x, int nh, int more, int* queue, int* place) {
    const int per_eight = 8 * nh + more;                      // tiles of this XCD among tiles 8 j .. 8 j + 7 of every head
    int at = i / per_eight * 8, left = i % per_eight, q;
    for (;;) {                                                // (ends within eight steps: q is every queue once)
        q = (x - at) & 7;
        const int here = nh + (q < more);
        if (left < here) break;
        left -= here;
        ++at;
    }
    *queue = left < nh ? x : q;
    *place = left;
    return at;
}

// Whether a launch deals: counts with up to four such heads (below eight any), where the longer queues hold four rounds of tiles or
// more, and in shorter launches where that saves a round; not in launches of less than four rounds of ranges whose queues share tiles
// differently, nor where KV-kind items fill four fifths of what the shorter queues leave idle (they go to whoever is free).
// Whole step, us, a queue's heads on its XCD / dealt: 3 heads, 64 requests of 64..1024 tokens 100.8 / 59.4; 17 heads, 247 of 32..300
// 861 / 671; 18 heads, 60 of 100..600 391 / 309; 41 heads, 109 of 10..90 686 / 617; 60 heads, 28 of 636..1941 12.8 / 11.4 ms; 26 heads, two
// of 1064 tokens 128 / 92.  Where the rule does not: 69 heads, 30 of 100..800 2778 / 2852 (each XCD reads the weights of all these
// heads; five to seven such heads were timed there and at 30 heads only); a round saved by nobody: 43 heads, three of 20..200 75.2 / 77.8,
// 36 heads, eleven of 28 69.2 / 73.6, and with four rounds of ranges in fewer of tiles 65 heads, 16 of 130..275 802 / 834, 20 heads, 91 of 29..95
// beside as many KV-kind ones 183 / 188 (of 60 attention calls with four rounds of ranges all nine that saved no round of less than four
// took 0.99 to 1.04 of the time dealt, the 13 that did 0.67 to 1.02); tiles shared by another queue's cap: 51 heads, twelve of 75 190 / 266; an
// idle share that is filled: six heads, 186 of 442..1199, a quarter hidden-kind 170 / 185 (60 such attention calls: 32 with less
// KV-kind time than that 0.61 to 0.99 of the time dealt, the other 28 0.96 to 1.09, 1.02 on average).
// A captured launch keeps its choice when it is replayed with another plan: outputs are the same bits either way.
template <int NC>
static inline bool apt_deals(const int32_t* ctx_lens, const int32_t* kinds, int B, int64_t kv_tokens, int H, int d, int chunk, uint32_t word,
                             int n_workgroups) {
    const int more = H % APT_N_QUEUES, per_queue = n_workgroups / APT_N_QUEUES;
    if (more == 0 || (more > 4 && H > APT_N_QUEUES)) return false;
    const int64_t heads = (H + APT_N_QUEUES - 1) / APT_N_QUEUES, four_rounds = 4 * (int64_t)per_queue;
    const int64_t kv = apt_kv_ns(kv_tokens, d) * n_workgroups, idle = apt_tile_ns(NC, d, NC, 1) * (heads * APT_N_QUEUES - H);   // a tile per head
    auto filled = [&](int64_t tiles) { return 5 * kv >= 4 * tiles * idle; };
    int64_t full = 0, tails = 0;
    int32_t count[NC + 1] = {0};
    for (int r = 0; r < B; ++r) {                             // (host time of every call: ends where the fewest tiles it can be are enough)
        if (kinds[r] != APT_KIND_HIDDEN) continue;
        full += ctx_lens[r] / chunk;
        if (ctx_lens[r] % chunk) ++tails, ++count[(ctx_lens[r] % chunk + APT_PACK_BLOCK - 1) / APT_PACK_BLOCK];
        const int64_t least = (full + tails) / apt_pack_tile<NC>::max_ranges;
        if (least * heads >= four_rounds && !filled(least)) return true;
    }
    const int full_blocks = chunk / APT_PACK_BLOCK;
    auto tiles_of = [&](int cap) {                            // of a head
        if (!cap) return full + tails;
        int32_t left[NC + 1];
        for (int c = 0; c <= NC; ++c) left[c] = count[c];
        int64_t tiles = full_blocks == NC ? full : 0;
        if (full_blocks < NC) left[full_blocks] += (int32_t)full;
        apt_pack_patterns<NC>(left, cap < NC ? cap : NC, [&](int32_t reps, const int32_t*) { tiles += reps; });
        return tiles;
    };
    const int cap = word & 15;
    const int64_t queues = tiles_of(cap) * heads;
    if (filled(queues / heads)) return false;
    if (queues >= four_rounds) return true;
    const bool alike = H < APT_N_QUEUES || cap == (int)(word >> (4 * more) & 15);
    if (!alike && (full + tails) * heads < four_rounds) return false;
    const int64_t tiles = tiles_of(apt_dealt_cap(word, H));
    const int64_t most = tiles * (H / APT_N_QUEUES) + tiles / APT_N_QUEUES * more + (tiles % APT_N_QUEUES < more ? tiles % APT_N_QUEUES : more);
    return (most + per_queue - 1) / per_queue < (queues + per_queue - 1) / per_queue;
}
