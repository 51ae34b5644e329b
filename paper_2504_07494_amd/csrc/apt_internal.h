// Internal definitions shared by the host planner and the kernel launchers.
#pragma once
#include <stdint.h>
#include "apt_hybrid.h"

// Plan blob: int32 words.
enum {
    APT_PW_MAGIC = 0,
    APT_PW_BATCH = 1,
    APT_PW_HEADS = 2,
    APT_PW_NITEMS = 3,
    APT_PW_NHIDDEN = 4,
    APT_PW_NPARTIALS = 5,
    APT_PW_HCHUNK = 6,
    APT_PW_KCHUNK = 7,
    APT_PW_HIMPL = 8,
    APT_PW_ITEMS_OFF = 9,   // word offset of items[]
    APT_PW_TOK_LO = 10,
    APT_PW_TOK_HI = 11,
    APT_PW_HTOK_LO = 12,
    APT_PW_HTOK_HI = 13,
    APT_PW_HEAD_DIM = 14,
    APT_PW_WORDS = 15,      // total words of the blob
    APT_PW_QUEUE0 = 16,     // 9 words: start of each hidden-kind queue (in items), then the end; KV-kind requests alone: 0, in the
                            // device copy the first 8 count the items done of a launch that merges (0 between launches)
    APT_PW_KV_TICKET = 25,  // device copy only: next KV-kind item to hand out, or the items done of a launch that merges (0 between launches)
    APT_PW_D_MODEL = 26,    // the shape the plan was made for
    APT_PW_BLOCK_SIZE = 27,
    APT_PW_MAX_BLOCKS = 28,
    APT_PW_DTYPE = 29,
    APT_PW_NHIDREQ = 30,    // number of hidden-kind requests
    APT_PW_TILES_OFF = 31,  // absorbed-weight path: word offset of its lists (tiles, ranges per unit, tile words, unit
                            // words up to the end of the blob), else 0
    APT_PW_SHARED_TILES = 31, // packed-weight path: blocks that a tile shared by short ranges may fill, four bits per
                            // queue from bit 0 on (apt_pack.h); 0: no shared tiles
    APT_PW_HEADER = 32
};
#define APT_N_QUEUES 8
#define APT_PLAN_MAGIC 0x41505431

// Tokens per work item.
#define APT_DEFAULT_KV_CHUNK 512         // shortest range the planner chooses by itself; it doubles it (to at most
#define APT_MAX_AUTO_KV_CHUNK 2048       // this) while the batch still yields APT_KV_ITEMS_TARGET KV-kind items:
#define APT_KV_ITEMS_TARGET 2048         // two per workgroup slot of a 256-CU device at four workgroups per CU
#define APT_MFMA_HIDDEN_CHUNK 320       // token rows of the MFMA kernel's tile: 320 ...
#define APT_MFMA_HIDDEN_CHUNK_SMALL 256 // ... or 256 (default for d_model < APT_MFMA_LARGE_TILE_D_MODEL)
#define APT_MFMA_LARGE_TILE_D_MODEL 8192
// Raw weights, 16-bit inputs: the tile of the matrix kernel is 256 tokens (head_dim 64) or 128 (head_dim 128).  Left
// open, the planner halves the range (to at least 64) while the batch yields fewer hidden-kind items than this, a bit
// under one per CU: with fewer the chip idles, with more the longer range wins because it reads the weights less often.
// Attention call at d_model 2048 (head_dim 64), us with ranges of 64 / 128 / 256 tokens: 1 request of 300 tokens 23 / 27 / 40
// (160 / 96 / 64 items), 2 requests 49 / 34 / 41 (608 / 320 / 192), 4 requests 71 / 62 / 48 (1152 / 608 / 352),
// 16 requests 167 / 131 / 125; at d_model 768, 4 requests 21 / 18 / 21 (432 / 228 / 132 items).
// fp32 inputs: 32 or 16 tokens by the same rule.  us with ranges of 16 / 32 / 64: d_model 256, 4 requests 12.6 / 12.8 / 16.7
// (108 / 60 / 32 items); d_model 1024, 4 requests 67 / 59 / 88 (1024 / 512 / 272), 64 requests 540 / 469 / 496; d_model 512,
// 12 requests 44 / 38 / 49 (1000 / 520 / 288).  Very few heads would gain from longer ranges, whose merge is shorter (1 head of
// 64, 8 requests, 2661 tokens: 19 / 14.5 / 13; 2 heads, fp16, 16 requests, 64 / 128 / 256: 13.3 / 11.3 / 11.1): not in the rule.
#define APT_RAW_AUTO_HIDDEN_CHUNK(dtype, hd) ((dtype) == APT_F32 ? 32 : 16384 / (hd))
#define APT_RAW_MAX_HIDDEN_CHUNK(dtype, hd) ((dtype) == APT_F32 ? 64 : 16384 / (hd))
#define APT_RAW_MIN_HIDDEN_CHUNK(dtype) ((dtype) == APT_F32 ? 16 : 64)
#define APT_RAW_ITEMS_TARGET 200
#define APT_RAW_PLAN_HIDDEN_CHUNK 32     // a call that leaves the range open also takes a plan of this length (any length runs)
#define APT_KV_MAX_PAGES_PER_WAVE 64
#define APT_ABSORBED_HEAD_GROUPS 4       // absorbed-weight kernels: threads of a workgroup = 64 x 4 (token or column
#define APT_ABSORBED_HEADS_PER_THREAD 10 // group, head group), 8 tokens/columns x 10 heads per thread
#define APT_ABSORBED_CHUNK 512           // = 64 groups x 8 tokens
#define APT_ABSORBED_TILE 256            // tokens of a tile of the 16-bit score kernel: one or two tiles per range
// Weighted sums of the 16-bit path: a unit is 1, 2 or 4 ranges of a request, the most with which the batch still gives this
// many units of 512 columns (three per CU, so that the longest do not decide when the kernel ends).  Longer units write and
// read again fewer fp32 sums: 72 heads, 96 requests, 102 k tokens: 255 MB with 4 ranges per unit, 637 MB with 1.
#define APT_ABSORBED_MAX_GROUP 4
#define APT_ABSORBED_UNITS_TARGET 768
#define APT_ABSORBED_OUT_ROWS 256        // d_model rows per partial of the output projection

// Absorbed-weight path, 16-bit inputs: which of its two passes over the hidden rows X reads them past the caches.  qt_bytes: the absorbed
// queries QT, written just before the scores read them.
// The sums: where X is more than half of the L2s (32 MB together); they are its last reader.  Attention call in a graph, us, cached / past:
// 17 heads, fp16, 300 tokens 32.0 / 34.2, 1.3 k (X 5 MB) 34.0 / 36.2; 24 heads, 8 requests of 100..900 (20 MB) 47.8 / 47.2; 40 heads, 60 of
// 400..800 (377 MB) 273 / 258; 72 heads, bf16, 96 of 64..2048 (1.9 GB) 1325 / 1297.
// The scores: X read through the caches stays in the memory-side one (256 MB) for the sums, as far as it has room, and takes that room
// from QT.  So past it where QT is large, by itself and beside X, and both do not fit, and where little of X would be left.
// cached / past (X, QT in MB):
//     40 heads, fp16, 32 requests of 100..500 (102, 31)    109 / 114       128..2048 (375, 31)                     237 / 246
//     24 heads, fp16, 150 of 30..400 (206, 58)             172 / 177       bf16 (206, 88)                          191 / 195
//     20 heads, bf16, 190 of 50..250 (148, 93)             157 / 161       40 heads, bf16, 100 of 100..600 (354, 147) 315 / 309
//     62 heads, 77 of 200, fp16 (244, 156)                 311 / 305       bf16 (244, 234)                         391 / 360
//     48 heads, 150 of 20..120, fp16 (133, 176)            320 / 307       bf16 (133, 265)                         385 / 373
//     56 heads, bf16, 60 of 300..900 (513, 165)            428 / 410       32 heads, 100 of 300..900, bf16 (497, 78) 319 / 313
//     17 heads, bf16, 150 of 300..1500 (597, 62)           329 / 321       72 heads, bf16, 48 of 96 of 64..2048 (900, 212) 968 / 953
//     16 heads, bf16, 180 of 400..2000 (906, 70)           454 / 444       72 heads, bf16, 96 of 64..2048 (1903, 424)  1297 / 1300
// Beyond 448 MB fp16 goes the way of bf16, though it is as often faster through the caches (72 heads, 96 of 64..2048 1129 / 1150, 24 heads,
// 150 of 300..900 311 / 320, 32 heads, 100 of 300..900 292 / 287, 180 of 100..600 360 / 356).
#define APT_AB_PAST_SCORES 1
#define APT_AB_PAST_SUMS 2
static inline int apt_absorbed_past(int64_t qt_bytes, int64_t x_bytes) {
    const int64_t mb = 1 << 20;
    const bool scores = (qt_bytes > 96 * mb && 4 * qt_bytes > x_bytes && qt_bytes + x_bytes > 256 * mb) || x_bytes > 448 * mb;
    return (scores ? APT_AB_PAST_SCORES : 0) | (x_bytes > 16 * mb ? APT_AB_PAST_SUMS : 0);
}

// per-request arrays of the plan blob, each B words, starting at APT_PW_HEADER
enum {
    APT_PA_SPLIT_COUNT = 0,    // ranges of the request
    APT_PA_WS_OFFSET = 1,      // its first partial
    APT_PA_KIND = 2,           // APT_KIND_*
    APT_PA_CTX_LEN = 3,        // cached tokens
    APT_PA_HID_INDEX = 4,      // hidden-kind requests only (-1 otherwise): index among them,
    APT_PA_HID_TOK_OFF = 5,    //   tokens of the hidden-kind requests before it,
    APT_PA_HID_CHUNK_OFF = 6,  //   ranges of the hidden-kind requests before it
    APT_PA_HID_REQ = 7,        // entry i: the request that is hidden-kind request i (-1 past their number)
    APT_PA_COUNT = 8
};

struct apt_resolved {
    apt_shape s;        // chunks and hidden_impl filled in
    int elem_bytes;
    bool hidden_auto;   // raw weights and hidden_chunk was 0: s.hidden_chunk holds the longest range, the
                        // planner may choose a shorter one, not below APT_RAW_MIN_HIDDEN_CHUNK
    bool kv_auto;       // kv_chunk was 0: s.kv_chunk holds the shortest range, the planner may choose a longer one
};

// Whether c tokens can be a KV-kind range of this shape (whole blocks, within the item kernel's page loop).
static inline bool apt_kv_chunk_ok(int c, int block_size) {
    return c >= block_size && c % block_size == 0 && c / block_size <= 4 * APT_KV_MAX_PAGES_PER_WAVE;
}

// Validates a shape and fills the defaults.  Returns an apt_status.
int apt_resolve(const apt_shape* in, apt_resolved* out);

static inline uint64_t apt_align256(uint64_t v) { return (v + 255u) & ~(uint64_t)255u; }

// Workspace sections.  Always: the partials (per slot head_dim floats of un-normalised output, then (m, l)).
// Absorbed-weight hidden path in addition (fp32): absorbed queries QT [n_hid_req][H][d] (16-bit inputs: 16-bit parts,
// [n_hid_req][d / KT][parts * R][KT] with R heads rounded up to whole fragments of 16 and k-tiles of KT = 32 or 64), score
// offsets CB [n_hid_req][H], score partials S [slices][H][hidden_tokens] (slice 0 then holds the scores), statistics
// ML [n_hid_req][H] (m, l), the weighted sums YP [n_hidden_chunks][H][d] (16-bit inputs: one per unit, at its first range),
// the output partials OP [slices][n_hid_req][H][hd], and (16-bit inputs) the softmax weights PP as 16-bit parts
// [16 n_hidden_chunks][parts * R][32].  The sizes are bounds that hold for every plan of the shape: S for ceil(d / 512) slices,
// OP for ceil(d / 256), QT and PP for heads padded to a multiple of 64, YP for a sum per range.
struct apt_ws_layout {
    uint64_t acc, ml, qt, cb, s, stat, yp, op, pp, total;
};
static inline apt_ws_layout apt_ws_sections(int64_t n_partials, int H, int hd, int himpl, int64_t n_hid_req,
                                            int64_t hidden_tokens, int64_t n_hid_chunks, int d, int dtype) {
    apt_ws_layout L;
    const uint64_t slots = (uint64_t)n_partials * (uint64_t)H;
    L.acc = 0;
    L.ml = slots * (uint64_t)hd * 4u;
    uint64_t end = L.ml + slots * 8u;
    L.qt = L.cb = L.s = L.stat = L.yp = L.op = L.pp = 0;
    if (himpl == APT_HIDDEN_ABSORBED) {
        const uint64_t ks = (uint64_t)(d + APT_ABSORBED_CHUNK - 1) / APT_ABSORBED_CHUNK;
        L.qt = apt_align256(end);
        // 16-bit inputs: QT is kept as 16-bit parts (2 for fp16, 3 for bf16), here of the heads padded to a multiple of 64
        const uint64_t head_groups = (uint64_t)(H + 63) / 64;
        const uint64_t qt_per_elem = dtype == APT_F32 ? (uint64_t)H * 4u : head_groups * (dtype == APT_F16 ? 256u : 384u);
        L.cb = apt_align256(L.qt + (uint64_t)n_hid_req * d * qt_per_elem);
        L.s = apt_align256(L.cb + (uint64_t)n_hid_req * H * 4u);
        L.stat = apt_align256(L.s + ks * (uint64_t)hidden_tokens * H * 4u);
        L.yp = apt_align256(L.stat + (uint64_t)n_hid_req * H * 8u);
        L.op = apt_align256(L.yp + (uint64_t)n_hid_chunks * H * d * 4u);
        const uint64_t os = (uint64_t)(d + APT_ABSORBED_OUT_ROWS - 1) / APT_ABSORBED_OUT_ROWS;
        L.pp = apt_align256(L.op + os * (uint64_t)n_hid_req * H * hd * 4u);
        // 16-bit inputs: the softmax weights as 16-bit parts, 16 tiles of 32 tokens per range
        end = L.pp + (dtype == APT_F32 ? 0u : (uint64_t)n_hid_chunks * 16u * 32u * qt_per_elem);
    }
    L.total = end;
    return L;
}

// Whether the last workgroups of the item kernel merge the partials (merge_by_last): KV-kind requests alone, a range to a workgroup of 1024
// threads (of 256 where the caller fixes kv_chunk), or raw weights, 256 threads.  Four channels a thread, their ranges asked for at once
// (256 threads: in two rounds), no more partials than when one workgroup merged them all, and not so many workgroups that they wait for
// each other at a ticket, 10 ns each.  Up to there the call takes the GPU no longer than with a merge kernel, and the host a launch less.
// Attention call in a graph, us, a kernel of its own / by the last workgroups, and in brackets steps of one layer back to back, planned,
// copied and launched from Python:
//     KV-kind, fp16, 1024 threads, heads of 128: 8 heads, 1100 tokens (24 ranges) 11.4 / 10.5, 24 heads, 2048 (96) 12.9 / 11.8, 40 heads, 1237
//     (120) 12.3 / 11.7 (18.5 / 15.8), 20 heads, 2 of 900..1000 (80) 12.3 / 11.1, 10 heads, 6 of 900 (120) 12.4 / 11.8; beyond: 64 heads,
//     1300 (192) 13.6 / 13.3, 20 heads, 3 of 2048 (240) 16.0 / 16.5, 8 heads, 2 of 2300 in five ranges each 12.7 / 12.7, 12 heads, 4096
//     in eight 12.4 / 13.2; heads of 64: 24 heads, 2048 (96) 9.5 / 8.9, 40 heads, 2048 (160) 10.0 / 10.1; beyond: 30 heads, 2 of 2000
//     (240) 11.1 / 11.9
//     256 threads: fp32, 4 heads of 64, 4 of 16..128 tokens 10.2 / 9.3 (18.6 / 15.5), fp16, 16 heads of 64, 250 tokens 13.6 / 13.1; beyond,
//     one workgroup for all: 8 heads, 6 of 60 (more than four channels a thread) 10.4 / 11.9, 8 heads, 4 of 200 (128 ranges) 10.7 / 12.0, one
//     head, 2048 tokens in 64 ranges 14.7 / 15.6
#define APT_MERGE_GROUPS 8               // KV-kind requests alone: parts of the heads, each merged by a workgroup
#define APT_MERGE_RANGES_MANY 4          // ranges that a thread of 1024 asks for at once
#define APT_MERGE_RANGES 8               // and one of 256
static inline bool apt_items_merge(bool kv_alone, int threads, int64_t batch, int heads, int head_dim, int64_t n_items, int most_ranges) {
    const int part = kv_alone ? (heads + APT_MERGE_GROUPS - 1) / APT_MERGE_GROUPS : heads;
    return batch * part * head_dim <= 4 * threads && n_items <= 160 && n_items * head_dim <= 16 * threads &&
           most_ranges <= (threads == 1024 ? APT_MERGE_RANGES_MANY : 2 * APT_MERGE_RANGES);
}

// Hidden-kind item of place g of a one-workgroup-per-item launch, -1 for none; queue = the nine APT_PW_QUEUE0 words of the
// plan, share = ceil(n_hidden_items / 8), places 0 .. 8 * share - 1.  Place g runs on XCD g % 8, which takes the first share
// items of queue g % 8, so that an XCD's workgroups share the weights of few heads in its L2.  What a queue holds beyond a
// share (head counts that are no multiple of eight) goes to the XCDs whose queues are shorter: every XCD gets the same number
// of items, and the launch has at most seven workgroups more than items.  Against one place per item of the longest queue, and
// empty workgroups in the shorter ones (more threads than a launch can have from 2.1 million items of one head on), 64-wide
// heads: 1 head, 256 requests of 1024..2048 tokens, fp32 1220 -> 213 us, fp16 148 -> 33; 64 requests of 256..1024 tokens,
// fp16: 4 heads 40.6 -> 28.3, 9 heads 113 -> 85, 12 heads 155 -> 131, 17 heads 280 -> 241; 8, 16 and 24 heads the same.
#ifdef __HIPCC__
__host__ __device__
#endif
static inline int apt_dealt_item(const int32_t* queue, int share, int g) {
    const int x = g & 7, len = queue[x + 1] - queue[x];
    int k = (g >> 3) - len;
    if (k < 0) return queue[x] + (g >> 3);
    // a spare place, the k-th of all: it gets the k-th of the items beyond a share
    for (int y = 0; y < x; ++y) {
        const int spare = share - (queue[y + 1] - queue[y]);
        if (spare > 0) k += spare;
    }
    for (int y = 0; y < APT_N_QUEUES; ++y) {
        const int over = queue[y + 1] - queue[y] - share;
        if (over > 0 && k < over) return queue[y] + share + k;
        if (over > 0) k -= over;
    }
    return -1;
}
