// Host side of the library: status strings, shape checks, the ragged work
// partitioner and the cache-map range check.  No device code here.
#include <string.h>
#include <algorithm>
#include <vector>
#include "apt_internal.h"
#include "apt_pack.h"

extern "C" const char* apt_strerror(int status) {
    switch (status) {
    case APT_OK: return "ok";
    case APT_EINVAL: return "invalid argument";
    case APT_ESHAPE: return "unsupported or inconsistent shape";
    case APT_EDTYPE: return "unsupported dtype";
    case APT_EWORKSPACE: return "buffer too small";
    case APT_EHIP: return "HIP runtime error";
    case APT_ERANGE: return "value out of range";
    case APT_EFULL: return "not enough unused cache blocks";
    default: return "unknown status";
    }
}

extern "C" int apt_version(void) { return 100; }

static bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int apt_resolve(const apt_shape* in, apt_resolved* out) {
    if (!in || !out) return APT_EINVAL;
    apt_shape s = *in;
    if (s.dtype != APT_F32 && s.dtype != APT_F16 && s.dtype != APT_BF16) return APT_EDTYPE;
    if (s.out_dtype != APT_F32 && s.out_dtype != s.dtype) return APT_EDTYPE;
    const int e = s.dtype == APT_F32 ? 4 : 2;
    if (s.d_model < 1 || s.n_heads < 1 || s.max_blocks_per_req < 1 || s.reserved != 0) return APT_ESHAPE;
    if (s.head_dim != 64 && s.head_dim != 128) return APT_ESHAPE;
    if ((int64_t)s.n_heads * s.head_dim != s.d_model) return APT_ESHAPE;
    if (!is_pow2(s.block_size) || s.block_size > 64) return APT_ESHAPE;
    // a (block, head) run of the K/V layout is read in 1 KB wave loads
    const int lanes_per_row = s.head_dim * e / 16;
    if ((s.block_size * lanes_per_row) % 64 != 0) return APT_ESHAPE;
    if (!(s.softmax_scale == s.softmax_scale)) return APT_EINVAL;

    out->hidden_auto = false;
    const bool mfma_ok = (s.dtype != APT_F32) && s.head_dim == 128 && (s.d_model % 128 == 0);
    if (s.hidden_impl == APT_HIDDEN_AUTO) s.hidden_impl = mfma_ok ? APT_HIDDEN_MFMA : APT_HIDDEN_VALU;
    if (s.hidden_impl == APT_HIDDEN_MFMA) {
        if (!mfma_ok) return APT_ESHAPE;
        // the larger tile moves fewer bytes per flop but costs more per item: it pays when an item's k loop is long
        if (s.hidden_chunk == 0)
            s.hidden_chunk = s.d_model >= APT_MFMA_LARGE_TILE_D_MODEL ? APT_MFMA_HIDDEN_CHUNK : APT_MFMA_HIDDEN_CHUNK_SMALL;
        if (s.hidden_chunk != APT_MFMA_HIDDEN_CHUNK && s.hidden_chunk != APT_MFMA_HIDDEN_CHUNK_SMALL) return APT_ESHAPE;
    } else if (s.hidden_impl == APT_HIDDEN_ABSORBED) {
        // heads: up to 8 fragments of 16 rows per operand part on the matrix cores (16-bit inputs), 4 x 10 register tiles otherwise
        const int max_heads = s.dtype == APT_F32 ? APT_ABSORBED_HEAD_GROUPS * APT_ABSORBED_HEADS_PER_THREAD : 128;
        if (s.d_model % 32 != 0 || s.n_heads > max_heads) return APT_ESHAPE;
        if (s.hidden_chunk == 0) s.hidden_chunk = APT_ABSORBED_CHUNK;
        if (s.hidden_chunk != APT_ABSORBED_CHUNK) return APT_ESHAPE;
    } else if (s.hidden_impl == APT_HIDDEN_VALU) {
        const int most = APT_RAW_MAX_HIDDEN_CHUNK(s.dtype, s.head_dim);
        out->hidden_auto = s.hidden_chunk == 0;
        if (s.hidden_chunk == 0) s.hidden_chunk = APT_RAW_AUTO_HIDDEN_CHUNK(s.dtype, s.head_dim);
        if (s.hidden_chunk < 1 || s.hidden_chunk > most) return APT_ESHAPE;
    } else {
        return APT_ESHAPE;
    }
    out->kv_auto = s.kv_chunk == 0;
    if (out->kv_auto) s.kv_chunk = APT_DEFAULT_KV_CHUNK;
    if (!apt_kv_chunk_ok(s.kv_chunk, s.block_size)) return APT_ESHAPE;
    out->s = s;
    out->elem_bytes = e;
    return APT_OK;
}

static int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }

static size_t plan_items_off(int B) {
    const size_t w = APT_PW_HEADER + APT_PA_COUNT * (size_t)B;
    return (w + 3) & ~(size_t)3;
}
// n_lists: words of the lists of the absorbed-weight path
static size_t plan_words(int B, int64_t n_items, int64_t n_lists) { return plan_items_off(B) + 4 * (size_t)n_items + (size_t)n_lists; }

extern "C" int apt_plan_max_bytes(const apt_shape* s, int B, int max_ctx, size_t* bytes) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (B < 1 || max_ctx < 1 || !bytes) return APT_EINVAL;
    const int hmin = rs.hidden_auto ? APT_RAW_MIN_HIDDEN_CHUNK(rs.s.dtype) : rs.s.hidden_chunk;
    const int cmin = hmin < rs.s.kv_chunk ? hmin : rs.s.kv_chunk;
    const int64_t n_items = (int64_t)B * rs.s.n_heads * ceil_div64(max_ctx, cmin);
    const int64_t n_lists = rs.s.hidden_impl == APT_HIDDEN_ABSORBED
        ? 2 + (int64_t)B * (ceil_div64(max_ctx, APT_ABSORBED_TILE) + ceil_div64(max_ctx, APT_ABSORBED_CHUNK)) : 0;
    *bytes = plan_words(B, n_items, n_lists) * 4;
    return APT_OK;
}

extern "C" int apt_workspace_bytes(const apt_shape* s, int max_batch, int max_ctx, size_t* dev_bytes, size_t* host_bytes) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (max_batch < 1 || max_ctx < 1 || (!dev_bytes && !host_bytes)) return APT_EINVAL;
    if ((int64_t)max_ctx > (int64_t)rs.s.max_blocks_per_req * rs.s.block_size) return APT_ERANGE;
    // every workspace section grows with each of these counts, so the layout of their separate maxima bounds
    // the layout of any batch: ranges are most numerous when every request is of the kind with the shorter
    // chunk; the sections of the absorbed-weight path are largest when every request is hidden-kind
    const int cmin = rs.s.hidden_chunk < rs.s.kv_chunk ? rs.s.hidden_chunk : rs.s.kv_chunk;
    int64_t n_partials = (int64_t)max_batch * ceil_div64(max_ctx, cmin);
    if (rs.hidden_auto) {
        // a range below the longest is chosen only while twice its length gives fewer than APT_RAW_ITEMS_TARGET
        // hidden-kind items, so it gives at most twice as many ranges as that; the KV-kind requests come on top
        const int64_t few = 2 * ((int64_t)(APT_RAW_ITEMS_TARGET - 1) / rs.s.n_heads) +
                            (int64_t)max_batch * ceil_div64(max_ctx, rs.s.kv_chunk);
        if (few > n_partials) n_partials = few;
    }
    const int64_t hid_chunks = (int64_t)max_batch * ceil_div64(max_ctx, rs.s.hidden_chunk);
    if (n_partials * (int64_t)rs.s.n_heads > 0x7fffffff || (int64_t)max_batch * max_ctx > 0x7fffffff) return APT_ERANGE;
    if (dev_bytes)
        *dev_bytes = (size_t)apt_ws_sections(n_partials, rs.s.n_heads, rs.s.head_dim, rs.s.hidden_impl, max_batch,
                                             (int64_t)max_batch * max_ctx, hid_chunks, rs.s.d_model, rs.s.dtype).total;
    if (host_bytes) return apt_plan_max_bytes(s, max_batch, max_ctx, host_bytes);
    return APT_OK;
}

// Shared tiles of the projection kernel (apt_pack.h): the cap of a head queue (0: a tile per range), when its last workgroup ends, and
// the time of all its tiles, ns.
struct QueueTiles { int cap; int64_t last, total; };

static constexpr int64_t kPatternsNs = 2500;               // what a workgroup's table of patterns takes

// Tiles of a head queue, dealt to its workgroups in rounds, every second one backwards.  Runs of equal tiles are added as differences
// between neighbouring workgroups, at most three to a run, so the time does not grow with the tiles.
struct Deal {
    static constexpr int kWorkgroups = 32;                 // per queue, on 256 compute units
    int64_t step[kWorkgroups + 1] = {0}, all = 0, total = 0;
    int at = 0;                                            // place in the current pair of rounds
    void add(int64_t ns, int64_t tiles) {
        all += tiles / (2 * kWorkgroups) * 2 * ns;         // two rounds give every workgroup two tiles, wherever they begin
        total += ns * tiles;
        for (int left = (int)(tiles % (2 * kWorkgroups)); left > 0;) {
            const int n = std::min(left, kWorkgroups - at % kWorkgroups);
            const int first = at < kWorkgroups ? at : 2 * kWorkgroups - at - n;
            step[first] += ns;
            step[first + n] -= ns;
            at = (at + n) % (2 * kWorkgroups);
            left -= n;
        }
    }
    QueueTiles result(int cap) const {
        int64_t most = 0, load = 0;
        for (int i = 0; i < kWorkgroups; ++i) most = std::max(most, load += step[i]);
        const int64_t begin = cap ? kPatternsNs : 0;
        return {cap, begin + all + most, begin * kWorkgroups + total};
    }
};

// The queues of a plan: one or two numbers of heads, the larger first, and how many queues have each.
struct HeadQueues { int n; int64_t heads[2], queues[2]; };

// When a launch ends, in 256ths of a ns: with the last workgroup of a queue, or with all its work shared evenly (the KV-kind items,
// kv ns, go to whoever is free); then the work itself.
struct LaunchTiles {
    int64_t end = INT64_MAX, total = INT64_MAX;
    int cap[2] = {0, 0};
    bool operator<(const LaunchTiles& o) const { return end < o.end || (end == o.end && total < o.total); }
};

// The caps with which a launch on tiles of NC blocks ends first.  full: ranges of full_blocks blocks, the longest; count[c]: shorter
// ranges of c blocks.  Up to one tile per workgroup of a queue nothing is shared: a fuller tile only takes longer.  Full ranges shorter
// than the tile share tiles as the others do (no cap 0).  75 batches, 3 to 72 heads, 3 to 193 requests of up to 2048 tokens, every cap
// timed: the choice took 0.6 % longer than the best one on average, 5 % at most; cost taken as proportional to d_model, without a
// fixed part, 1.9 %, and up to 20 % where d_model is small (4 heads, 64 requests, attention call: a tile per range 60.9 us, its choice 73.8).
template <int NC>
static LaunchTiles shared_tiles(int d, int64_t full, int full_blocks, const int32_t* count, const HeadQueues& q, int64_t kv) {
    const bool whole = full_blocks == NC;                  // a full range is a tile of its own
    QueueTiles option[2][NC];
    int n_options[2] = {0, 0};
    bool share[2] = {true, true};
    int64_t tails = 0;
    for (int c = 1; c < APT_PACK_MAX_BLOCKS + 1; ++c) tails += count[c];
    for (int i = 0; i < q.n && whole; ++i) {
        Deal deal;
        deal.add(apt_tile_ns(NC, d, NC, 1), full * q.heads[i]);
        for (int c = NC; c >= 1; --c) deal.add(apt_tile_ns(NC, d, c, 1), count[c] * q.heads[i]);
        option[i][n_options[i]++] = deal.result(0);
        share[i] = tails >= 2 && (full + tails) * q.heads[i] > Deal::kWorkgroups;
    }
    for (int k = NC; k >= (whole ? 4 : full_blocks + 1) && (share[0] || share[1]); --k) {
        int32_t left[NC + 1];
        std::copy(count, count + NC + 1, left);
        if (!whole) left[full_blocks] += (int32_t)full;
        Deal deal[2];
        for (int i = 0; i < q.n; ++i)
            if (whole) deal[i].add(apt_tile_ns(NC, d, NC, 1), full * q.heads[i]);
        apt_pack_patterns<NC>(left, k, [&](int32_t reps, const int32_t* take) {
            int blocks = 0, ranges = 0;
            for (int c = 1; c <= NC; ++c) { blocks += c * take[c]; ranges += take[c]; }
            for (int i = 0; i < q.n; ++i) deal[i].add(apt_tile_ns(NC, d, blocks, ranges), reps * q.heads[i]);
        });
        for (int i = 0; i < q.n; ++i)
            if (share[i]) option[i][n_options[i]++] = deal[i].result(k);
    }
    LaunchTiles best;
    for (int a = 0; a < n_options[0]; ++a)
        for (int b = 0; b < std::max(n_options[1], 1); ++b) {
            const QueueTiles none = {0, 0, 0}, &x = option[0][a], &y = q.n == 2 ? option[1][b] : none;
            LaunchTiles t;
            t.total = q.queues[0] * x.total + q.queues[1] * y.total;
            t.end = std::max(std::max(x.last, y.last) * APT_N_QUEUES * Deal::kWorkgroups, t.total + kv * APT_N_QUEUES * Deal::kWorkgroups);
            t.cap[0] = x.cap, t.cap[1] = y.cap;
            if (t < best) best = t;
        }
    return best;
}

// The word APT_PW_SHARED_TILES of a batch with packed weights.  Integers throughout, so that a batch has one plan whatever the compiler
// makes of sums and ties.
static uint32_t shared_tiles_word(const int32_t* ctx_lens, const uint8_t* cache_kind, int B, int H, int d, int chunk, int64_t kv_tokens) {
    int64_t full = 0;
    int32_t count[APT_PACK_MAX_BLOCKS + 1] = {0};
    for (int r = 0; r < B; ++r) {
        if (cache_kind[r] != APT_KIND_HIDDEN) continue;
        full += ctx_lens[r] / chunk;
        if (ctx_lens[r] % chunk) ++count[ceil_div64(ctx_lens[r] % chunk, APT_PACK_BLOCK)];
    }
    const int64_t kv = apt_kv_ns(kv_tokens, d);
    const int rest = H % APT_N_QUEUES;
    HeadQueues q = {1, {(H + APT_N_QUEUES - 1) / APT_N_QUEUES, H / APT_N_QUEUES}, {rest ? rest : APT_N_QUEUES, rest ? APT_N_QUEUES - rest : 0}};
    if (H > APT_N_QUEUES && rest) q.n = 2;
    LaunchTiles t;
    if (chunk == APT_MFMA_HIDDEN_CHUNK) t = shared_tiles<10>(d, full, 10, count, q, kv);
    else {
        t = shared_tiles<8>(d, full, 8, count, q, kv);
        // Ranges of 256 tokens in tiles of 320 rows, a full range beside a short one, where that saves a round: 40 heads, requests of
        // 415, 513 and 619 tokens (40 tiles a queue, then 30), attention call 176 -> 157 us.
        const LaunchTiles wide = shared_tiles<10>(d, full, 8, count, q, kv);
        if (wide < t) t = wide;
    }
    uint32_t word = 0;
    for (int x = 0; x < APT_N_QUEUES && x < H; ++x) word |= (uint32_t)t.cap[q.n == 2 && x >= rest] << (4 * x);
    return word;
}

extern "C" int apt_plan(const apt_shape* s, const int32_t* ctx_lens, const uint8_t* cache_kind, int B,
                        void* plan_host, size_t plan_bytes, apt_plan_info* info) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (!ctx_lens || !cache_kind || !plan_host || B < 1) return APT_EINVAL;
    const int H = rs.s.n_heads;
    const int64_t max_len = (int64_t)rs.s.max_blocks_per_req * rs.s.block_size;

    if (rs.hidden_auto) {
        auto hidden_items = [&](int c) {
            int64_t n = 0;
            for (int r = 0; r < B; ++r)
                if (cache_kind[r] == APT_KIND_HIDDEN && ctx_lens[r] > 0) n += ceil_div64(ctx_lens[r], c) * H;
            return n;
        };
        while (rs.s.hidden_chunk > APT_RAW_MIN_HIDDEN_CHUNK(rs.s.dtype) && hidden_items(rs.s.hidden_chunk) < APT_RAW_ITEMS_TARGET)
            rs.s.hidden_chunk /= 2;
    }

    // KV-kind range length left to the library: a short range costs an item's start-up and wind-down more often
    // per byte, a long one leaves too few items to fill the device; take the longest that still yields enough items
    if (rs.kv_auto) {
        for (int c = APT_MAX_AUTO_KV_CHUNK; c > rs.s.kv_chunk; c /= 2) {
            if (!apt_kv_chunk_ok(c, rs.s.block_size)) continue;
            int64_t kv_items = 0;
            for (int r = 0; r < B; ++r)
                if (cache_kind[r] == APT_KIND_KV && ctx_lens[r] > 0) kv_items += ceil_div64(ctx_lens[r], c) * H;
            if (kv_items >= APT_KV_ITEMS_TARGET) { rs.s.kv_chunk = c; break; }
        }
    }

    // pass 1: validate and count
    const bool absorbed = rs.s.hidden_impl == APT_HIDDEN_ABSORBED;
    int64_t n_partials = 0, n_hidden_items = 0, n_items = 0, tok = 0, htok = 0, n_hid_req = 0, n_tiles = 0;
    for (int r = 0; r < B; ++r) {
        const int n = ctx_lens[r];
        if (n < 1) return APT_EINVAL;
        if (n > max_len) return APT_ERANGE;
        if (cache_kind[r] != APT_KIND_KV && cache_kind[r] != APT_KIND_HIDDEN) return APT_EINVAL;
        const bool hid = cache_kind[r] == APT_KIND_HIDDEN;
        const int64_t sp = ceil_div64(n, hid ? rs.s.hidden_chunk : rs.s.kv_chunk);
        const int64_t per_range = (hid && absorbed) ? 1 : H;      // absorbed: one item serves all heads
        n_partials += sp;
        n_items += sp * per_range;
        if (hid) { n_hidden_items += sp * per_range; htok += n; ++n_hid_req; if (absorbed) n_tiles += ceil_div64(n, APT_ABSORBED_TILE); }
        tok += n;
    }
    if (n_items > 0x7fffffff || n_partials * (int64_t)H > 0x7fffffff || htok > 0x7fffffff) return APT_ERANGE;
    // absorbed-weight path: ranges per unit of the weighted sums (fp32 inputs: one)
    int group = 1;
    int64_t n_units = n_hidden_items;
    if (absorbed && rs.s.dtype != APT_F32) {
        for (int g = APT_ABSORBED_MAX_GROUP; g > 1; g /= 2) {
            int64_t n = 0;
            for (int r = 0; r < B; ++r)
                if (cache_kind[r] == APT_KIND_HIDDEN) n += ceil_div64(ctx_lens[r], (int64_t)g * APT_ABSORBED_CHUNK);
            if (n * ceil_div64(rs.s.d_model, 512) >= APT_ABSORBED_UNITS_TARGET) { group = g; n_units = n; break; }
        }
    }
    const size_t words = plan_words(B, n_items, absorbed ? 2 + n_tiles + n_units : 0);
    if (plan_bytes < words * 4) return APT_EWORKSPACE;

    int32_t* w = (int32_t*)plan_host;
    const size_t items_off = plan_items_off(B);
    memset(w, 0, items_off * 4);
    w[APT_PW_MAGIC] = APT_PLAN_MAGIC;
    w[APT_PW_BATCH] = B;
    w[APT_PW_HEADS] = H;
    w[APT_PW_NITEMS] = (int32_t)n_items;
    w[APT_PW_NHIDDEN] = (int32_t)n_hidden_items;
    w[APT_PW_NPARTIALS] = (int32_t)n_partials;
    w[APT_PW_HCHUNK] = rs.s.hidden_chunk;
    w[APT_PW_KCHUNK] = rs.s.kv_chunk;
    w[APT_PW_HIMPL] = rs.s.hidden_impl;
    w[APT_PW_ITEMS_OFF] = (int32_t)items_off;
    w[APT_PW_TOK_LO] = (int32_t)(tok & 0xffffffff);
    w[APT_PW_TOK_HI] = (int32_t)(tok >> 32);
    w[APT_PW_HTOK_LO] = (int32_t)(htok & 0xffffffff);
    w[APT_PW_HTOK_HI] = (int32_t)(htok >> 32);
    w[APT_PW_HEAD_DIM] = rs.s.head_dim;
    w[APT_PW_WORDS] = (int32_t)words;
    w[APT_PW_D_MODEL] = rs.s.d_model;
    w[APT_PW_BLOCK_SIZE] = rs.s.block_size;
    w[APT_PW_MAX_BLOCKS] = rs.s.max_blocks_per_req;
    w[APT_PW_DTYPE] = rs.s.dtype;
    w[APT_PW_NHIDREQ] = (int32_t)n_hid_req;
    w[APT_PW_TILES_OFF] = absorbed ? (int32_t)(items_off + 4 * (size_t)n_items) : 0;

    int32_t* split_count = w + APT_PW_HEADER + APT_PA_SPLIT_COUNT * B;
    int32_t* ws_offset = w + APT_PW_HEADER + APT_PA_WS_OFFSET * B;
    int32_t* kind = w + APT_PW_HEADER + APT_PA_KIND * B;
    int32_t* hid_index = w + APT_PW_HEADER + APT_PA_HID_INDEX * B;
    int32_t* hid_tok_off = w + APT_PW_HEADER + APT_PA_HID_TOK_OFF * B;
    int32_t* hid_chunk_off = w + APT_PW_HEADER + APT_PA_HID_CHUNK_OFF * B;
    int32_t* hid_req = w + APT_PW_HEADER + APT_PA_HID_REQ * B;
    int32_t* ctx_len = w + APT_PW_HEADER + APT_PA_CTX_LEN * B;
    for (int r = 0; r < B; ++r) hid_req[r] = -1;
    int32_t run = 0, hi = 0, ht = 0, hc = 0;
    for (int r = 0; r < B; ++r) {
        const bool hid = cache_kind[r] == APT_KIND_HIDDEN;
        split_count[r] = (int32_t)ceil_div64(ctx_lens[r], hid ? rs.s.hidden_chunk : rs.s.kv_chunk);
        ws_offset[r] = run;
        run += split_count[r];
        kind[r] = cache_kind[r];
        ctx_len[r] = ctx_lens[r];
        if (hid) hid_req[hi] = r;
        hid_index[r] = hid ? hi : -1;
        hid_tok_off[r] = hid ? ht : -1;
        hid_chunk_off[r] = hid ? hc : -1;
        if (hid) { ++hi; ht += ctx_lens[r]; hc += split_count[r]; }
    }
    // pass 2: items.  Hidden kind first, in APT_N_QUEUES queues by head % 8; in a queue the
    // full ranges come first (request, range, head order), then the last, shorter ranges by
    // decreasing length.  Then the KV kind by decreasing range length.
    int32_t* it = w + items_off;
    int32_t* const it0 = it;
    // Requests with a shorter last range, by its length: the same for every queue of a kind.  apt_plan, us, sorted for every queue /
    // once: 64 requests, 40 heads 34.3 / 19.5, 256 requests, 71 heads 149.9 / 75.0.
    std::vector<int32_t> tails;
    auto order_tails = [&](uint8_t want, int c) {
        tails.clear();
        for (int r = 0; r < B; ++r)
            if (cache_kind[r] == want && ctx_lens[r] % c != 0) tails.push_back(r);
        std::stable_sort(tails.begin(), tails.end(),
                         [&](int32_t a, int32_t b) { return ctx_lens[a] % c > ctx_lens[b] % c; });
    };
    auto emit_kind = [&](uint8_t want, int c, int h_first, int h_step) {
        for (int r = 0; r < B; ++r) {       // full ranges
            if (cache_kind[r] != want) continue;
            const int nfull = ctx_lens[r] / c;
            for (int sp = 0; sp < nfull; ++sp)
                for (int h = h_first; h < H; h += h_step) {
                    it[0] = r; it[1] = h; it[2] = sp * c; it[3] = sp * c + c;
                    it += 4;
                }
        }
        for (int32_t r : tails) {
            const int t0 = (ctx_lens[r] / c) * c;
            for (int h = h_first; h < H; h += h_step) {
                it[0] = r; it[1] = h; it[2] = t0; it[3] = ctx_lens[r];
                it += 4;
            }
        }
    };
    if (!absorbed) order_tails(APT_KIND_HIDDEN, rs.s.hidden_chunk);
    for (int x = 0; x < APT_N_QUEUES; ++x) {
        w[APT_PW_QUEUE0 + x] = (int32_t)((it - it0) / 4);
        if (!absorbed) {
            emit_kind(APT_KIND_HIDDEN, rs.s.hidden_chunk, x, APT_N_QUEUES);
        } else if (x == 0) {           // one item per range, by request and range, all in queue 0
            for (int r = 0; r < B; ++r) {
                if (cache_kind[r] != APT_KIND_HIDDEN) continue;
                for (int sp = 0; sp < split_count[r]; ++sp) {
                    const int t0 = sp * rs.s.hidden_chunk;
                    it[0] = r; it[1] = 0; it[2] = t0;
                    it[3] = t0 + rs.s.hidden_chunk < ctx_lens[r] ? t0 + rs.s.hidden_chunk : ctx_lens[r];
                    it += 4;
                }
            }
        }
    }
    w[APT_PW_QUEUE0 + APT_N_QUEUES] = (int32_t)((it - it0) / 4);
    if (rs.s.hidden_impl == APT_HIDDEN_MFMA && n_hidden_items > 0)
        w[APT_PW_SHARED_TILES] = (int32_t)shared_tiles_word(ctx_lens, cache_kind, B, H, rs.s.d_model, rs.s.hidden_chunk, tok - htok);
    order_tails(APT_KIND_KV, rs.s.kv_chunk);
    emit_kind(APT_KIND_KV, rs.s.kv_chunk, 0, 1);
    // absorbed-weight path: the 256-token tiles of the hidden-kind ranges in their order, 2 * item + half; then the units
    // (their first ranges), longest first
    if (absorbed) {
        int32_t* at = w + w[APT_PW_TILES_OFF];
        *at++ = (int32_t)n_tiles;
        *at++ = group;
        for (int32_t i = 0; i < (int32_t)n_hidden_items; ++i)
            for (int half = 0; half * APT_ABSORBED_TILE < it0[4 * i + 3] - it0[4 * i + 2]; ++half) *at++ = 2 * i + half;
        int32_t* const units = at;
        const int unit_tokens = group * APT_ABSORBED_CHUNK;
        for (int32_t i = 0; i < (int32_t)n_hidden_items; ++i)
            if (it0[4 * i + 2] % unit_tokens == 0) *at++ = i;
        std::stable_sort(units, at, [&](int32_t a, int32_t b) {
            return std::min(ctx_lens[it0[4 * a]] - it0[4 * a + 2], unit_tokens) > std::min(ctx_lens[it0[4 * b]] - it0[4 * b + 2], unit_tokens);
        });
    }
    if (info) return apt_plan_get_info(plan_host, info);
    return APT_OK;
}

extern "C" int apt_plan_get_info(const void* plan_host, apt_plan_info* info) {
    if (!plan_host || !info) return APT_EINVAL;
    const int32_t* w = (const int32_t*)plan_host;
    if (w[APT_PW_MAGIC] != APT_PLAN_MAGIC) return APT_EINVAL;
    memset(info, 0, sizeof(*info));
    info->batch = w[APT_PW_BATCH];
    info->n_items = w[APT_PW_NITEMS];
    info->n_hidden_items = w[APT_PW_NHIDDEN];
    info->n_partials = w[APT_PW_NPARTIALS];
    info->hidden_chunk = w[APT_PW_HCHUNK];
    info->kv_chunk = w[APT_PW_KCHUNK];
    info->hidden_impl = w[APT_PW_HIMPL];
    info->total_tokens = ((int64_t)w[APT_PW_TOK_HI] << 32) | (uint32_t)w[APT_PW_TOK_LO];
    info->hidden_tokens = ((int64_t)w[APT_PW_HTOK_HI] << 32) | (uint32_t)w[APT_PW_HTOK_LO];
    info->plan_bytes = (uint64_t)(uint32_t)w[APT_PW_WORDS] * 4u;
    info->workspace_bytes = apt_ws_sections(w[APT_PW_NPARTIALS], w[APT_PW_HEADS], w[APT_PW_HEAD_DIM], w[APT_PW_HIMPL],
                                            w[APT_PW_NHIDREQ], info->hidden_tokens, w[APT_PW_NHIDDEN], w[APT_PW_D_MODEL],
                                            w[APT_PW_DTYPE]).total;
    return APT_OK;
}

extern "C" int apt_validate_host(const apt_shape* s, const int32_t* ctx_lens, const uint8_t* cache_kind,
                                 const int32_t* block_tables, int B, int64_t n_pool_blocks) {
    apt_resolved rs;
    int rc = apt_resolve(s, &rs);
    if (rc) return rc;
    if (!ctx_lens || !cache_kind || !block_tables || B < 1 || n_pool_blocks < 1) return APT_EINVAL;
    const int mb = rs.s.max_blocks_per_req, bs = rs.s.block_size;
    // the MFMA kernel addresses hidden rows by 32-bit offsets in 16-byte units
    if (rs.s.hidden_impl == APT_HIDDEN_MFMA &&
        (uint64_t)n_pool_blocks * (uint64_t)bs * (uint64_t)rs.s.d_model * (uint64_t)rs.elem_bytes > ((uint64_t)1 << 36))
        return APT_ERANGE;
    for (int r = 0; r < B; ++r) {
        const int n = ctx_lens[r];
        if (n < 1) return APT_EINVAL;
        if (cache_kind[r] != APT_KIND_KV && cache_kind[r] != APT_KIND_HIDDEN) return APT_EINVAL;
        const int nb = (n + bs - 1) / bs;
        if (nb > mb) return APT_ERANGE;
        const int rows = cache_kind[r] == APT_KIND_KV ? 2 : 1;
        for (int row = 0; row < rows; ++row)
            for (int i = 0; i < nb; ++i) {
                const int32_t b = block_tables[((int64_t)r * 2 + row) * mb + i];
                if (b < 0 || b >= n_pool_blocks) return APT_ERANGE;
            }
    }
    return APT_OK;
}
