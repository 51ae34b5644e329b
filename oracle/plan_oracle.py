"""Plain reference of the ragged work partition.  TEST INFRASTRUCTURE ONLY.

The decode attention step over a batch of requests with two cache kinds
(Section 4.2: the cache type is chosen per request; Section 4.3: one cache map
per request) is cut into independent work items, one per (request, head, token
range).  The paper does not prescribe an intra-kernel partition; the rule below
is this build's, stated in full so that the library's planner can be checked
against it bit for bit:

* a request of n tokens is cut into ceil(n / C) ranges [s*C, min(n, (s+1)*C)),
  with C = hidden_chunk for hidden-kind and C = kv_chunk for KV-kind requests;
* split_count[r] = number of ranges of request r; ws_offset[r] = sum of
  split_count over requests before r (request order);
* the partial result of (request r, range s, head h) is stored in slot
  (ws_offset[r] + s) * H + h;
* an item is (r, h, t0, t1).  Items are listed hidden-kind first, then KV-kind.
* hidden-kind items are grouped into N_QUEUES = 8 queues, queue x holding the items
  whose head h has h % 8 == x; the queues are concatenated in order x = 0..7 and
  queue_offset[x] (9 entries) is the position of queue x's first item.  Inside a
  queue: first the items whose range is a full hidden_chunk, ordered by request,
  range, head; then the shorter (last) ranges, ordered by decreasing length, ties by
  request, then head.
* KV-kind items are ordered by decreasing length of their range, ties by request,
  range, head.
* when the caller leaves kv_chunk open, it is the longest of 2048, 1024 and 512 tokens
  that consists of whole blocks, at most 256 of them, and with which the KV-kind
  requests of the batch still make at least 2048 items (ranges x heads); 512 if neither
  of the longer ones does (auto_kv_chunk below).
* when the caller leaves hidden_chunk open and K and V are projected from the raw weights, it is the longest of the lengths
  below with which the hidden-kind requests of the batch make at least 200 items (ranges x heads), the shortest if none does:
  fp32 inputs 32 or 16 tokens; 16-bit inputs 256 (head_dim 64 only), 128 or 64 (auto_hidden_chunk below).
* the absorbed-weight path adds two lists (absorbed_lists below).  Tiles: every hidden-kind item is cut into tiles of 256
  tokens, one or two; a tile is the word 2 * item + (0 or 1), in item order.  Units: 1, 2 or 4 neighbouring ranges of one
  request are summed together, the most with which the batch still has 768 units x ceil(d_model / 512) column slices (fp32
  inputs, and batches that never have: 1); a unit is the word of its first item, longest unit first, ties in item order.
* with packed weights the plan's word 31 says how the shorter last ranges share tiles (shared_tiles_word below).

Block arithmetic of the cache map (Section 4.3): token j of a request lives in
its (j // block_size)-th block at slot j % block_size; a request of n tokens owns
ceil(n / block_size) blocks per cached vector type (K and V for the KV kind, the
input hidden vector for the hidden kind).
"""
import itertools

KIND_KV = 0
KIND_HIDDEN = 1
N_QUEUES = 8


def ceil_div(a, b):
    return -(-a // b)


def auto_kv_chunk(ctx_lens, cache_kind, n_heads, block_size):
    """The range length of KV-kind requests when the caller does not fix it."""
    kv_lens = [int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_KV]
    for c in (2048, 1024):
        if c % block_size or c // block_size > 256:
            continue
        if sum(ceil_div(n, c) for n in kv_lens) * n_heads >= 2048:
            return c
    return 512


def auto_hidden_chunk(ctx_lens, cache_kind, n_heads, dtype, head_dim):
    """The range length of hidden-kind requests with raw weights when the caller does not fix it."""
    hid_lens = [int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_HIDDEN]
    choices = (32, 16) if dtype == "f32" else (256, 128, 64) if head_dim == 64 else (128, 64)
    for c in choices:
        if sum(ceil_div(n, c) for n in hid_lens) * n_heads >= 200:
            return c
    return choices[-1]


def absorbed_lists(ctx_lens, cache_kind, d_model, dtype):
    """(tiles, ranges per unit, units) of the absorbed-weight path; items are its 512-token ranges by request."""
    hid = [r for r in range(len(ctx_lens)) if int(cache_kind[r]) == KIND_HIDDEN]
    ranges = [(r, t0) for r in hid for t0 in range(0, int(ctx_lens[r]), 512)]
    tiles = []
    for i, (r, t0) in enumerate(ranges):
        tiles.append(2 * i)
        if int(ctx_lens[r]) - t0 > 256:
            tiles.append(2 * i + 1)
    group = 1
    if dtype != "f32":
        for g in (2, 4):
            if sum(ceil_div(int(ctx_lens[r]), 512 * g) for r in hid) * ceil_div(d_model, 512) >= 768:
                group = g
    units = [i for i, (r, t0) in enumerate(ranges) if t0 % (512 * group) == 0]
    units.sort(key=lambda i: -min(512 * group, int(ctx_lens[ranges[i][0]]) - ranges[i][1]))
    return tiles, group, units


def tile_patterns(count, cap, blocks):
    """Which ranges share a tile of `blocks` blocks of 32 rows of which `cap` may be filled.  count[c]: ranges of c blocks.  A tile takes as
    many of the largest class as fit and are left, then of the next smaller one, and so on, at most 6 (tile of 10 blocks) or 8
    ranges; a range longer than the cap is alone.  The pattern is used as often as the ranges last.  [(tiles, {class: ranges})]."""
    left, out = dict(enumerate(count)), []
    most = 6 if blocks == 10 else 8
    while any(left[c] for c in range(1, blocks + 1)):
        take, room = {}, cap
        for c in range(blocks, 0, -1):
            t = min(room // c, most - sum(take.values()), left[c])
            if not take and left[c] and c > room:
                t = 1
            if t:
                take[c] = t
                room = max(0, room - t * c)
        tiles = min(left[c] // t for c, t in take.items())
        for c, t in take.items():
            left[c] -= tiles * t
        out.append((tiles, take))
    return out


def tile_ns(blocks, d_model, filled, ranges):
    """Time of a tile of `blocks` blocks of which `filled` hold tokens of `ranges` ranges."""
    f = max(filled, 2)
    if blocks == 8:
        return 10000 + d_model * (20000 + 11100 * f) // 5120 + 800 * (ranges - 1)
    k_loop = 4300 + 2280 * f if d_model < 8192 else 11100 + 1880 * f
    return 11000 + 800 * f + d_model * k_loop // 1024 + 1100 * (ranges - 1)


def _queue_options(n_full, full_blocks, count, heads, blocks, d_model):
    """[(cap, end of the last of the queue's 32 workgroups, time of all tiles)] of a queue with `heads` heads.  Tiles are dealt in
    rounds, every second one backwards.  Full ranges as long as the tile have tiles of their own; shorter ones are ranges like the
    others, and then there is no cap 0.  Sharing costs a workgroup 2500 ns at its begin."""
    def option(cap, tiles):
        begin = 2500 if cap else 0
        load = [begin] * 32
        for i, ns in enumerate(tiles):
            load[i % 32 if (i // 32) % 2 == 0 else 31 - i % 32] += ns
        return cap, max(load), sum(load)

    own = full_blocks == blocks
    fulls = [tile_ns(blocks, d_model, blocks, 1)] * (n_full * heads if own else 0)
    out = []
    if own:
        tiles = fulls + [tile_ns(blocks, d_model, c, 1) for c in range(blocks, 0, -1) for _ in range(count[c] * heads)]
        out.append(option(0, tiles))
        if sum(count) < 2 or len(tiles) <= 32:
            return out
    for cap in range(blocks, 3 if own else full_blocks, -1):
        ranges = list(count)
        if not own:
            ranges[full_blocks] += n_full
        tiles = list(fulls)
        for n, take in tile_patterns(ranges, cap, blocks):
            tiles += [tile_ns(blocks, d_model, sum(c * t for c, t in take.items()), sum(take.values()))] * (n * heads)
        out.append(option(cap, tiles))
    return out


def shared_tiles_word(ctx_lens, cache_kind, n_heads, d_model, hidden_chunk):
    """Word 31 of a plan with packed weights and hidden-kind requests: four bits per queue, the blocks a shared tile may fill (0: a
    tile per range).  Tiles have hidden_chunk rows, or 320 rows for ranges of 256 where the launch is done sooner with them.  A
    launch is done when its last workgroup is, but not before all its work, the KV-kind items' included, is spread evenly over 256;
    of equals, the one with less work, then the first (cap 0, then the larger caps)."""
    hid = [int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_HIDDEN]
    kv = sum(int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_KV) * d_model // 1375
    count = [0] * 11
    for n in hid:
        if n % hidden_chunk:
            count[ceil_div(n % hidden_chunk, 32)] += 1
    n_full = sum(n // hidden_chunk for n in hid)
    heads = [ceil_div(n_heads - x, N_QUEUES) for x in range(min(n_heads, N_QUEUES))]
    sizes = sorted(set(heads), reverse=True)

    best = None
    for blocks in [hidden_chunk // 32] + ([10] if hidden_chunk == 256 else []):
        options = [_queue_options(n_full, hidden_chunk // 32, count, h, blocks, d_model) for h in sizes]
        for choice in itertools.product(*options):
            total = sum(heads.count(h) * o[2] for h, o in zip(sizes, choice))
            key = max(256 * max(o[1] for o in choice), total + 256 * kv), total
            if best is None or key < best[0]:
                best = key, {h: o[0] for h, o in zip(sizes, choice)}
    return sum(best[1][h] << 4 * x for x, h in enumerate(heads))


def deals_heads(ctx_lens, cache_kind, n_heads, hidden_chunk, word, n_workgroups=256):
    """Whether a launch with packed weights deals the heads that not every queue has to all XCDs.  word: the plan's word 31."""
    more, per_queue = n_heads % N_QUEUES, n_workgroups // N_QUEUES
    if more == 0 or (more > 4 and n_heads > N_QUEUES):
        return False
    lens = [int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_HIDDEN]
    caps = [(word >> 4 * x) & 15 for x in range(N_QUEUES)]
    blocks = 10 if hidden_chunk == 320 or max(caps) > 8 else 8
    ranges, heads = sum(ceil_div(n, hidden_chunk) for n in lens), ceil_div(n_heads, N_QUEUES)

    def tiles(cap):
        if not cap:
            return ranges
        count, own = [0] * (blocks + 1), 0
        for n in lens:
            for t0 in range(0, n, hidden_chunk):
                c = ceil_div(min(n - t0, hidden_chunk), 32)
                own += n - t0 >= hidden_chunk == 32 * blocks
                count[c] += not n - t0 >= hidden_chunk == 32 * blocks
        return own + sum(n for n, _ in tile_patterns(count, cap, blocks))

    longer, shorter = caps[0], caps[more if n_heads > N_QUEUES else 0]
    undealt, d = tiles(longer) * heads, 128 * n_heads
    kv = sum(int(n) for n, k in zip(ctx_lens, cache_kind) if int(k) == KIND_KV) * d // 1375
    if 5 * kv * n_workgroups >= 4 * tiles(longer) * tile_ns(blocks, d, blocks, 1) * (heads * N_QUEUES - n_heads):
        return False
    if undealt >= 4 * per_queue:
        return True
    if longer != shorter and ranges * heads < 4 * per_queue:
        return False
    n = tiles((longer if more >= 4 else shorter) or max(longer, shorter))
    dealt = [n * (n_heads // N_QUEUES) + sum((t + q) % N_QUEUES == x for t in range(n) for q in range(more)) for x in range(N_QUEUES)]
    return ceil_div(max(dealt), per_queue) < ceil_div(undealt, per_queue)


def plan(ctx_lens, cache_kind, n_heads, hidden_chunk, kv_chunk, hidden_item_per_head=True):
    """hidden_item_per_head=False: the absorbed-weight hidden path, whose items serve all heads of a
    range at once: one item (r, 0, t0, t1) per range of a hidden-kind request, by request and range,
    all in queue 0."""
    B = len(ctx_lens)
    split_count, ws_offset = [], []
    run = 0
    for r in range(B):
        n = int(ctx_lens[r])
        if n < 1:
            raise ValueError("ctx_len must be >= 1")
        if int(cache_kind[r]) not in (KIND_KV, KIND_HIDDEN):
            raise ValueError("unknown cache kind")
        c = hidden_chunk if int(cache_kind[r]) == KIND_HIDDEN else kv_chunk
        split_count.append(ceil_div(n, c))
        ws_offset.append(run)
        run += split_count[-1]
    def all_items(kind, c):
        out = []
        for r in range(B):
            if int(cache_kind[r]) != kind:
                continue
            n = int(ctx_lens[r])
            for s in range(split_count[r]):
                for h in range(n_heads):
                    out.append((r, h, s * c, min(n, (s + 1) * c)))
        return out

    items = []
    queue_offset = []
    hidden = all_items(KIND_HIDDEN, hidden_chunk)
    if not hidden_item_per_head:
        hidden = [it for it in hidden if it[1] == 0]
    for x in range(N_QUEUES):
        queue_offset.append(len(items))
        if not hidden_item_per_head:
            if x == 0:
                items += sorted(hidden, key=lambda it: (it[0], it[2]))
            continue
        mine = [it for it in hidden if it[1] % N_QUEUES == x]
        full = [it for it in mine if it[3] - it[2] == hidden_chunk]
        tails = [it for it in mine if it[3] - it[2] != hidden_chunk]
        full.sort(key=lambda it: (it[0], it[2], it[1]))
        tails.sort(key=lambda it: (-(it[3] - it[2]), it[0], it[1]))
        items += full + tails
    queue_offset.append(len(items))
    n_hidden_items = len(items)
    kv = all_items(KIND_KV, kv_chunk)
    kv.sort(key=lambda it: (-(it[3] - it[2]), it[0], it[2], it[1]))
    items += kv
    return {
        "split_count": split_count,
        "ws_offset": ws_offset,
        "items": items,
        "n_hidden_items": n_hidden_items,
        "n_partials": run,
        "queue_offset": queue_offset,
    }


def partial_slot(ws_offset, n_heads, r, s, h):
    return (ws_offset[r] + s) * n_heads + h


def token_location(block_list, block_size, j):
    """(block id, slot) of token j given the request's list of blocks."""
    return block_list[j // block_size], j % block_size


def blocks_for(n_tokens, block_size):
    return ceil_div(n_tokens, block_size)


def cache_bytes(n_tokens, d_model, elem_bytes, kind):
    """Bytes of cached vectors for n tokens of one layer (un-padded)."""
    per_token = d_model * elem_bytes
    return n_tokens * per_token * (1 if kind == KIND_HIDDEN else 2)
