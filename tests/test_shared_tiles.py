"""Tiles of the packed-weight projection kernel that hold the short ranges of several requests (csrc/apt_pack.h)."""
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import plan_oracle as po
from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl
from tests.helpers import oracle_attn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HID, KV = 1, 0


def _patterns(tmp_path, blocks, cases):
    """The library's patterns for (cap, counts of class 1 ..): [(tiles, ranges of class 0, 1, ..)] per case, compiled for the host."""
    src = tmp_path / f"pack{blocks}.cpp"
    src.write_text(f"""
#include <stdio.h>
#include "apt_pack.h"
int main() {{
    int cap, left[{blocks} + 1] = {{0}};
    while (scanf("%d", &cap) == 1) {{
        for (int c = 1; c <= {blocks}; ++c) if (scanf("%d", left + c) != 1) return 1;
        apt_pack_patterns<{blocks}>(left, cap, [](int reps, const int* take) {{
            printf("%d", reps);
            for (int c = 0; c <= {blocks}; ++c) printf(" %d", take[c]);
            printf(";");
        }});
        printf("\\n");
    }}
}}
""")
    exe = tmp_path / f"pack{blocks}"
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2504_07494_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    text = "\n".join(" ".join(map(str, [cap, *counts])) for cap, counts in cases)
    lines = subprocess.run([str(exe)], input=text, text=True, capture_output=True, check=True).stdout.split("\n")
    return [[list(map(int, p.split())) for p in line.split(";") if p] for line in lines[:len(cases)]]


@pytest.mark.parametrize("blocks", [8, 10])
def test_patterns_take_every_range_once_and_fit_a_tile(tmp_path, blocks):
    g = np.random.default_rng(blocks)
    cases = [(cap, [0] * blocks) for cap in (4, blocks)]
    for _ in range(3000):
        top = int(10 ** g.uniform(0, 4))
        cases.append((int(g.integers(4, blocks + 1)), (g.integers(0, top + 1, size=blocks) * (g.random(blocks) < g.random())).tolist()))
    most = 0
    for (cap, counts), pats in zip(cases, _patterns(tmp_path, blocks, cases)):
        used = np.zeros(blocks + 1, dtype=np.int64)
        for reps, *take in pats:
            size, n = sum(c * t for c, t in enumerate(take)), sum(take)
            assert reps > 0 and take[0] == 0 and 1 <= n <= (8 if blocks == 8 else 6)
            assert size <= cap or (n == 1 and size <= blocks)
            used += reps * np.array(take)
        assert used[1:].tolist() == counts
        most = max(most, len(pats))
    assert 10 < most <= (20 if blocks == 8 else 27)      # the device's tables hold 32


def _caps(info, buf):
    return [(int(np.uint32(buf[31])) >> (4 * x)) & 15 for x in range(8)]


def _plan(lens, kinds, **kw):
    shape = ab.make_shape(kw["heads"] * 128, kw["heads"], 128, 16, "f16", 128, 0.1, hidden_chunk=kw.get("tile", 0))
    buf = np.zeros(ab.apt_plan_max_bytes(shape, len(lens), 2048) // 4, dtype=np.int32)
    return _caps(ab.apt_plan(shape, np.array(lens, dtype=np.int32), np.array(kinds, dtype=np.uint8), buf), buf)


def test_planner_shares_tiles_only_beyond_one_tile_per_workgroup():
    assert _plan([60] * 32, [HID] * 32, heads=8) == [0] * 8               # 32 tiles of a queue, 32 workgroups
    assert _plan([60] * 33, [HID] * 33, heads=8) == [5] * 8               # two to a tile are enough for one round
    assert _plan([60] * 20, [HID] * 20, heads=12) == [5] * 4 + [0] * 4    # 40 tiles in the queues of two heads, 20 in the others
    assert _plan([100, 60, 60] * 640, [HID] * 1920, heads=8) == [8] * 8   # many rounds: full tiles
    assert _plan([250] * 64, [HID] * 64, heads=8) == [0] * 8              # nothing fits together
    assert _plan([512] * 40, [HID] * 40, heads=8) == [0] * 8              # full ranges only
    # 33 full ranges and 31 of half a tile: two rounds either way, shorter with a tile per range
    assert _plan([384] * 31 + [256], [HID] * 32, heads=8) == [0] * 8
    assert _plan([60] * 40, [KV] * 40, heads=8) == [0] * 8
    # ranges of 256 tokens in tiles of 320 rows where that saves a round, and not beyond a few rounds
    assert _plan([256] * 28 + [257, 300, 320, 316], [HID] * 32, heads=8) == [10] * 8
    assert _plan([256] * 28 + [257, 300, 320, 316], [HID] * 32, heads=7) == [10] * 7 + [0]
    assert _plan([320] * 640, [HID] * 640, heads=8) == [8] * 8


def test_planner_word_against_the_plain_rule():
    """Few and many heads, queues of two sizes, batches of one round and of many, both chunks, any share of KV-kind requests."""
    g = np.random.default_rng(31)
    seen = set()
    for i in range(1200):
        heads = int(g.integers(1, 73))
        B = int(10 ** g.uniform(0, 2.4))
        top = int(10 ** g.uniform(1, 3.3))
        lens = g.integers(1, top + 1, size=B) if i % 4 else np.minimum(2048, 32 * g.integers(1, 20, size=B))
        kinds = (g.random(B) < g.choice([0.1, 0.5, 0.9, 1.0])).astype(np.uint8)
        tile = int(g.choice([256, 320]))
        caps = _plan(lens, kinds, heads=heads, tile=tile)
        word = po.shared_tiles_word(lens, kinds, heads, 128 * heads, tile) if kinds.any() else 0
        assert caps == [(word >> 4 * x) & 15 for x in range(8)], (heads, tile, lens.tolist(), kinds.tolist())
        seen.update((tile, c) for c in caps)
    assert seen == {(t, c) for t in (256, 320) for c in [0, *range(4, 11)]}


LENS = {256: [255, 225, 224, 193, 161, 160, 129, 128, 97, 96, 65, 64, 63, 33, 32, 31, 2, 1, 256, 257, 300, 511, 700],
        320: [319, 289, 288, 257, 225, 161, 160, 159, 129, 97, 96, 65, 64, 33, 32, 31, 2, 1, 320, 321, 400, 639, 700]}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,tile,H,bs,n_one", [("f16", 256, 8, 16, 22), ("bf16", 256, 3, 64, 40), ("f16", 320, 8, 16, 22),
                                                   ("bf16", 320, 9, 4, 10)])
def test_shared_tiles_against_the_oracle(oracle, dtype, tile, H, bs, n_one):
    """Every block count, ranges that end on and next to a block, one-token ranges many to a tile, both kinds; twice the
    tails of a queue, so that patterns repeat."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] shared tiles {dtype} tile {tile} heads {H} block {bs}", flush=True)
    lens = np.array(LENS[tile] + LENS[tile][:14] + [1] * n_one + [90, 300], dtype=np.int32)
    kinds = np.array([HID] * (len(lens) - 2) + [KV, KV], dtype=np.uint8)
    order = np.random.default_rng(H).permutation(len(lens))
    lens, kinds = lens[order], kinds[order]
    cfg = wl.small_config(name="shared", dtype=dtype, d_model=128 * H, n_heads=H, head_dim=128, block_size=bs, batch=len(lens),
                          len_lo=1, len_hi=700, hidden_ratio=0.9)
    batch = wl.make_batch(cfg, lens, kinds)
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, hidden_chunk=tile)
    caps = _caps(rn.info, rn.plan_host.numpy())
    assert rn.info.hidden_chunk == tile and caps[0] > 0
    dl = rn.upload(layer)
    rn.run(dl)
    got = rn.out_f64().copy()
    want = oracle_attn(oracle, batch, layer).reshape(got.shape)
    assert np.max(np.abs(got - want)) < 2e-4
    # a tile per range (the planner's word cleared): the same sums, cut in halves elsewhere
    rn.plan_dev[31] = 0
    rn.run(dl)
    assert np.max(np.abs(rn.out_f64() - got)) < 2e-5


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,H", [("f16", 8), ("bf16", 7)])
def test_short_ranges_beside_full_ones_in_larger_tiles(oracle, dtype, H):
    """Ranges of 256 tokens in tiles of 320 rows; then the same launch with the words a replayed capture could meet: plans for
    shared tiles of 8 blocks and for a tile per range."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] wide tiles {dtype} heads {H}", flush=True)
    lens = np.array([256] * 28 + [257, 300, 320, 316, 100], dtype=np.int32)
    kinds = np.array([HID] * 32 + [KV], dtype=np.uint8)
    cfg = wl.small_config(name="wide", dtype=dtype, d_model=128 * H, n_heads=H, head_dim=128, block_size=16, batch=len(lens),
                          len_lo=1, len_hi=320, hidden_ratio=0.9)
    batch = wl.make_batch(cfg, lens, kinds)
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch)
    assert rn.info.hidden_chunk == 256 and _caps(rn.info, rn.plan_host.numpy())[0] == 10
    dl = rn.upload(layer)
    rn.run(dl)
    got = rn.out_f64().copy()
    assert np.max(np.abs(got - oracle_attn(oracle, batch, layer).reshape(got.shape))) < 2e-4
    for word in (0x88888888 - (1 << 32), 0):
        rn.plan_dev[31] = word
        rn.run(dl)
        assert np.max(np.abs(rn.out_f64() - got)) < 2e-5
    # the kernel of 256-row tiles with a plan for larger ones
    rn.plan()
    torch.cuda.synchronize()                  # the copy of the plan has read the host's words
    rn.plan_host[31] = 0
    assert int(np.uint32(rn.plan_dev[31].item() & 0xffffffff)) & 15 == 10
    rn.run(dl)
    torch.cuda.synchronize()
    assert np.max(np.abs(rn.out_f64() - got)) < 2e-5


@pytest.mark.gpu
def test_a_request_with_infinities_leaves_the_others_of_its_tile_alone():
    from paper_2504_07494_amd.harness import DecodeRunner
    print("[case] shared tiles, infinite hidden vectors", flush=True)
    lens = np.array([31, 64, 100, 1] * 12, dtype=np.int32)
    cfg = wl.small_config(name="sharedinf", dtype="f16", d_model=1024, n_heads=8, head_dim=128, block_size=16, batch=len(lens),
                          len_lo=1, len_hi=100, hidden_ratio=1.0)
    batch = wl.make_batch(cfg, lens, np.full(len(lens), HID, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch)
    assert min(_caps(rn.info, rn.plan_host.numpy())) > 0
    dl = rn.upload(layer)
    rn.run(dl)
    want = rn.out_f64().copy()
    bad = [1, 6, 20]
    pool = layer.pool.view(np.uint16).reshape(layer.pool.shape[0], -1)
    for r in bad:
        pool[batch.block_tables[r, 0, 0], :1024] = 0x7c00              # first token of the request
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    good = np.setdiff1d(np.arange(len(lens)), bad)
    assert np.array_equal(got[good], want[good]) and not np.isfinite(got[bad]).all()


@pytest.mark.gpu
@pytest.mark.parametrize("n_kv", [0, 3])
def test_a_cap_for_a_queue_without_heads_is_passed_over(n_kv):
    """Queue 7 of 7 heads holds no items: what follows it in the list are KV-kind ranges of up to 512 tokens, or nothing.  Queues of
    a plan without heads have no cap; one that is there all the same changes nothing."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] cap for an empty queue, {n_kv} KV-kind requests", flush=True)
    lens = np.array([31, 64, 100, 1] * 10 + [600, 512, 90][:n_kv], dtype=np.int32)
    cfg = wl.small_config(name="emptyqueue", dtype="f16", d_model=128 * 7, n_heads=7, head_dim=128, block_size=16, batch=len(lens),
                          len_lo=1, len_hi=600, hidden_ratio=1.0)
    batch = wl.make_batch(cfg, lens, np.array([HID] * 40 + [KV] * n_kv, dtype=np.uint8))
    rn = DecodeRunner(batch)
    caps = _caps(rn.info, rn.plan_host.numpy())
    assert min(caps[:7]) > 0 and caps[7] == 0
    dl = rn.upload(wl.make_layer(batch))
    rn.run(dl)
    want = rn.out.clone()
    torch.cuda.synchronize()
    rn.plan_dev[31] = int(rn.plan_dev[31]) | 5 << 28
    rn.run(dl)
    assert torch.equal(rn.out, want) and bool(torch.isfinite(want).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,tile,H,bs", [("f16", 256, 8, 16), ("bf16", 256, 9, 8), ("f16", 320, 3, 32), ("bf16", 320, 8, 16)])
def test_output_of_a_hidden_kind_request_does_not_depend_on_the_batch(dtype, tile, H, bs):
    """Bit for bit: with shared tiles of every cap, with a tile per range, in tiles of 320 rows for ranges of 256 tokens, and each
    request in a batch of its own."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] batch invariance {dtype} tile {tile} heads {H}", flush=True)
    lens = np.array(LENS[tile] + LENS[tile][:16] + [33, 34, 64, 95] * 4 + [1, 30], dtype=np.int32)
    lens = lens[np.random.default_rng(tile + H).permutation(len(lens))]
    cfg = wl.small_config(name="invariant", dtype=dtype, d_model=128 * H, n_heads=H, head_dim=128, block_size=bs, batch=len(lens),
                          len_lo=1, len_hi=700, hidden_ratio=1.0)
    batch = wl.make_batch(cfg, lens, np.full(len(lens), HID, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, hidden_chunk=tile)
    assert _caps(rn.info, rn.plan_host.numpy())[0] > 0
    dl = rn.upload(layer)
    rn.run(dl)
    want = rn.out.clone()
    torch.cuda.synchronize()
    queues = min(H, 8)
    for wide in (0, 1) if tile == 256 else (0,):                  # the host's word picks the kernel, the device's the caps
        for cap in (0, 4, 5, 6, 7, 8, 9, 10):
            word = sum(cap << 4 * x for x in range(queues))
            rn.plan_host[31] = 10 * wide
            rn.plan_dev[31] = word - (1 << 32) if word >= 1 << 31 else word
            rn.out.fill_(float("nan"))
            rn.run(dl)
            assert torch.equal(rn.out, want), (wide, cap)
    for r in range(0, len(lens), 3):
        one = wl.make_batch(wl.replace(cfg, batch=1), lens[r:r + 1], np.array([HID], dtype=np.uint8))
        rn1 = DecodeRunner(one, hidden_chunk=tile)
        rn1.block_tables = rn.block_tables[r:r + 1, :, :one.max_blocks].contiguous()     # its blocks in the same pool
        dl.q, q = dl.q[r:r + 1].contiguous(), dl.q
        rn1.run(dl)
        dl.q = q
        assert torch.equal(rn1.out[0], want[r]), int(lens[r])
