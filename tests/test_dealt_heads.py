"""Packed weights, head counts that are no multiple of eight: the tiles of the heads that not every queue has are dealt to all XCDs in turn
where csrc/apt_pack.h says so.  A range's partial does not depend on its place, so every request has the same bits in a dealt launch and
alone in a batch of its own that is not dealt."""
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import plan_oracle as po
from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl
from tests.helpers import launched_kernels

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run_host(tmp_path, main, text):
    """Output of a host program around apt_pack.h."""
    src, exe = tmp_path / "dealt.cpp", tmp_path / "dealt"
    src.write_text('#include <stdio.h>\n#include <vector>\n#include "apt_pack.h"\nint main() {\n' + main + "\n}\n")
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2504_07494_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], input=text, text=True, capture_output=True, check=True).stdout


def test_every_tile_of_every_head_is_one_xcds(tmp_path):
    """Tiles 0 .. of an XCD until the first that its heads do not have: all (head, tile) pairs once, no XCD more than one round of eight
    tiles' worth beyond another, a dealt head's tile t where (t + queue) % 8 says."""
    out = _run_host(tmp_path, """
    for (int H = 1; H <= 72; ++H)
        for (int tiles = 0; H % 8 && tiles < 40; tiles += tiles < 18 ? 1 : 7)
            for (int x = 0; x < 8; ++x)
                for (int i = 0;; ++i) {
                    int queue, place, t = apt_dealt_tile(i, x, H / 8, H % 8, &queue, &place);
                    if (t >= tiles) {
                        printf("%d %d %d -1 %d %d\\n", H, tiles, x, apt_dealt_tile(i + 1, x, H / 8, H % 8, &queue, &place) >= tiles, i);
                        break;
                    }
                    printf("%d %d %d %d %d %d\\n", H, tiles, x, t, queue, place);
                }""", "")
    rows = np.array(out.split(), dtype=np.int64).reshape(-1, 6)
    launches = 0
    for H in range(1, 73):
        of_h = rows[rows[:, 0] == H]
        for tiles in np.unique(of_h[:, 1]):
            r = of_h[of_h[:, 1] == tiles]
            ends, r = r[r[:, 3] < 0], r[r[:, 3] >= 0]
            assert len(ends) == 8 and (ends[:, 4] == 1).all() and ends[:, 5].max() - ends[:, 5].min() <= H % 8
            head = r[:, 4] + 8 * r[:, 5]
            assert len(r) == H * tiles == len(set(zip(head.tolist(), r[:, 3].tolist()))) and (head < H).all()
            own = r[:, 5] < H // 8
            assert (r[own, 4] == r[own, 2]).all() and ((r[~own, 3] + r[~own, 4]) % 8 == r[~own, 2]).all()
            launches += 1
    assert launches == 63 * 22


def _plan(lens, kinds, heads, tile):
    shape = ab.make_shape(heads * 128, heads, 128, 16, "f16", 512, 0.1, hidden_chunk=tile)
    buf = np.zeros(ab.apt_plan_max_bytes(shape, len(lens), 8192) // 4, dtype=np.int32)
    info = ab.apt_plan(shape, np.asarray(lens, dtype=np.int32), np.asarray(kinds, dtype=np.uint8), buf)
    return buf[:int(info.plan_bytes) // 4]


def test_rule_against_the_plain_one(tmp_path):
    g = np.random.default_rng(12)
    lines, want, seen = [], [], set()
    for i in range(3000):
        H, B, tile = int(g.integers(1, 73)), int(10 ** g.uniform(0, 2.2)), int(g.choice([256, 320]))
        top = int(10 ** g.uniform(1, 3.4))
        lens = g.integers(1, top + 1, size=B) if i % 3 else np.full(B, int(g.choice([tile, 2 * tile, 1000, 64, top])))
        kinds = (g.random(B) < g.choice([0.3, 1.0])).astype(np.uint8)
        word = int(np.uint32(_plan(lens, kinds, H, tile)[31]))
        workgroups = int(g.choice([256, 256, 304, 64, 8]))
        kv_tokens = int(lens[kinds == 0].sum())
        lines.append(" ".join(map(str, [B, H, tile, word, workgroups, kv_tokens, *lens, *kinds])))
        want.append(po.deals_heads(lens, kinds, H, tile, word, workgroups))
        ranges = sum(-(-int(n) // tile) for n, k in zip(lens, kinds) if k) * -(-H // 8)
        seen.add((H < 8, ranges >= workgroups // 2, want[-1]))
    got = _run_host(tmp_path, """
    int B, H, chunk, workgroups, kv;
    unsigned word;
    while (scanf("%d %d %d %u %d %d", &B, &H, &chunk, &word, &workgroups, &kv) == 6) {
        std::vector<int32_t> lens(B), kinds(B);
        for (int& v : lens) if (scanf("%d", &v) != 1) return 1;
        for (int& v : kinds) if (scanf("%d", &v) != 1) return 1;
        const bool rows320 = chunk == 320 || apt_pack_wide(word);
        printf("%d\\n", (rows320 ? apt_deals<10> : apt_deals<8>)(lens.data(), kinds.data(), B, kv, H, 128 * H, chunk, word, workgroups));
    }""", "\n".join(lines))
    assert [int(v) for v in got.split()] == [int(v) for v in want]
    # below eight heads and beyond, with four rounds of ranges and with fewer, dealt and not
    assert seen == {(few, many, dealt) for few in (False, True) for many in (False, True) for dealt in (False, True)}


@pytest.mark.parametrize("heads,lens,tile,dealt", [
    (3, [200] * 140, 256, True), (7, [90] * 400, 320, True), (17, [300] * 100, 256, True),              # four rounds of tiles
    (7, [90] * 300, 320, True), (3, [200] * 60 + [31] * 80, 256, True), (65, [130, 180, 230, 275] * 4, 256, True),   # of ranges; a round saved
    (7, [90, 33, 320] * 50, 320, False), (20, [31, 64, 95] * 30, 256, False), (5, [40] * 140, 256, False),           # of ranges; no round saved
    (10, [4608] * 2, 256, True), (9, [130] * 36, 256, True), (20, [512] * 18, 256, True), (5, [256] * 33, 256, True),    # a round saved
    (10, [64] * 36, 256, False), (12, [1064] * 2, 256, False), (7, [60] * 20, 320, False),               # no round saved
    (10, [100] * 36, 256, False),                                                                        # queues share tiles differently
    (13, [200] * 300, 256, False), (23, [512] * 18, 256, False), (16, [512] * 18, 256, False)])           # more than four such heads, none
def test_batches_of_every_branch(heads, lens, tile, dealt):
    word = int(np.uint32(_plan(lens, [1] * len(lens), heads, tile)[31]))
    assert word == po.shared_tiles_word(lens, [1] * len(lens), heads, 128 * heads, tile)
    assert po.deals_heads(lens, [1] * len(lens), heads, tile, word) == dealt


@pytest.mark.parametrize("heads,hidden,kv,dealt", [(6, [800] * 45, 0, True), (6, [800] * 45, 50, True), (6, [800] * 45, 140, False),
                                                   (33, [1200] * 20, 20, True), (33, [1200] * 20, 160, False), (3, [200] * 60, 400, False)])
def test_what_kv_kind_items_fill_is_not_dealt(heads, hidden, kv, dealt):
    lens, kinds = hidden + [800] * kv, [1] * len(hidden) + [0] * kv
    word = int(np.uint32(_plan(lens, kinds, heads, 256)[31]))
    assert po.deals_heads(lens, kinds, heads, 256, word) == dealt
    assert po.deals_heads(hidden, [1] * len(hidden), heads, 256, word)


def _deals(rn, lens, kinds):
    """Whether the runner's attention call is a dealt launch, by the name of its kernel; the oracle's rule says the same."""
    n_wg = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    want = po.deals_heads(lens, kinds, rn.cfg.n_heads, rn.info.hidden_chunk, int(np.uint32(int(rn.plan_host[31]) & 0xffffffff)), n_wg)
    name, = [n for n in launched_kernels(rn.call) if "apt_items_mfma_kernel" in n]
    assert ("Lb1E" in name) == want and ("Lb0E" in name) != want, name
    return want


def _runner(batch, dl=None, **kw):
    from paper_2504_07494_amd.harness import DecodeRunner
    rn = DecodeRunner(batch, **kw)
    dl = dl or rn.upload(wl.make_layer(batch))
    rn.call = lambda: rn.run(dl)
    return rn, dl


def _against_alone(batch, kw, requests):
    """Outputs of the batch, finite; the named requests alone, not dealt, have the same bits.  Returns whether the batch is dealt."""
    rn, dl = _runner(batch, **kw)
    dealt = _deals(rn, batch.ctx_lens, batch.cache_kind)
    rn.out.fill_(float("nan"))
    rn.run(dl)
    torch.cuda.synchronize()
    got = rn.out.clone()
    assert bool(torch.isfinite(got).all())
    for r in requests:
        one, _ = _runner(wl.replace(batch, ctx_lens=batch.ctx_lens[r:r + 1].copy(), cache_kind=batch.cache_kind[r:r + 1].copy(),
                                    block_tables=batch.block_tables[r:r + 1].copy()), dl, **kw)
        if batch.cache_kind[r] == wl.KIND_HIDDEN:
            assert not _deals(one, batch.ctx_lens[r:r + 1], batch.cache_kind[r:r + 1])
        q = dl.q
        dl.q = q[r:r + 1].contiguous()
        one.run(dl)
        torch.cuda.synchronize()
        dl.q = q
        assert torch.equal(one.out[0], got[r]), (r, int(batch.ctx_lens[r]))
    return dealt


def _batch(dtype, H, lens, kinds, block=16):
    cfg = wl.small_config(name="dealt", dtype=dtype, d_model=128 * H, n_heads=H, head_dim=128, block_size=block, batch=len(lens), len_lo=1,
                          len_hi=int(np.max(lens)), hidden_ratio=0.8, permute_pages=True)
    return wl.make_batch(cfg, np.asarray(lens, dtype=np.int32), np.asarray(kinds, dtype=np.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 17, 20])
@pytest.mark.parametrize("tile,what", [(256, "short"), (256, "long"), (320, "mixed")])
def test_every_request_as_alone(H, tile, what):
    print(f"[case] dealt heads {H} tile {tile} {what}", flush=True)
    rng = np.random.default_rng(H)
    lens = {"short": rng.integers(1, 200, size=70), "long": rng.choice([256, 512, 513, 700], size=40),
            "mixed": rng.integers(1, 900, size=50)}[what].astype(np.int32)
    kinds = np.ones(len(lens), dtype=np.uint8) * wl.KIND_HIDDEN
    if what == "mixed":
        kinds[::5] = wl.KIND_KV
    _against_alone(_batch("bf16", H, lens, kinds), dict(hidden_chunk=tile, kv_chunk=256), list(range(0, len(lens), 9)) + [len(lens) - 1])


@pytest.mark.gpu
@pytest.mark.parametrize("H,lens,tile,dealt", [
    (3, [200] * 60 + [31] * 80, 256, True), (7, [90, 33, 320] * 90, 320, True),                        # four rounds of ranges, below eight heads
    (7, [90, 33, 320] * 50, 320, False), (20, [31, 64, 95] * 30, 256, False),                           # in tiles less, and no round saved
    (10, [4608] * 2, 256, True), (9, [130] * 36, 256, True), (20, [512] * 18, 256, True),              # a round saved, beyond eight
    (26, [512, 512, 256, 256, 768], 256, True),
    (10, [64] * 36, 256, False), (10, [100] * 36, 256, False), (13, [200] * 100, 256, False), (16, [512] * 18, 256, False)])
def test_each_reason_to_deal_and_not_to(H, lens, tile, dealt):
    print(f"[case] dealt heads {H} tile {tile} {len(lens)} requests", flush=True)
    kinds = np.full(len(lens), wl.KIND_HIDDEN, dtype=np.uint8)
    picks = [r for r in sorted({0, 1, len(lens) // 2, len(lens) - 1}) if lens[r] < 4000]
    assert _against_alone(_batch("f16", H, lens, kinds, block=32), dict(hidden_chunk=tile), picks) == dealt


@pytest.mark.gpu
@pytest.mark.parametrize("dealt_first", [True, False])
def test_captured_launch_replayed_with_a_plan_of_the_other_choice(dealt_first):
    """Plans of the same counts, one that is dealt and one that is not: a replay has the eager call's bits whichever was captured."""
    print(f"[case] dealt capture first={dealt_first}", flush=True)
    n, H = 36, 10
    plans = [np.full(n, 256, dtype=np.int32), np.random.default_rng(5).integers(33, 97, size=n).astype(np.int32)]
    batch = _batch("f16", H, plans[0], np.full(n, wl.KIND_HIDDEN, dtype=np.uint8))
    rn, dl = _runner(batch, hidden_chunk=256)
    eager = []
    for lens, dealt in zip(plans, (True, False)):
        rn.plan(lens)
        assert _deals(rn, lens, batch.cache_kind) == dealt
        eager.append(rn.run(dl).clone())
    first = plans[0 if dealt_first else 1]
    rn.plan(first)
    out = torch.empty_like(rn.out)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        rn.run(dl, out=out)
    for rep in range(6):
        i = rep % 2
        rn.plan(plans[i])
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager[i]), rep
