"""The merge of the ranges' partials on both its ways, by the last workgroups of the item kernel (small calls) and in a kernel of its own,
around the sizes where one takes over from the other and around the ranges whose partials are asked for at once (four by 1024 threads,
twice eight by 256, eight in the kernel).  fp32 sums of at most 2048 products: errors a few hundred times 2^-24 of the values' size,
1e-4 is ten times that (as for the KV-kind batches)."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

from paper_2504_07494_amd import workloads as wl
from tests.helpers import oracle_attn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KV, HID = wl.KIND_KV, wl.KIND_HIDDEN


def _word(name):
    """Place of a word in the plan blob, from the library's header."""
    with open(os.path.join(ROOT, "paper_2504_07494_amd", "csrc", "apt_internal.h")) as f:
        return int(re.search(rf"\b{name} = (\d+)", f.read())[1])


# merges: the last workgroups do
CASES = [
    # 256 threads, 4096 values: 16, 17 and 33 ranges of 16 tokens; a request of one range beside them
    ("f16", "f16", 64, 3, 16, 16, [16, 256, 7], [KV, KV, KV], True), ("f16", "f32", 64, 3, 16, 16, [257, 40], [KV, KV], False),
    ("bf16", "bf16", 64, 1, 16, 16, [128, 129, 528], [KV, KV, KV], False), ("f32", "f32", 128, 2, 16, 16, [255, 1], [KV, KV], False),
    ("f32", "f32", 128, 2, 16, 16, [257], [KV], False),
    ("f16", "f16", 64, 8, 16, 64, [500], [KV], True), ("bf16", "f32", 128, 16, 16, 256, [500], [KV], True),
    ("f16", "f16", 64, 17, 8, 128, [130, 260], [KV, KV], False),
    # 1024 threads, 16384 values, 160 ranges: up to four ranges of 512 tokens; fewer heads than parts, a multiple, some beyond
    ("f16", "f16", 128, 32, 16, 0, [1743], [KV], True), ("bf16", "f32", 128, 33, 16, 0, [1743], [KV], False),
    ("f16", "f16", 128, 1, 8, 0, [1800, 1], [KV, KV], True), ("f32", "f32", 128, 7, 16, 0, [1300, 900, 1], [KV] * 3, True),
    ("bf16", "bf16", 128, 9, 16, 0, [700, 1100], [KV, KV], True), ("f16", "f32", 64, 40, 16, 0, [2048], [KV], True),
    ("f16", "f16", 64, 41, 16, 0, [2048], [KV], False), ("f16", "f16", 128, 40, 16, 0, [1237], [KV], True),
    ("bf16", "f32", 128, 4, 16, 0, [2049], [KV], False), ("f32", "f32", 64, 5, 16, 0, [1100] * 10, [KV] * 10, True),
    # raw weights, both kinds; 256 threads, 1024 channels
    ("f32", "f32", 64, 4, 16, 0, [128, 100, 60, 16], [KV, HID, KV, HID], True), ("f32", "f32", 64, 3, 4, 16, [150, 2, 33], [HID, KV, HID], True),
    ("f16", "f16", 64, 5, 8, 0, [300, 64, 65, 1], [HID, HID, KV, HID], False), ("bf16", "f32", 64, 9, 8, 0, [300, 200], [HID, KV], False),
    ("f16", "f16", 64, 8, 8, 0, [130, 64], [HID, HID], True), ("bf16", "bf16", 64, 8, 8, 0, [130, 600], [HID, KV], True),
    ("f32", "f32", 64, 1, 16, 0, [270, 30], [HID, HID], False), ("f32", "f32", 128, 2, 16, 0, [33, 100], [HID, HID], True)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out,hd,H,bs,chunk,lens,kinds,merges", CASES)
def test_merge_of_small_calls(oracle, dtype, out, hd, H, bs, chunk, lens, kinds, merges):
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] {dtype} -> {out} hd={hd} heads={H} chunk={chunk} lens={lens} merges={merges}", flush=True)
    cfg = wl.small_config(name="merge", dtype=dtype, d_model=hd * H, n_heads=H, head_dim=hd, block_size=bs, batch=len(lens),
                          len_lo=1, len_hi=max(lens), hidden_ratio=0.5, permute_pages=True)
    batch = wl.make_batch(cfg, np.array(lens, dtype=np.int32), np.array(kinds, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, out_dtype=out, kv_chunk=chunk)
    dl = rn.upload(layer)
    rn.workspace.fill_(255)
    rn.run(dl)
    first = rn.out.clone()
    assert not bool((rn.workspace == 255).all())     # ranges and partials, not whole contexts
    tickets = [_word("APT_PW_KV_TICKET")]
    if HID not in kinds:
        tickets += [_word("APT_PW_QUEUE0") + g for g in range(8)]
    for _ in range(3):                               # the tickets are 0 again after every call: the same plan serves the next
        rn.out.fill_(float("nan"))
        rn.run(dl)
        assert torch.equal(rn.out, first)
        assert int(rn.plan_dev[tickets].abs().sum()) == 0
    got = rn.out_f64()
    want = oracle_attn(oracle, batch, layer).reshape(got.shape)
    assert np.all(np.abs(got - want) <= 1e-4 + np.abs(want) * {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[out])
    # which way it went: with tickets that are not 0 no workgroup finds itself the last, and a merge kernel does not look at them
    rn.plan_dev[tickets] = 1000
    rn.out.fill_(float("nan"))
    rn.run(dl)
    assert bool(torch.isnan(rn.out).all()) == merges and (merges or torch.equal(rn.out, first))
    rn.plan()
    rn.run(dl)
    assert torch.equal(rn.out, first)


def test_rule_for_the_last_workgroups(tmp_path):
    """The library's rule, compiled for the host: calls that took the GPU longer than with a merge kernel are left to one, and none has more
    channels or partials than the threads that merge can take."""
    src, exe = tmp_path / "merge.cpp", tmp_path / "merge"
    src.write_text("""
#include <stdio.h>
#include "apt_internal.h"
int main() {
    int alone, threads, heads, hd, ranges;
    long long batch, items;
    while (scanf("%d %d %lld %d %d %lld %d", &alone, &threads, &batch, &heads, &hd, &items, &ranges) == 7)
        printf("%d\\n", apt_items_merge(alone, threads, batch, heads, hd, items, ranges));
}
""")
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2504_07494_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def rule(cases):
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases)
        return [int(v) for v in subprocess.run([str(exe)], input=text, text=True, capture_output=True, check=True).stdout.split()]
    slower = [(1, 1024, 2, 30, 64, 240, 4), (1, 1024, 3, 20, 128, 240, 4), (1, 1024, 1, 12, 128, 96, 8), (0, 256, 6, 8, 64, 48, 1),
              (0, 256, 4, 8, 64, 128, 4), (1, 256, 1, 1, 64, 64, 64)]
    assert rule(slower) == [0] * len(slower)
    g = np.random.default_rng(7)
    cases = []
    for _ in range(4000):
        batch, heads, ranges = int(2 ** g.uniform(0, 7)), int(g.integers(1, 73)), int(2 ** g.uniform(0, 6))
        total = int(g.integers(batch + ranges - 1, batch * ranges + 1))
        cases.append((g.integers(0, 2), g.choice([256, 1024]), batch, heads, g.choice([64, 128]), total * heads, ranges))
    got = rule(cases)
    assert 100 < sum(got) < len(got) / 2
    for (alone, threads, batch, heads, hd, items, ranges), merges in zip(cases, got):
        if merges:
            assert batch * (-(-heads // 8) if alone else heads) * hd // 4 <= threads and items <= 160
            assert items * hd <= 16 * threads and ranges <= (4 if threads == 1024 else 16)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,hd,H,lens,whole", [("bf16", 64, 2, [1269, 1017, 739, 996, 1229, 1065], False), ("bf16", 128, 9, [843], False),
                                                   ("f16", 64, 1, [1282, 789, 868, 991], False), ("f16", 128, 32, [563], True),
                                                   ("f32", 64, 9, [371, 586, 340, 593, 569], True)])
def test_whole_contexts_beside_a_merge_by_the_last_workgroups(oracle, dtype, hd, H, lens, whole):
    """Whole contexts only where they are faster than ranges whose partials the last workgroups merge (they leave the workspace as it was)."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] {dtype} hd={hd} heads={H} lens={lens} whole={whole}", flush=True)
    cfg = wl.small_config(name="mergewhole", dtype=dtype, d_model=hd * H, n_heads=H, head_dim=hd, block_size=16, batch=len(lens),
                          len_lo=1, len_hi=max(lens), hidden_ratio=0.0, permute_pages=True)
    batch = wl.make_batch(cfg, np.array(lens, dtype=np.int32), np.full(len(lens), KV, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch)
    rn.out.fill_(float("nan"))
    rn.workspace.fill_(255)
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    assert bool((rn.workspace == 255).all()) == whole
    assert np.max(np.abs(got - oracle_attn(oracle, batch, layer).reshape(got.shape))) <= 1e-4
