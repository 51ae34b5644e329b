"""Batches of KV-kind requests alone, against the CPU oracle, on every path that the launch takes for them: whole contexts with
sixteen waves (as many (request, head) pairs as CUs, or fewer) or with four (every context one range), and ranges with a merge.
fp32 sums of at most 1037 weights and 128 products: errors of the scores and of the value sums are a few hundred times 2^-24 of
their size, 1e-4 is ten times that."""
import numpy as np
import pytest
import torch

from paper_2504_07494_amd import workloads as wl
from paper_2504_07494_amd.harness import DecodeRunner
from tests.helpers import oracle_attn

pytestmark = pytest.mark.gpu


# lengths around a page of every wave (4 and 16 waves; pages of 4 to 32 tokens), a lone token, whole and open ranges of 512 tokens
SHORT = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 257, 511, 512]
LONG = SHORT + [513, 1037]


@pytest.mark.parametrize("dtype,out,hd,bs", [("f16", "f32", 128, 16), ("bf16", "bf16", 128, 8), ("f16", "f16", 64, 32), ("bf16", "f32", 64, 8),
                                             ("f32", "f32", 128, 16), ("f32", "f32", 64, 4)])
@pytest.mark.parametrize("lens,n_heads", [(SHORT, 4), (SHORT, 18), (SHORT, 19), (LONG, 4), (LONG, 16), (LONG, 17)])
def test_kv_batches_with_and_without_partials(oracle, dtype, out, hd, bs, lens, n_heads):
    print(f"[case] {dtype} hd={hd} bs={bs} heads={n_heads} requests={len(lens)}", flush=True)
    cfg = wl.small_config(name="kvwaves", dtype=dtype, d_model=hd * n_heads, n_heads=n_heads, head_dim=hd, block_size=bs,
                          batch=len(lens), len_lo=1, len_hi=max(lens), hidden_ratio=0.0, permute_pages=True)
    batch = wl.make_batch(cfg, np.array(lens, dtype=np.int32), np.full(len(lens), wl.KIND_KV, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, out_dtype=out)
    rn.out.fill_(float("nan"))
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    want = oracle_attn(oracle, batch, layer).reshape(got.shape)
    assert np.all(np.isfinite(got))
    err = np.abs(got - want)
    print(f"[parity] max_abs={err.max():.3e}", flush=True)
    # the last rounding of a 16-bit output: half a unit in the last place of its 11 or 8 bits
    assert np.all(err <= 1e-4 + np.abs(want) * {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[out])


# 16 requests of one or two ranges: 4 and 16 heads, no more (request, head) pairs than CUs
PAIRS = SHORT + [513, 600]


@pytest.mark.parametrize("dtype,hd,bs,lens,n_heads,whole", [
    ("f16", 128, 16, PAIRS, 16, True), ("bf16", 64, 8, PAIRS, 16, True), ("f32", 64, 16, PAIRS, 4, True), ("f32", 128, 16, SHORT, 19, True),
    ("f16", 128, 16, LONG, 4, False), ("bf16", 128, 16, [1743, 1100, 854], 40, False), ("f16", 64, 16, [2048], 40, False),
    ("f32", 128, 16, LONG, 4, False), ("f16", 128, 16, PAIRS, 17, False)])
def test_whole_contexts_where_they_pay(oracle, dtype, hd, bs, lens, n_heads, whole):
    """Which path ran shows in the workspace: whole contexts leave it as it was, ranges write their partials."""
    print(f"[case] {dtype} hd={hd} bs={bs} heads={n_heads} requests={len(lens)} whole={whole}", flush=True)
    cfg = wl.small_config(name="kvwhole", dtype=dtype, d_model=hd * n_heads, n_heads=n_heads, head_dim=hd, block_size=bs,
                          batch=len(lens), len_lo=1, len_hi=max(lens), hidden_ratio=0.0, permute_pages=True)
    batch = wl.make_batch(cfg, np.array(lens, dtype=np.int32), np.full(len(lens), wl.KIND_KV, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch)
    rn.out.fill_(float("nan"))
    rn.workspace.fill_(255)
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    assert bool((rn.workspace == 255).all()) == whole
    heads = sorted({0, n_heads // 2, n_heads - 1})
    want = oracle_attn(oracle, batch, layer, pairs=[(r, h) for r in range(len(lens)) for h in heads])
    assert np.max(np.abs(got[:, heads] - want.reshape(len(lens), len(heads), hd))) <= 1e-4


@pytest.mark.parametrize("dtype,hd,bs,chunk", [("f16", 128, 16, 256), ("bf16", 64, 8, 512), ("f32", 64, 16, 128), ("f32", 128, 4, 512)])
def test_a_given_range_length_fixes_the_sums_of_a_request(dtype, hd, bs, chunk):
    """Bit for bit: a KV-kind request by itself, in a small and in a large batch, and beside hidden-kind requests."""
    print(f"[case] {dtype} hd={hd} bs={bs} kv_chunk={chunk}", flush=True)
    lens = np.array(LONG + LONG, dtype=np.int32)
    cfg = wl.small_config(name="kvfixed", dtype=dtype, d_model=hd * 12, n_heads=12, head_dim=hd, block_size=bs, batch=len(lens),
                          len_lo=1, len_hi=max(lens), hidden_ratio=0.0, permute_pages=True)
    batch = wl.make_batch(cfg, lens, np.full(len(lens), wl.KIND_KV, dtype=np.uint8))
    layer = wl.make_layer(batch)
    full = DecodeRunner(batch, kv_chunk=chunk)
    assert full.info.n_items > 256                                    # four waves to a workgroup
    dl = full.upload(layer)
    full.run(dl)
    want = full.out.clone()

    def of(rows, kinds=None):
        part = wl.make_batch(wl.replace(cfg, batch=len(rows)), lens[rows], np.zeros(len(rows), dtype=np.uint8) if kinds is None else kinds)
        rn = DecodeRunner(part, kv_chunk=chunk)
        rn.block_tables = full.block_tables[rows][:, :, :part.max_blocks].contiguous()      # its blocks in the same pool
        q = dl.q
        dl.q = q[rows].contiguous()
        rn.run(dl)
        dl.q = q
        return rn.out
    for rows in ([15], [4], [13, 12, 14], list(range(16))):
        same = torch.equal(of(rows), want[rows])
        assert same, rows
    rows = [15, 3, 14, 13]                                            # request 3 read as hidden-kind: its output is another one
    same = torch.equal(of(rows, np.array([0, 1, 0, 0], dtype=np.uint8))[[0, 2, 3]], want[[15, 14, 13]])
    assert same
