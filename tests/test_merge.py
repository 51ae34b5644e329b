"""The merge of the ranges' partials on both its ways, the last workgroup of the item kernel (small calls) and a kernel of its own,
around the size where one takes over from the other and around the eight ranges whose partials are asked for at once.  fp32 sums of at
most 1024 products: errors a few hundred times 2^-24 of the values' size, 1e-4 is ten times that (as for the KV-kind batches)."""
import numpy as np
import pytest
import torch

from paper_2504_07494_amd import workloads as wl
from paper_2504_07494_amd.harness import DecodeRunner
from tests.helpers import oracle_attn

pytestmark = pytest.mark.gpu

KV, HID = wl.KIND_KV, wl.KIND_HIDDEN


@pytest.mark.parametrize("dtype,out,hd,H,bs,chunk,lens,kinds", [
    # 256 threads, 4096 values: 16, 17 and 33 ranges of 16 tokens; a request of one range beside them
    ("f16", "f16", 64, 3, 16, 16, [16, 256, 7], [KV, KV, KV]), ("f16", "f32", 64, 3, 16, 16, [257, 40], [KV, KV]),
    ("bf16", "bf16", 64, 1, 16, 16, [128, 129, 528], [KV, KV, KV]), ("f32", "f32", 128, 2, 16, 16, [255, 1], [KV, KV]),
    ("f32", "f32", 128, 2, 16, 16, [257], [KV]),
    # 1024 threads, 16384 values: four ranges of 512 tokens
    ("f16", "f16", 128, 32, 16, 0, [1743], [KV]), ("bf16", "f32", 128, 33, 16, 0, [1743], [KV]),
    # raw weights, both kinds
    ("f32", "f32", 64, 4, 16, 0, [128, 100, 60, 16], [KV, HID, KV, HID]), ("f32", "f32", 64, 3, 4, 16, [150, 2, 33], [HID, KV, HID]),
    ("f16", "f16", 64, 5, 8, 0, [300, 64, 65, 1], [HID, HID, KV, HID]), ("bf16", "f32", 64, 9, 8, 0, [300, 200], [HID, KV])])
def test_merge_of_small_calls(oracle, dtype, out, hd, H, bs, chunk, lens, kinds):
    print(f"[case] {dtype} -> {out} hd={hd} heads={H} chunk={chunk} lens={lens}", flush=True)
    cfg = wl.small_config(name="merge", dtype=dtype, d_model=hd * H, n_heads=H, head_dim=hd, block_size=bs, batch=len(lens),
                          len_lo=1, len_hi=max(lens), hidden_ratio=0.5, permute_pages=True)
    batch = wl.make_batch(cfg, np.array(lens, dtype=np.int32), np.array(kinds, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, out_dtype=out, kv_chunk=chunk)
    dl = rn.upload(layer)
    rn.workspace.fill_(255)
    rn.run(dl)
    first = rn.out.clone()
    ticket = 25
    for _ in range(3):                               # the ticket is 0 again after every call: the same plan serves the next
        rn.out.fill_(float("nan"))
        rn.run(dl)
        assert torch.equal(rn.out, first)
        assert int(rn.plan_dev[ticket]) == 0
    got = rn.out_f64()
    want = oracle_attn(oracle, batch, layer).reshape(got.shape)
    assert np.all(np.abs(got - want) <= 1e-4 + np.abs(want) * {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[out])
