"""Absorbed queries of the absorbed-weight hidden path (csrc/apt_absorb16.hip) at the edges of their workgroups: 64 or 128 requests,
16 to a fragment, eight neighbouring heads, 128 rows of W_K; both head widths, whose queries lie in LDS in different orders.

Short contexts: the error of an output is that of its scores, fp32 sums of at most 4416 products of order 1, and of the values, far
below the 2e-4 that the other tests of this path allow."""
import numpy as np
import pytest

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl
from paper_2504_07494_amd.harness import DecodeRunner
from tests.helpers import oracle_attn

pytestmark = pytest.mark.gpu
HID, KV = 1, 0


@pytest.mark.parametrize("dtype,hd,H,n_hid", [
    ("f16", 64, 5, 1), ("bf16", 64, 7, 64), ("bf16", 128, 5, 65), ("f16", 128, 9, 81),      # 64 requests to a workgroup
    ("bf16", 64, 33, 70), ("f16", 64, 33, 129), ("bf16", 128, 24, 128), ("bf16", 64, 69, 15)])   # 128
def test_absorbed_queries_at_workgroup_edges(oracle, dtype, hd, H, n_hid):
    print(f"[case] absorbed queries {dtype} hd={hd} H={H} n={n_hid}", flush=True)
    lens = np.array([1 + 5 * i % 23 for i in range(n_hid)] + [30, 9], dtype=np.int32)
    kinds = np.array([HID] * n_hid + [KV, KV], dtype=np.uint8)
    order = np.random.RandomState(H).permutation(len(lens))          # the hidden-kind requests are not the first ones
    cfg = wl.small_config(name="absorbedq", dtype=dtype, d_model=hd * H, n_heads=H, head_dim=hd, block_size=16, batch=len(lens),
                          len_lo=1, len_hi=30, hidden_ratio=0.5, permute_pages=True)
    batch = wl.make_batch(cfg, lens[order], kinds[order])
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, hidden_impl=ab.APT_HIDDEN_ABSORBED)
    rn.out.fill_(float("nan"))
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    pairs = [(r, h) for r in range(batch.B) for h in sorted({0, min(7, H - 1), H // 2, H - 1})]
    want = oracle_attn(oracle, batch, layer, pairs=pairs).reshape(len(pairs), hd)
    assert np.all(np.isfinite(got))
    err = np.abs(np.stack([got[r, h] for r, h in pairs]) - want)
    print(f"[parity] max_abs={err.max():.3e}", flush=True)
    assert err.max() <= 2e-4
