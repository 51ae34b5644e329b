"""Raw weights, 64-wide heads: ranges around the edges of the 64-, 128-, 192- and 256-row tiles, against the oracle.  fp32 sums of at most 256
products and 256 weights: errors a few hundred times 2^-24 of the values' size, 1e-4 is ten times that (as for the merges)."""
import numpy as np
import pytest

from paper_2504_07494_amd import workloads as wl
from paper_2504_07494_amd.harness import DecodeRunner
from tests.helpers import oracle_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H", [("f16", 4), ("bf16", 3)])
def test_ranges_around_the_edges_of_the_tiles(oracle, dtype, H):
    print(f"[case] raw tiles {dtype} heads={H}", flush=True)
    lens = np.array([1, 63, 64, 65, 127, 128, 129, 160, 191, 192, 193, 255, 256, 257, 256 + 129, 512 + 192], dtype=np.int32)
    cfg = wl.small_config(name="rawtiles", dtype=dtype, d_model=64 * H, n_heads=H, head_dim=64, block_size=8, batch=len(lens),
                          len_lo=1, len_hi=int(lens.max()), hidden_ratio=1.0, permute_pages=True)
    batch = wl.make_batch(cfg, lens, np.full(len(lens), wl.KIND_HIDDEN, dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, hidden_chunk=256)
    rn.out.fill_(float("nan"))
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    want = oracle_attn(oracle, batch, layer).reshape(got.shape)
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - want)) <= 1e-4
