"""Absorbed-weight path, 16-bit inputs: the rule for the passes that read the hidden rows past the caches (csrc/apt_internal.h), and a batch on
either side of it."""
import os
import subprocess

import numpy as np
import pytest

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl
from tests.helpers import oracle_attn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCORES, SUMS = 1, 2


def _past(tmp_path, batches):
    """The rule, compiled for the host, for (heads of 128, type, hidden-kind requests, their tokens)."""
    src, exe = tmp_path / "past.cpp", tmp_path / "past"
    src.write_text("""
#include <stdio.h>
#include "apt_internal.h"
int main() {
    long long q, x;
    while (scanf("%lld %lld", &q, &x) == 2) printf("%d\\n", apt_absorbed_past(q, x));
}
""")
    subprocess.run(["g++", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2504_07494_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    lines = []
    for H, dtype, n, tokens in batches:
        frags = max(2, -(-H // 16))
        rows = 16 * (8 if frags == 7 else frags) * {"f16": 2, "bf16": 3}[dtype]
        lines.append(f"{n * rows * H * 128 * 2} {tokens * H * 128 * 2}")
    out = subprocess.run([str(exe)], input="\n".join(lines), text=True, capture_output=True, check=True).stdout
    return [int(v) for v in out.split()]


def test_hidden_rows_that_fit_stay_in_the_caches(tmp_path):
    small = [(H, t, n, n * m) for H in (1, 17, 40, 72, 128) for t in ("f16", "bf16") for n in (1, 3, 6) for m in (1, 300, 600)]
    got = _past(tmp_path, small)
    for (H, t, n, tokens), past in zip(small, got):
        x = tokens * H * 256
        assert past == (SUMS if x > 16 << 20 else 0), (H, t, n, tokens)
    # a working set that the memory-side cache holds, and rows of up to twice that beside small queries, are read through it by the scores
    assert _past(tmp_path, [(40, "f16", 32, 9600), (40, "f16", 32, 34816), (24, "bf16", 150, 32250)]) == [SUMS] * 3
    assert _past(tmp_path, [(62, "bf16", 77, 15400), (48, "bf16", 150, 10500), (56, "f16", 100, 11000)]) == [SUMS | SCORES] * 3
    assert _past(tmp_path, [(16, "f16", 180, 216000), (72, "bf16", 96, 101376)]) == [SUMS | SCORES] * 2


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,H,n_hid,lo,hi,past", [
    ("bf16", 48, 110, 50, 120, SUMS | SCORES), ("f16", 65, 70, 60, 200, SUMS | SCORES), ("f16", 33, 20, 90, 300, SUMS),
    ("bf16", 17, 9, 30, 700, 0)])
def test_both_sides_of_the_rule_against_the_oracle(oracle, tmp_path, dtype, H, n_hid, lo, hi, past):
    # errors of the scores and of the value sums as in the other tests of this path
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] hidden rows past the caches {dtype} heads={H} n={n_hid}", flush=True)
    lens = np.random.default_rng(H).integers(lo, hi + 1, size=n_hid).astype(np.int32)
    assert _past(tmp_path, [(H, dtype, n_hid, int(lens.sum()))]) == [past]
    cfg = wl.small_config(name="abcaches", dtype=dtype, d_model=128 * H, n_heads=H, head_dim=128, block_size=16, batch=n_hid,
                          len_lo=lo, len_hi=hi, hidden_ratio=1.0, permute_pages=True)
    batch = wl.make_batch(cfg, lens, np.full(n_hid, wl.KIND_HIDDEN, dtype=np.uint8))
    layer = wl.make_layer(batch, workers=16)
    rn = DecodeRunner(batch, hidden_impl=ab.APT_HIDDEN_ABSORBED)
    rn.out.fill_(float("nan"))
    rn.run(rn.upload(layer))
    got = rn.out_f64()
    pairs = [(0, 0), (1, H - 1), (n_hid // 2, H // 2), (n_hid - 1, H - 1), (int(np.argmax(lens)), 3), (int(np.argmin(lens)), 5)]
    want = oracle_attn(oracle, batch, layer, pairs=pairs).reshape(len(pairs), 128)
    err = np.abs(np.stack([got[r, h] for r, h in pairs]) - want)
    print(f"[parity] max_abs={err.max():.3e}", flush=True)
    assert np.all(np.isfinite(got)) and err.max() <= 2e-4
