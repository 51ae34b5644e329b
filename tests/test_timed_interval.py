"""What the events of apt_hybrid_decode_attn_timed enclose."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_interval_of_the_absorbed_form_holds_its_last_kernel():
    """1024 requests of one token: the last kernel reads twelve output partials of 12.6 MB each.  Nothing of the call may be left after
    the second event but an empty stream's way to the next one: 4.4 us, with that kernel 22 to 23."""
    from bench import HipEvents
    from paper_2504_07494_amd.harness import DecodeRunner
    print("[case] events around the absorbed form", flush=True)
    B, H = 1024, 24
    cfg = wl.small_config(name="interval", dtype="f16", d_model=128 * H, n_heads=H, head_dim=128, block_size=4, batch=B,
                          len_lo=1, len_hi=4, hidden_ratio=1.0)
    batch = wl.make_batch(cfg, np.full(B, 1, dtype=np.int32), np.full(B, wl.KIND_HIDDEN, dtype=np.uint8))
    rn = DecodeRunner(batch, hidden_impl=ab.APT_HIDDEN_ABSORBED)
    dl = rn.upload(wl.make_layer(batch))
    rn.run(dl)
    ev, after = HipEvents(2), []
    for i in range(6):
        rn.run(dl, ev.pairs[0][0], ev.pairs[0][1])
        assert ev.hip.hipEventRecord(ev.pairs[1][0], ctypes.c_void_p(rn.stream())) == 0
        torch.cuda.synchronize()
        ms = ctypes.c_float()
        assert ev.hip.hipEventElapsedTime(ctypes.byref(ms), ev.pairs[0][1], ev.pairs[1][0]) == 0
        after.append(ms.value * 1e3)
    inside = ev.elapsed_ms(0) * 1e3
    ev.close()
    print(f"[interval] {inside:.1f} us, after it {min(after):.1f} .. {max(after):.1f} us", flush=True)
    assert min(after) < 10.0
