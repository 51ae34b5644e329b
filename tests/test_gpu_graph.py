"""The attention call inside a HIP graph: it launches kernels on the caller's stream only (no
allocation, no synchronisation, no memset nodes), so it can be captured once and replayed.  Every
replay is compared with the eager call on the same inputs, with eager work and synchronisations
between the replays."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl

pytestmark = pytest.mark.gpu

KV, HID = wl.KIND_KV, wl.KIND_HIDDEN


@pytest.mark.parametrize("impl", [ab.APT_HIDDEN_AUTO, ab.APT_HIDDEN_ABSORBED])
def test_captured_attention_call_replays_like_the_eager_call(oracle, impl):
    from paper_2504_07494_amd.harness import DecodeRunner, _to_dev
    print(f"[case] graph capture hidden_impl={impl}", flush=True)
    cfg = wl.small_config(name="graph", dtype="f16", d_model=512, n_heads=4, head_dim=128, block_size=16,
                          batch=6, len_lo=1, len_hi=900, hidden_ratio=0.5)
    batch = wl.make_batch(cfg, np.array([900, 257, 1, 512, 513, 33], dtype=np.int32),
                          np.array([HID, HID, HID, KV, KV, KV], dtype=np.uint8))
    layer = wl.make_layer(batch)
    rn = DecodeRunner(batch, hidden_impl=impl)
    dl = rn.upload(layer)
    rn.run(dl)                                   # eager warm-up (one-off function attributes are set here)
    torch.cuda.synchronize()
    g = np.random.default_rng(3)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    out_graph = torch.empty_like(rn.out)
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            rn.run(dl, out=out_graph)            # uses the capturing stream (torch's current stream)
    torch.cuda.synchronize()
    for rep in range(4):
        q = wl.round_to_dtype(g.standard_normal((batch.B, cfg.n_heads, cfg.head_dim), dtype=np.float32), cfg.dtype)
        dl.q.copy_(_to_dev(q, rn.device))        # new queries in the captured buffer
        eager = rn.run(dl).clone()
        torch.cuda.synchronize()
        out_graph.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_graph, eager), rep
        assert bool(torch.isfinite(out_graph).all())
    # and the last replay against the oracle
    layer.q[...] = q
    from tests.helpers import oracle_attn
    want = oracle_attn(oracle, batch, layer).reshape(batch.B, cfg.n_heads, cfg.head_dim)
    assert np.max(np.abs(out_graph.float().cpu().numpy().astype(np.float64) - want)) < 2e-4


@pytest.mark.parametrize("heads,lens,other,whole", [
    (8, [300, 512, 17] * 5, [511, 2, 90] * 5, True), (24, [300, 512, 17] * 4, [511, 2, 90] * 4, True),   # a range each; 16 waves, 4
    (16, [700, 513, 700, 600] * 4, [520, 1000, 600, 800] * 4, True),                                 # two ranges each
    (12, [1500, 1100, 2000], [1200, 1480, 1990], False)])
def test_captured_call_of_kv_requests_alone_replays_another_plan_of_the_same_counts(heads, lens, other, whole):
    """The plan's upload is captured with the attention call, so a replay serves the plan that the host buffer then holds."""
    from paper_2504_07494_amd.harness import DecodeRunner
    print(f"[case] capture of KV-kind requests alone, {heads} heads {lens}", flush=True)
    top = np.maximum(lens, other).astype(np.int32)
    cfg = wl.small_config(name="graphkv", dtype="f16", d_model=128 * heads, n_heads=heads, head_dim=128, block_size=16,
                          batch=len(lens), len_lo=1, len_hi=2048, hidden_ratio=0.0)
    batch = wl.make_batch(cfg, top, np.zeros(len(lens), dtype=np.uint8))
    rn = DecodeRunner(batch)
    dl = rn.upload(wl.make_layer(batch))
    a, b = (np.array(x, dtype=np.int32) for x in (lens, other))
    eager = {}
    for name, x in (("a", a), ("b", b)):
        rn.plan(x)
        rn.workspace.fill_(255)
        eager[name] = rn.run(dl).clone()
        assert bool((rn.workspace == 255).all()) == whole
    torch.cuda.synchronize()
    host = torch.empty_like(rn.plan_host).pin_memory()
    ab.apt_plan(rn.shape, a, batch.cache_kind, host)
    side, graph, out = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.empty_like(rn.out)
    rn.plan_host = host
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            ab.apt_plan_upload(host, rn.plan_dev, rn.stream())
            rn.run(dl, out=out)
    for x, name in ((a, "a"), (b, "b"), (a, "a"), (b, "b")):
        ab.apt_plan(rn.shape, x, batch.cache_kind, host)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        # (a sum may be associated by another number of waves than the eager call of that plan chose)
        assert float((out - eager[name]).abs().max()) < 1e-5, name


@pytest.mark.parametrize("n_requests", [1, 77, 78, 200])
def test_plan_upload_small_blobs_are_read_at_once_and_captured_ones_at_replay(n_requests):
    """Blobs below, just below (77 requests: 3824 bytes), just above and far above the size that travels with a kernel launch."""
    print(f"[case] plan upload {n_requests}", flush=True)
    shape = ab.make_shape(128, 1, 128, 16, "f16", 8, 1.0)
    lens, kinds = np.full(n_requests, 17, dtype=np.int32), np.zeros(n_requests, dtype=np.uint8)
    kinds[::2] = 1
    host = torch.zeros(ab.apt_plan_max_bytes(shape, n_requests, 128) // 4, dtype=torch.int32, pin_memory=True)
    info = ab.apt_plan(shape, lens, kinds, host)
    n = int(info.plan_bytes) // 4
    assert (info.plan_bytes <= ab.APT_PLAN_INLINE_BYTES) == (n_requests <= 77)
    want = host[:n].clone()
    dev = torch.full((n + 1,), -7, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    ab.apt_plan_upload(host, dev, stream)
    if info.plan_bytes <= ab.APT_PLAN_INLINE_BYTES:
        host.fill_(5)                       # already read
    torch.cuda.synchronize()
    assert torch.equal(dev[:n].cpu(), want) and int(dev[n]) == -7
    host[:n] = want
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        ab.apt_plan_upload(host, dev, side.cuda_stream)
    for value in (1, 2):
        host[17] = value                    # a replay reads the host buffer as it is then
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dev[:n].cpu(), host[:n])


@pytest.mark.parametrize("n_requests", [1, 200])
def test_plan_upload_is_not_disturbed_by_an_error_an_earlier_call_left(n_requests):
    """A failed HIP call of the program leaves its error in the runtime; the upload (small blob: a launch, large blob: a copy)
    reports its own outcome only."""
    print(f"[case] plan upload after an error {n_requests}", flush=True)
    shape = ab.make_shape(128, 1, 128, 16, "f16", 8, 1.0)
    host = torch.zeros(ab.apt_plan_max_bytes(shape, n_requests, 128) // 4, dtype=torch.int32, pin_memory=True)
    info = ab.apt_plan(shape, np.full(n_requests, 17, dtype=np.int32), np.zeros(n_requests, dtype=np.uint8), host)
    n = int(info.plan_bytes) // 4
    dev = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    torch.cuda.synchronize()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    try:
        assert hip.hipSetDevice(9999) != 0            # refused on the host
        ab.apt_plan_upload(host, dev, stream)
    finally:
        hip.hipGetLastError()                         # clears it
    torch.cuda.synchronize()
    assert torch.equal(dev.cpu(), host[:n])
