"""Performance cases of the hybrid-cache decode attention library.

A case is one decode step as a serving loop issues it, through the package's public calls: partition the batch on the
host, copy the plan, one attention call per layer (``DecodeRunner.plan`` / ``run``), where stated with the cache append
of the new token before it; or one prefill cache write.  Lengths and cache kinds belong to the case (``lens_seed``), the
values of all tensors and the placement of the blocks belong to the seed.

Shapes are those of ``workloads.CONFIGS`` (OPT-13B/30B/66B-shaped layers, the fp32 tiny layer) and generic smaller
layers with head_dim 64, which the library takes as well; lengths reach from a few tokens to the 2048-token limit.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2504_07494_amd import binding as ab
from paper_2504_07494_amd import workloads as wl
from paper_2504_07494_amd.harness import DecodeRunner

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
IMPL = {"auto": ab.APT_HIDDEN_AUTO, "absorbed": ab.APT_HIDDEN_ABSORBED}
W_STD = 0.02


def _case(name, what, heads, head_dim, dtype, batch, lo, hi, ratio, **kw):
    c = dict(name=name, what=what, heads=heads, head_dim=head_dim, dtype=dtype, batch=batch, lo=lo, hi=hi, ratio=ratio,
             dist="uniform", block=16, permute=False, impl="auto", out="f32", layers=1, append=False, lens_seed=1)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: the fp32 tiny layer with both kinds, where launches, the plan copy and host time are all there is
        _case("tiny_f32", "decode", 4, 64, "f32", 4, 16, 128, 0.5),
        # one user alone on the server: one KV-kind request, append of the new token, then attention
        _case("one_request_kv", "decode", 40, 128, "f16", 1, 1237, 1237, 0.0, append=True, out="f16"),
        # a nearly idle server under memory pressure: a few short requests, all on the hidden cache
        _case("few_hidden", "decode", 40, 128, "f16", 3, 33, 700, 1.0, append=True, permute=True, out="f16"),
        # the OPT-13B-shaped layer at the batch the headline metric is quoted on, half of the requests hidden-kind
        _case("opt13b_mixed", "decode", 40, 128, "f16", 64, 128, 2048, 0.5),
        # a layer with 64-wide heads (the small members of the model family), half hidden-kind
        _case("heads64_mixed", "decode", 32, 64, "f16", 48, 32, 1024, 0.5, permute=True),
        # lognormal chat-like lengths, mostly hidden cache, scattered pages
        _case("opt30b_chat", "decode", 56, 128, "f16", 128, 32, 2048, 0.7, dist="lognormal", permute=True),
        # plenty of memory: every request on the KV cache (the HBM-bound end)
        _case("opt66b_kv", "decode", 72, 128, "f16", 256, 64, 2048, 0.0),
        # the largest single-layer batch, half hidden-kind (the matrix-bound end; default workload of bench.py)
        _case("opt66b_mixed", "decode", 72, 128, "f16", 256, 64, 2048, 0.5),
        # several layers of one bf16 step: one plan, one attention call per layer
        _case("opt13b_layers_bf16", "decode", 40, 128, "bf16", 384, 256, 1024, 0.5, layers=3, out="bf16"),
        # the absorbed-weight form of the hidden path, asked for by the caller, both 16-bit types
        _case("absorbed_f16", "decode", 40, 128, "f16", 64, 128, 2048, 0.5, impl="absorbed"),
        _case("absorbed_bf16", "decode", 72, 128, "bf16", 96, 64, 2048, 1.0, impl="absorbed", permute=True, out="bf16"),
        # prefill: the prompts' vectors go to the caches, both kinds
        _case("prefill_write", "write", 40, 128, "f16", 16, 61, 1024, 0.5, permute=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: small and large batches, short and long contexts, every kind mix, dtype and
    hidden path, with odd head counts, lengths and block sizes; capped by the work of the largest listed case."""
    family = rng.choice(["small_f32", "few", "batch", "batch", "kv", "heads64", "absorbed", "absorbed", "write"])
    kw = dict(lens_seed=rng.randrange(1 << 30), permute=rng.random() < 0.6, block=rng.choice([16, 16, 16, 8, 32]))
    dtype = rng.choice(["f16", "bf16"])
    out = rng.choice(["f32", dtype])
    ratio = rng.choice([0.25, 0.5, 0.7, 0.75, 1.0])
    hi = _log_int(rng, 64, 2048)
    lo = rng.randint(1, max(1, hi // 3))
    if family == "small_f32":
        c = _case("", "decode", rng.randint(2, 8), rng.choice([64, 128]), "f32", _log_int(rng, 1, 12), 1,
                  rng.randint(17, 300), ratio, **kw)
    elif family == "few":
        c = _case("", "decode", rng.randint(16, 72), 128, dtype, rng.randint(1, 6), lo, hi, rng.choice([0.0, 0.5, 1.0]),
                  append=rng.random() < 0.5, out=out, **kw)
    elif family == "batch":
        c = _case("", "decode", rng.randint(16, 72), 128, dtype, _log_int(rng, 8, 256), lo, hi, ratio,
                  dist=rng.choice(["uniform", "lognormal"]), layers=rng.choice([1, 1, 2]), out=out, **kw)
    elif family == "kv":
        c = _case("", "decode", rng.randint(12, 72), rng.choice([128, 128, 64]), dtype, _log_int(rng, 4, 256), lo, hi, 0.0,
                  out=out, **kw)
    elif family == "heads64":
        c = _case("", "decode", rng.randint(8, 40), 64, dtype, _log_int(rng, 2, 64), lo, min(hi, 1024), ratio, out=out, **kw)
    elif family == "absorbed":
        c = _case("", "decode", rng.randint(16, 72), 128, dtype, _log_int(rng, 4, 192), lo, hi, ratio, impl="absorbed",
                  out=out, **kw)
    else:
        c = _case("", "write", rng.randint(16, 72), 128, dtype, _log_int(rng, 1, 32), lo, min(hi, 1024), rng.choice([0.0, 0.5, 1.0]),
                  **kw)
    del c["name"]
    # no dearer than the largest listed case: 64-wide heads run at a fraction of the matrix rate, so they get less work
    top_flops = 3e11 if (c["head_dim"] == 64 or c["dtype"] == "f32") else 4e13
    while c["batch"] > 1 and (work(c)["flops"] > top_flops or work(c)["bytes"] > 8e9):
        c["batch"] = max(1, c["batch"] * 3 // 4)
    return c


def _meta(c):
    """Lengths, cache kinds and cache maps of a case (host)."""
    d = c["heads"] * c["head_dim"]
    cfg = wl.Config("case", d, c["heads"], c["head_dim"], c["dtype"], c["batch"], c["dist"], c["lo"], c["hi"], c["ratio"],
                    block_size=c["block"], permute_pages=c["permute"], lognormal_median=max(c["lo"], c["hi"] / 4),
                    seed=wl.BASE_SEED + c["lens_seed"])
    return cfg, wl.draw_ctx_lens(cfg), wl.draw_cache_kind(cfg)


def _normal(gen, shape, std, dtype):
    t = torch.empty(shape, dtype=TORCH[dtype], device="cuda")
    t.normal_(0.0, std, generator=gen)
    return t


def prepare(case, seed):
    c = case
    cfg, lens, kinds = _meta(c)
    # the blocks' places in the pool come from the seed; lengths and kinds from the case
    batch = wl.make_batch(wl.replace(cfg, seed=wl.BASE_SEED + seed), lens, kinds)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    d, H, hd, B, e = cfg.d_model, cfg.n_heads, cfg.head_dim, batch.B, c["dtype"]
    pool_shape = (batch.n_pool_blocks, cfg.block_size * d)
    s = SimpleNamespace(what=c["what"], append=c["append"], B=B)
    s.lens_dev = torch.from_numpy(batch.ctx_lens).cuda()
    s.kind_dev = torch.from_numpy(batch.cache_kind).cuda()
    if c["what"] == "write":
        # vectors the prefill of these prompts has produced: x for hidden-kind requests, k and v for the others
        offsets = np.concatenate([[0], np.cumsum(batch.ctx_lens)]).astype(np.int32)
        rows = int(offsets[-1])
        s.shape = ab.make_shape(d, H, hd, cfg.block_size, e, batch.max_blocks, cfg.softmax_scale)
        s.offsets = torch.from_numpy(offsets).cuda()
        s.max_new = int(batch.ctx_lens.max())
        s.x = _normal(gen, (rows, d), 1.0, e) if kinds.max() == wl.KIND_HIDDEN else None
        s.k = _normal(gen, (rows, d), cfg.kv_std, e) if kinds.min() == wl.KIND_KV else None
        s.v = _normal(gen, (rows, d), cfg.kv_std, e) if kinds.min() == wl.KIND_KV else None
        s.tables = torch.from_numpy(batch.block_tables).cuda()
        s.pool = torch.zeros(pool_shape, dtype=TORCH[e], device="cuda")
        return s
    s.runner = DecodeRunner(batch, out_dtype=c["out"], hidden_impl=IMPL[c["impl"]])
    scale = torch.from_numpy(np.where(batch.block_type == 3, 1.0, cfg.kv_std).astype(np.float32)).cuda().to(TORCH[e])
    s.layers, s.outs = [], []
    for _ in range(c["layers"]):
        dl = SimpleNamespace(W_K=None, W_V=None, W_packed=None, b_K=None, b_V=None)
        dl.pool = _normal(gen, pool_shape, 1.0, e)
        dl.pool.mul_(scale[:, None])
        dl.k_pool = dl.v_pool = dl.pool                 # one unified pool
        dl.q = _normal(gen, (B, H, hd), 1.0, e)
        dl.W_K, dl.W_V = _normal(gen, (d, d), W_STD, e), _normal(gen, (d, d), W_STD, e)
        dl.b_K, dl.b_V = _normal(gen, (d,), W_STD, e), _normal(gen, (d,), W_STD, e)
        if s.runner.info.hidden_impl == ab.APT_HIDDEN_MFMA:
            dl.W_packed = torch.empty(ab.apt_packed_weight_bytes(s.runner.shape), dtype=torch.uint8, device="cuda")
            ab.apt_pack_weights(s.runner.shape, dl.W_K, dl.W_V, dl.W_packed, s.runner.stream())
        if c["append"]:
            dl.x_new = _normal(gen, (B, d), 1.0, e)
            dl.k_new, dl.v_new = _normal(gen, (B, d), cfg.kv_std, e), _normal(gen, (B, d), cfg.kv_std, e)
        s.layers.append(dl)
        s.outs.append(torch.empty_like(s.runner.out))
    return s


def run(s):
    if s.what == "write":
        ab.apt_cache_write(s.shape, s.B, s.offsets, s.max_new, s.x, s.k, s.v, s.pool, s.pool, s.pool, s.tables, s.lens_dev,
                           s.kind_dev, torch.cuda.current_stream().cuda_stream)
        return s.pool
    if not s.append:
        s.runner.run_step(s.layers, s.outs)
        return s.outs
    s.runner.plan()
    for dl, out in zip(s.layers, s.outs):
        ab.apt_cache_append(s.runner.shape, s.B, dl.x_new, dl.k_new, dl.v_new, dl.pool, dl.pool, dl.pool,
                            s.runner.block_tables, s.lens_dev, s.kind_dev, s.runner.stream())
        s.runner.run(dl, out=out)
    return [s.outs, [dl.pool for dl in s.layers]]


def work(case):
    """Bytes: every cached vector, weight, query and output once.  Flops: the projections of the hidden-kind tokens
    (4 d^2 each; absorbed form: 4 d H per token and 4 d^2 per request) and the attention itself (4 d per token)."""
    c = case
    cfg, lens, kinds = _meta(c)
    d, H, B = cfg.d_model, cfg.n_heads, len(lens)
    e = wl.ELEM_BYTES[c["dtype"]]
    hid = int(lens[kinds == wl.KIND_HIDDEN].astype(np.int64).sum())
    kv = int(lens.astype(np.int64).sum()) - hid
    n_hid = int((kinds == wl.KIND_HIDDEN).sum())
    if c["what"] == "write":
        return {"bytes": 2.0 * (hid + 2 * kv) * d * e, "flops": 0.0}
    by = (hid + 2 * kv) * d * e + B * d * (e + wl.ELEM_BYTES[c["out"]])
    fl = 4.0 * d * kv
    if n_hid:
        by += 2 * d * d * e + 2 * d * e
        fl += (4.0 * d * H * hid + 4.0 * d * d * n_hid) if c["impl"] == "absorbed" else (4.0 * d * d + 4.0 * d) * hid
    if c["append"]:
        by += 2 * (n_hid + 2 * (B - n_hid)) * d * e
    return {"bytes": float(by) * c["layers"], "flops": fl * c["layers"]}


def tolerance(case):
    """fp32 accumulation throughout.  Measured between two orders of the same sums (the two hidden paths, two KV range
    lengths): fp32 outputs 1.2e-6 of their norm, 1.7e-5 at most; 16-bit outputs differ by one step of the last rounding
    where a value lies at a tie (f16 2.1e-5 and 9.7e-4, bf16 7.7e-5 and 7.8e-3).  Stated: four times that."""
    if case["what"] == "write":
        return "exact"
    if case["out"] == "f16":
        return {"rel": 8e-5, "max": 4e-3}
    if case["out"] == "bf16":
        return {"rel": 3e-4, "max": 3.2e-2}
    return {"rel": 5e-6, "max": 7e-5}
