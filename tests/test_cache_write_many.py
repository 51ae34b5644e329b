"""Cache write of more requests than a grid dimension holds (65 535): the kernel's workgroups then take several each.  And the
largest run of new tokens that a call takes."""
import numpy as np
import pytest

from paper_2504_07494_amd import binding as ab


@pytest.mark.gpu
@pytest.mark.parametrize("B,hidden_only", [(65536, False), (131107, False), (65535 + 64, True)])
def test_every_request_is_written_once(B, hidden_only):
    import torch
    print(f"[case] cache write of {B} requests, hidden_only={hidden_only}", flush=True)
    bs, d = 8, 64                                     # one head: a K or V block is [slot][64], as a hidden one
    g = np.random.default_rng(B)
    lens = g.integers(1, bs + 1, size=B).astype(np.int32)
    n_new = g.integers(0, lens + 1).astype(np.int32)
    kinds = np.ones(B, dtype=np.uint8) if hidden_only else g.integers(0, 2, size=B).astype(np.uint8)
    tables = g.permutation(2 * B).astype(np.int32).reshape(B, 2, 1)
    off = np.concatenate([[0], np.cumsum(n_new)]).astype(np.int32)
    x, k, v = (g.integers(1, 30000, size=(int(off[-1]), d)).astype(np.int16) for _ in range(3))
    want = np.zeros((2 * B, bs, d), dtype=np.int16)
    req = np.repeat(np.arange(B), n_new)
    slot = np.arange(off[-1]) - off[req] + lens[req] - n_new[req]
    hid = kinds[req] == 1
    want[tables[req[hid], 0, 0], slot[hid]] = x[hid]
    want[tables[req[~hid], 0, 0], slot[~hid]] = k[~hid]
    want[tables[req[~hid], 1, 0], slot[~hid]] = v[~hid]
    shape = ab.make_shape(d, 1, 64, bs, "f16", 1, 1.0)
    pool = torch.zeros((2 * B, bs, d), dtype=torch.int16, device="cuda:0")
    dev = [torch.from_numpy(a).cuda() for a in (off, x, k, v, tables, lens, kinds)]
    if hidden_only:
        dev[2] = dev[3] = None
    ab.apt_cache_write(shape, B, dev[0], bs, dev[1], dev[2], dev[3], pool, pool, pool, dev[4], dev[5], dev[6],
                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(pool.cpu().numpy(), want)


@pytest.mark.gpu
def test_largest_run_of_new_tokens():
    """524280 new tokens size the grid, one more is refused; a request here has three."""
    import torch
    print("[case] cache write, largest max_new_tokens", flush=True)
    shape = ab.make_shape(64, 1, 64, 8, "f16", 1, 1.0)
    pool = torch.zeros((1, 8, 64), dtype=torch.int16, device="cuda:0")
    x = torch.arange(1, 3 * 64 + 1, dtype=torch.int16, device="cuda:0").reshape(3, 64)
    dev = [torch.tensor(a, dtype=t, device="cuda:0") for a, t in (([0, 3], torch.int32), ([[[0], [0]]], torch.int32), ([3], torch.int32), ([1], torch.uint8))]
    stream = torch.cuda.current_stream().cuda_stream
    with pytest.raises(ab.AptError) as e:
        ab.apt_cache_write(shape, 1, dev[0], 524281, x, None, None, pool, pool, pool, *dev[1:], stream)
    assert e.value.status == ab.APT_ERANGE
    ab.apt_cache_write(shape, 1, dev[0], 524280, x, None, None, pool, pool, pool, *dev[1:], stream)
    torch.cuda.synchronize()
    assert torch.equal(pool[0, :3], x) and int(pool[0, 3:].abs().sum()) == 0
