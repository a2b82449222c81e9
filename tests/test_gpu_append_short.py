"""flux_kv_append / flux_kv_append_ring where the launch changes its kernel or a workgroup is not full: batches on both sides of
64, the whole cache bit for bit (it is a copy) against rows placed one after the other, through several calls."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_07394_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctx(F):
    c = F.flux_create(0, 0)
    yield c
    F.flux_destroy(c)


def test_long_copies_of_few_sequences(F, ctx):
    """More workgroups than are resident at once, which count themselves on several words; a row past the capacity is left out."""
    hkv, d, lens, new, cap = 8, 64, [3, 0, 70], [40000, 1, 9000], 40001
    g = torch.Generator(device="cuda").manual_seed(3)
    total = sum(new)
    kn, vn = (torch.randint(-30000, 30000, (total, hkv, d), generator=g, device="cuda", dtype=torch.int16) for _ in range(2))
    k, v = (torch.zeros(3, hkv, cap, d, dtype=torch.int16, device="cuda") for _ in range(2))
    cache = F.KVCache(k.view(torch.bfloat16), v.view(torch.bfloat16), torch.tensor(lens, dtype=torch.int32, device="cuda"))
    cu = torch.tensor([0, 40000, 40001, total], dtype=torch.int32, device="cuda")
    F.flux_last_device_status(ctx)
    F.flux_kv_append(ctx, cache, hkv, d, kn.view(torch.bfloat16), vn.view(torch.bfloat16), cu, total, max(new))
    for got, rows in ((k, kn), (v, vn)):
        want, t = torch.zeros_like(got), 0
        for b in range(3):
            n = min(new[b], cap - lens[b])
            want[b, :, lens[b]:lens[b] + n] = rows[t:t + n].transpose(0, 1)
            t += new[b]
        assert torch.equal(got, want)
    assert cache.kv_len.tolist() == [min(cap, a + b) for a, b in zip(lens, new)]
    assert F.flux_last_device_status(ctx) & F.FLUX_DEV_KV_OVERFLOW


@pytest.mark.parametrize("ring", [False, True])
@pytest.mark.parametrize("hkv,d", [(8, 128), (3, 64), (40, 128)])
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65])
def test_append_places_every_row(F, ctx, batch, hkv, d, ring):
    rng = np.random.default_rng(batch * 100 + hkv)
    n_sink, window = 5, 32
    cap = n_sink + window if ring else 61 if batch > 1 else 301
    lens = rng.integers(0, 12, batch).astype(np.int32)
    k, v = (torch.zeros(batch, hkv, cap, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    cache = F.KVCache(k, v, torch.from_numpy(lens).cuda())
    want_k, want_v = np.zeros((2, batch, cap, hkv, d), np.int16)
    overflow = False
    for call in range(3):
        new = rng.integers(0, 24, batch)
        new[batch // 2] = 0 if batch > 1 and call == 0 else 40 if batch > 1 else 90 + call
        total = int(new.sum())
        rows = rng.integers(-30000, 30000, (2, total, hkv, d)).astype(np.int16)
        kn, vn = (torch.from_numpy(r).cuda().view(torch.bfloat16) for r in rows)
        cu = torch.from_numpy(np.concatenate([[0], np.cumsum(new)]).astype(np.int32)).cuda()
        if ring:
            F.flux_kv_append_ring(ctx, cache, hkv, d, n_sink, window, kn, vn, cu, total, int(new.max()))
        else:
            F.flux_kv_append(ctx, cache, hkv, d, kn, vn, cu, total, int(new.max()))
        t = 0
        for b in range(batch):
            for pos in range(lens[b], lens[b] + new[b]):
                row = pos if not ring or pos < n_sink else n_sink + (pos - n_sink) % window
                overflow |= row >= cap
                if row < cap:
                    want_k[b, row], want_v[b, row] = rows[0, t], rows[1, t]
                t += 1
            lens[b] += new[b]
            if not ring:
                lens[b] = min(lens[b], cap)
        assert np.array_equal(cache.kv_len.cpu().numpy(), lens), call
        for got, want in ((k, want_k), (v, want_v)):
            assert np.array_equal(got.view(torch.int16).cpu().numpy().transpose(0, 2, 1, 3), want), call
    assert bool(F.flux_last_device_status(ctx) & F.FLUX_DEV_KV_OVERFLOW) == overflow


@pytest.mark.parametrize("lens,new,hkv", [([3], [20000], 8), ([700], [8190], 8), ([0, 5000], [9000, 3], 5), ([1, 4], [30000, 800], 8), ([9, 0, 40, 2], [3000, 65, 64, 4097], 17), ([3, 0, 70], [20000, 30, 64], 16)])
def test_long_ring_appends_keep_the_sinks_and_the_window(F, ctx, lens, new, hkv):
    """Many workgroups, most of whose rows are dropped: what stays is the sinks and the last 64 rows of every sequence."""
    d, n_sink, window, batch = 64, 7, 64, len(lens)
    g = torch.Generator(device="cuda").manual_seed(sum(new))
    kn, vn = (torch.randint(-30000, 30000, (sum(new), hkv, d), generator=g, device="cuda", dtype=torch.int16) for _ in range(2))
    k, v = (torch.zeros(batch, hkv, n_sink + window + 2, d, dtype=torch.int16, device="cuda") for _ in range(2))
    cache = F.KVCache(k.view(torch.bfloat16), v.view(torch.bfloat16), torch.tensor(lens, dtype=torch.int32, device="cuda"))
    cu = torch.tensor(np.concatenate([[0], np.cumsum(new)]), dtype=torch.int32, device="cuda")
    F.flux_kv_append_ring(ctx, cache, hkv, d, n_sink, window, kn.view(torch.bfloat16), vn.view(torch.bfloat16), cu, sum(new), max(new))
    for got, rows in ((k, kn), (v, vn)):
        want, t = torch.zeros_like(got), 0
        for b in range(batch):
            for r in list(range(min(n_sink, new[b]))) + list(range(max(0, new[b] - window), new[b])):
                pos = lens[b] + r
                if pos < n_sink or pos >= lens[b] + new[b] - window:
                    want[b, :, pos if pos < n_sink else n_sink + (pos - n_sink) % window] = rows[t + r]
            t += new[b]
        assert torch.equal(got, want)
    assert cache.kv_len.tolist() == [a + n for a, n in zip(lens, new)]
    assert F.flux_last_device_status(ctx) == 0


def test_more_rows_than_a_launch_has_threads_for(F, ctx):
    """2^24 rows of more than 128 pieces of 16 bytes, of which a ring keeps 71: a thread per piece would be 2^32 threads."""
    hkv, d, n, n_sink, window = 17, 64, 1 << 24, 7, 64
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("the rows take 36.5 GB")
    rows = torch.empty(n, hkv, d, dtype=torch.bfloat16, device="cuda")
    for part in (rows[:n_sink], rows[-window:]):
        part.copy_(torch.randint(-99, 99, part.shape, device="cuda"))
    cu = torch.tensor([0, n, n, n], dtype=torch.int32, device="cuda")
    for batch in (1, 3):
        cache = F.KVCache(*(torch.zeros(batch, hkv, n_sink + window, d, dtype=torch.bfloat16, device="cuda") for _ in range(2)),
                          torch.zeros(batch, dtype=torch.int32, device="cuda"))
        F.flux_kv_append_ring(ctx, cache, hkv, d, n_sink, window, rows, rows, cu[:batch + 1], n, n)
        assert cache.kv_len.tolist() == [n, 0, 0][:batch]
        want = torch.cat([rows[:n_sink], rows[-window:].roll((n - window - n_sink) % window, 0)]).transpose(0, 1)
        for got in (cache.k, cache.v):
            assert torch.equal(got[0], want) and not got[1:].any()
    del rows
    torch.cuda.empty_cache()
