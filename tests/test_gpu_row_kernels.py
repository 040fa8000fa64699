"""Combine by whole row pieces, and the dispatch index's three block sizes."""
import numpy as np
import pytest
import torch

from paper_2504_01337_amd import workloads as wl
from helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


# rows of one, two and three 2 KB pieces, and ones that are not whole pieces (the other kernel); 1 to 64 slots and one more; few and
# odd token counts; tokens without any local slot, rows that nobody points at hold NaNs
@pytest.mark.parametrize("dtype,T,K,d", [("bf16", 1, 1, 1024), ("bf16", 37, 4, 2048), ("bf16", 5, 64, 1024), ("bf16", 6, 65, 1024),
                                         ("bf16", 9, 3, 3072), ("bf16", 9, 3, 1536), ("f32", 33, 7, 512), ("f32", 3, 2, 1536)])
def test_combine_by_row_pieces(c2r, orc, dtype, T, K, d):
    rng = np.random.default_rng(T + K + d)
    store = wl.round_bf16 if dtype == "bf16" else (lambda a: a)
    A = T * K
    inv = rng.permutation(A).astype(np.int32).reshape(T, K)
    inv[rng.random((T, K)) < 0.4] = -1
    inv[T // 2] = -1
    yp = store(rng.standard_normal((A, d)).astype(np.float32))
    gates = rng.random((T, K)).astype(np.float32)
    ys = store(rng.standard_normal((T, d)).astype(np.float32))
    used = np.zeros(A, dtype=bool)
    used[inv[inv >= 0]] = True
    poisoned = np.where(used[:, None], yp, np.float32(np.nan))
    for shared in (None, ys):
        y = c2r.combine(dev(poisoned, dtype), dev(gates), dev(inv.reshape(-1)), None if shared is None else dev(shared, dtype))
        ref = orc.combine(yp, gates, inv.reshape(-1), T, K, shared)
        # one rounding of the result, and K + 1 of the fp32 sum
        tol = 2.0 ** -8 if dtype == "bf16" else (K + 1) * 2.0 ** -24
        scale = max((np.abs(gates).sum(1).max() + 1) * max(np.abs(yp).max(), np.abs(ys).max()), 1.0)
        assert np.abs(host(y) - ref).max() <= tol * (scale if dtype == "f32" else max(np.abs(ref).max(), 1.0))


# up to 32768 tokens 256 of them per block where the scratch has room, 512 otherwise, and 1024 beyond: scratch of exactly what the
# call asks for and plenty of it
@pytest.mark.parametrize("T,K,n_dev", [(1, 4, 5), (255, 4, 3), (256, 2, 64), (257, 4, 4), (5000, 4, 60), (32768, 4, 4), (32769, 4, 4),
                                       (2000, 9, 7)])
def test_dispatch_index_at_every_block_size(c2r, orc, T, K, n_dev):
    rng = np.random.default_rng(T + n_dev)
    E = 64
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    idx[rng.random((T, K)) < 0.1] = -1
    devmap = rng.integers(-1, n_dev, size=E).astype(np.int32)
    rc, ro, rt, rr = orc.dedup_dispatch(idx, E, devmap, n_dev)
    least = ((T + 1023) // 1024 * n_dev * 4 + 255) // 256 * 256
    assert c2r.workspace_bytes(c2r.STAGE_DEDUP_DISPATCH, T, 0, n_dev, K, 0, c2r.F32) == least
    for ws in (None, torch.empty(least, dtype=torch.uint8, device="cuda"), torch.empty(4 * least, dtype=torch.uint8, device="cuda")):
        if ws is None:
            counts, offsets, tok, row = c2r.dedup_dispatch(dev(idx), E, dev(devmap), n_dev)
        else:
            i32 = dict(dtype=torch.int32, device="cuda")
            counts, offsets = torch.empty(n_dev, **i32), torch.empty(n_dev + 1, **i32)
            tok, row = torch.full((T * K,), -1, **i32), torch.empty(T * K, **i32)
            i, m = dev(idx), dev(devmap)
            p = lambda t: t.data_ptr()
            assert c2r.lib().c2r_dedup_dispatch(p(i), T, K, E, p(m), n_dev, p(counts), p(offsets), p(tok), p(row), p(ws),
                                                ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        n = int(ro[-1])
        assert np.array_equal(host(counts), rc) and np.array_equal(host(offsets), ro)
        assert np.array_equal(host(tok)[:n], rt[:n]) and np.array_equal(host(row).reshape(-1), np.asarray(rr).reshape(-1))


# the dispatch index on either side of its rules (4096 and 524288 assignments), blocks of 1024 assignments and their remainders, one slot,
# all slots, slots shared by experts, empty and out-of-range entries
@pytest.mark.parametrize("T,E,El,K", [(1024, 60, 60, 4), (1025, 60, 60, 4), (4097, 64, 64, 1), (2050, 64, 33, 2), (700, 8, 1, 6), (12289, 60, 15, 4),
                                      (65537, 17, 9, 8), (1366, 3, 3, 3)])
def test_dispatch_index_sizes(orc, T, E, El, K):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    idx = rng.integers(0, E, size=(T, K)).astype(np.int32)
    idx[rng.random((T, K)) < 0.01] = -1
    ls = None if El == E else np.where(np.arange(E) % 3 == 1, -1, np.arange(E) % El).astype(np.int32)
    counts, offsets, perm, inv, _ = c2r.permute(None, dev(idx), E, None if ls is None else dev(ls), El)
    rc, ro, rp, ri = orc.permute(idx, E, ls, El)
    assert np.array_equal(host(counts), rc) and np.array_equal(host(offsets), ro)
    assert np.array_equal(host(perm)[:ro[-1]], rp) and np.array_equal(host(inv), ri)


# the dispatch index in one launch, on either side of its rules (1024, 4096 and 8192 tokens, four devices, four slots) and of its 64-token steps;
# indices that are not 16-byte aligned
@pytest.mark.parametrize("T", [1, 63, 65, 1024, 1025, 2049, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("K,n_dev", [(4, 4), (4, 5), (3, 64), (1, 1), (5, 6)])
def test_dedup_index_in_one_launch(c2r, orc, T, K, n_dev):
    rng = np.random.default_rng(T * 7 + K)
    E = 64
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    idx[rng.random((T, K)) < 0.1] = -1
    idx[T // 3] = E
    devmap = rng.integers(-1, n_dev, size=E).astype(np.int32)
    rc, ro, rt, rr = orc.dedup_dispatch(np.where(idx < E, idx, -1), E, devmap, n_dev)
    n = int(ro[-1])
    for shift in (0, 1):
        i = torch.empty(T * K + shift, dtype=torch.int32, device="cuda")[shift:].view(T, K)
        i.copy_(dev(idx))
        counts, offsets, tok, row = c2r.dedup_dispatch(i, E, dev(devmap), n_dev)
        assert np.array_equal(host(counts), rc) and np.array_equal(host(offsets), ro)
        assert np.array_equal(host(tok)[:n], rt[:n]) and np.all(host(tok)[n:] == -1)
        assert np.array_equal(host(row).reshape(-1), np.asarray(rr).reshape(-1))


# the two-level combine by whole row pieces: one, two and three of them, and rows that are not; 1 to 64 slots and one more (the other kernels); tokens without
# a copy, an expert that is not computed here
@pytest.mark.parametrize("dtype,T,K,d", [("bf16", 1, 1, 1024), ("bf16", 37, 4, 2048), ("bf16", 9, 3, 3072), ("bf16", 3, 64, 1024), ("f32", 33, 7, 512),
                                         ("f32", 5, 2, 1536), ("bf16", 70, 4, 1536), ("bf16", 6, 65, 1024)])
def test_two_level_combine_by_row_pieces(c2r, orc, dtype, T, K, d):
    rng = np.random.default_rng(T + K + d)
    store = wl.round_bf16 if dtype == "bf16" else (lambda a: a)
    E, n_dev = 64, 5
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    idx = np.concatenate([idx, np.full((T, K - idx.shape[1]), -1, dtype=np.int32)], axis=1)  # (no more than E are there)
    idx[T // 2] = -1
    devmap = rng.integers(-1, n_dev, size=E).astype(np.int32)
    inv = rng.permutation(T * K).astype(np.int32)
    inv[rng.random(T * K) < 0.2] = -1
    g = rng.random((T, K)).astype(np.float32)
    yp, ys = (store(rng.standard_normal((n, d)).astype(np.float32)) for n in (T * K, T))
    _, offsets, tok, row = c2r.dedup_dispatch(dev(idx), E, dev(devmap), n_dev)
    _, ro, _, rr = orc.dedup_dispatch(idx, E, devmap, n_dev)
    n = int(ro[-1])
    part = torch.full((T * K, d), float("nan"), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    c2r.combine_partial(dev(yp, dtype), dev(g), dev(inv), tok, row, offsets, part)
    ref = orc.combine_partial(yp, g, inv, rr, T, K, n)
    # one rounding of the result, and K + 1 of the fp32 sum
    tol = 2.0 ** -8 if dtype == "bf16" else (K + 1) * 2.0 ** -24
    bound = lambda r, terms: tol * (max(np.abs(r).max(initial=0.0), 1.0) if dtype == "bf16" else terms)
    assert np.isnan(host(part)[n:]).all()
    if n:
        assert np.abs(host(part)[:n] - ref).max() <= bound(ref, K * np.abs(yp).max())
    for shared in (None, ys):
        y = c2r.combine_copies(part, row, T, K, None if shared is None else dev(shared, dtype))
        ref2 = orc.combine_copies(host(part)[:n], rr, T, K, shared)
        assert np.abs(host(y) - ref2).max() <= bound(ref2, K * max(np.abs(host(part)[:n]).max(initial=0.0), np.abs(ys).max()))


# entries of the send list past its copies: left as they are, or -1, in one launch and in two (one token, two and four per thread)
@pytest.mark.parametrize("T,K,n_dev", [(1, 4, 4), (4096, 4, 4), (4097, 4, 4), (5000, 5, 60), (32769, 3, 7), (40000, 9, 2)])
def test_dedup_list_past_its_copies(c2r, orc, T, K, n_dev):
    rng = np.random.default_rng(T + K)
    E = 60
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    devmap = rng.integers(0, n_dev, size=E).astype(np.int32)
    rt = orc.dedup_dispatch(idx, E, devmap, n_dev)[2]
    i, m, i32 = dev(idx), dev(devmap), dict(dtype=torch.int32, device="cuda")
    p = lambda t: t.data_ptr()
    least = c2r.workspace_bytes(c2r.STAGE_DEDUP_DISPATCH, T, 0, n_dev, K, 0, c2r.F32)
    for call, past in ((c2r.lib().c2r_dedup_dispatch, 123), (c2r.lib().c2r_dedup_dispatch_filled, -1)):
        for ws in (torch.empty(least, dtype=torch.uint8, device="cuda"), torch.empty(4 * least, dtype=torch.uint8, device="cuda")):
            tok = torch.full((T * K + 3,), 123, **i32)
            counts, offsets, row = torch.empty(n_dev, **i32), torch.empty(n_dev + 1, **i32), torch.empty(T * K, **i32)
            assert call(p(i), T, K, E, p(m), n_dev, p(counts), p(offsets), p(tok), p(row), p(ws), ws.numel(),
                        torch.cuda.current_stream().cuda_stream) == 0
            n = int(offsets[-1])
            got = host(tok)
            assert np.array_equal(got[:n], rt[:n]) and np.all(got[n:T * K] == past) and np.all(got[T * K:] == 123)
