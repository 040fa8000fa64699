"""Router and dispatch index of small batches: the partial sums on 16 x 16 x 4 matrix instructions (bit-exact logits in the
declared order) and, inside the layer call, selection and index in one launch (what the separate stages give, bit for bit)."""
import numpy as np
import pytest
import torch

from paper_2504_01337_amd import workloads as wl
from helpers import GATE_RTOL, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


# token tiles of 16, 32 and 64 (by the expert count) and their remainders; expert blocks of 16 and their remainders, rows of W_g
# that are no whole 16-byte vectors; chunks of 256, shorter ones and ragged last ones; and the first batches past the rule, which
# take the other kernel (12289 tokens of one chunk, 1537 and 3073 tokens of 16 and 8)
@pytest.mark.parametrize("T,E,d,dtype", [
    (1, 60, 2048, "bf16"), (15, 64, 256, "bf16"), (17, 61, 520, "bf16"), (33, 33, 264, "f32"), (31, 32, 8, "bf16"),
    (65, 17, 1032, "f32"), (64, 16, 512, "bf16"), (63, 3, 24, "f32"), (130, 9, 1000, "bf16"), (1000, 8, 256, "f32"), (2, 1, 16, "bf16"),
    (3072, 34, 2048, "bf16"), (3088, 34, 2048, "bf16"), (12288, 5, 264, "f32"), (12289, 5, 264, "f32"), (12289, 20, 248, "bf16")])
def test_small_route_logits_bit_exact(c2r, orc, T, E, d, dtype):
    rng = np.random.default_rng(T + E + d)
    x = rng.standard_normal((T, d)).astype(np.float32) * np.exp2(rng.integers(-6, 7, size=(T, 1))).astype(np.float32)
    x = wl.round_bf16(x) if dtype == "bf16" else x
    Wg = rng.standard_normal((d, E)).astype(np.float32)
    bias = rng.standard_normal(E).astype(np.float32)
    K = min(E, 4)
    idx, gates, logits = c2r.route(dev(x, dtype), dev(Wg), dev(bias), K, None, want_logits=True)
    ref = orc.logits_canon_f32(x, Wg, bias)
    assert np.array_equal(host(logits), ref)
    ri, rg = orc.route(ref, K)
    assert np.array_equal(host(idx), ri)
    # logits of up to 64 sqrt(d) here: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero
    np.testing.assert_allclose(host(gates), rg, rtol=114 / 34 * GATE_RTOL, atol=1e-37)


# one workgroup's selection and index: 1 to 64 tokens, up to 1024 assignments (64 x 16), and the first calls past either limit;
# lists that cannot fill the slots, NaN and infinite logits, experts that are not local
@pytest.mark.parametrize("T,E,K,El,dtype", [(1, 60, 4, 60, "bf16"), (64, 60, 4, 15, "bf16"), (65, 60, 4, 15, "bf16"), (64, 64, 16, 64, "bf16"),
                                            (61, 64, 17, 30, "bf16"), (5, 3, 3, 3, "f32"), (63, 17, 1, 9, "f32"), (37, 8, 2, 8, "f32"),
                                            # at the start of the gate/up pass: up to 16 tokens, 32 assignments, two per expert; the first calls past
                                            # each; the index of 128 assignments and of one more
                                            (16, 16, 2, 16, "bf16"), (16, 17, 1, 8, "bf16"), (17, 64, 1, 64, "bf16"), (1, 64, 32, 64, "bf16"),
                                            (1, 64, 33, 64, "bf16"), (3, 40, 9, 20, "bf16"), (7, 60, 4, 60, "bf16"), (2, 60, 4, 4, "bf16"),
                                            (4, 5, 3, 2, "bf16"), (32, 60, 4, 60, "bf16"), (43, 60, 3, 31, "bf16")])
def test_layer_call_of_a_small_batch_routes_like_the_stages(c2r, T, E, K, El, dtype):
    _layer_call_routes_like_the_stages(c2r, T, E, K, El, dtype, 64)


# selection, index and rows in one launch: up to 1024 tokens, 16 experts, 4 slots and 128 KB of chunk results (16 experts, d 4096: 128 tokens), and the
# first calls past each; one and several chunks, rows of one and several vectors per lane
@pytest.mark.parametrize("T,E,K,El,dtype,d", [
    (65, 16, 4, 16, "bf16", 64), (128, 16, 4, 7, "bf16", 4096), (129, 16, 4, 7, "bf16", 4096), (1024, 8, 2, 8, "f32", 256), (1025, 8, 2, 8, "f32", 256),
    (512, 16, 3, 5, "f32", 520), (513, 5, 5, 5, "f32", 64), (70, 17, 4, 17, "f32", 64), (3, 8, 2, 8, "f32", 2056), (1, 2, 1, 2, "f32", 8), (67, 1, 1, 1, "f32", 24),
    (999, 13, 4, 2, "bf16", 264)])
def test_selection_index_and_rows_in_one_launch(c2r, T, E, K, El, dtype, d):
    _layer_call_routes_like_the_stages(c2r, T, E, K, El, dtype, d)


def _layer_call_routes_like_the_stages(c2r, T, E, K, El, dtype, d):
    rng = np.random.default_rng(T * E + K)
    F = 64
    w = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), dtype)
    ls = None
    if El < E:
        ls = np.full(E, -1, dtype=np.int32)
        ls[rng.permutation(E)[:El]] = rng.permutation(El).astype(np.int32)
    lists = rng.integers(-1, E + 2, size=(E, max(K, 2))).astype(np.int32)  # duplicates, the expert itself, out of range
    bias = rng.standard_normal(E).astype(np.float32)
    if E > 8:
        bias[[2, 7]] = np.nan, np.inf
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16 if dtype == "bf16" else torch.float32,
                         dev(rng.standard_normal((d, E)).astype(np.float32)), dev(bias), dev(lists), w(El, F, d), w(El, F, d),
                         w(El, d, F), local_slot=dev(ls), E_local=El)
    x = w(T, d)
    layer.forward(x)
    idx, gates, _ = c2r.route(x, layer.Wg, layer.bias, K, layer.collab_idx)
    counts, offsets, perm, inv, rows = c2r.permute(x, idx, E, layer.local_slot, El)
    torch.cuda.synchronize()
    assert torch.equal(layer.idx, idx) and torch.equal(layer.gates.view(torch.int32), gates.view(torch.int32))
    assert torch.equal(layer.counts, counts) and torch.equal(layer.offsets, offsets) and torch.equal(layer.inv_perm, inv)
    n = int(offsets[-1])
    assert torch.equal(layer.perm[:n], perm[:n]) and bool((layer.perm[n:] == -1).all())
    if layer.x_perm is not None:
        assert torch.equal(layer.x_perm[:n], rows[:n])


# the same with lists of distinct experts and logits that spread the tokens over all of them, whose gates are numbers, and with NaNs and
# infinities in the logits of some tokens only (both forms of the scan in one batch)
@pytest.mark.parametrize("T,E,K,El,dtype,d", [
    (1, 60, 4, 60, "bf16", 64), (16, 16, 2, 16, "bf16", 64), (8, 60, 4, 60, "bf16", 64), (10, 40, 3, 20, "bf16", 64), (32, 60, 4, 60, "bf16", 64), (43, 60, 3, 31, "bf16", 64),
    (64, 60, 4, 15, "bf16", 64), (64, 64, 16, 64, "bf16", 64), (61, 64, 17, 30, "bf16", 64), (63, 17, 2, 9, "f32", 64),
    (65, 16, 4, 16, "bf16", 64), (128, 16, 4, 7, "bf16", 4096), (1024, 8, 2, 8, "f32", 256), (512, 16, 3, 5, "f32", 520), (999, 13, 4, 2, "bf16", 264)])
def test_layer_call_routes_like_the_stages_over_all_experts(c2r, T, E, K, El, dtype, d):
    rng = np.random.default_rng(T * E + K)
    w = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), dtype)
    ls = None
    if El < E:
        ls = np.full(E, -1, dtype=np.int32)
        ls[rng.permutation(E)[:El]] = rng.permutation(El).astype(np.int32)
    lists = np.stack([rng.permutation(np.delete(np.arange(E), e))[:min(K + 3, E - 1)] for e in range(E)]).astype(np.int32)
    layer = c2r.C2RLayer(T, d, E, K, 64, torch.bfloat16 if dtype == "bf16" else torch.float32, dev(rng.standard_normal((d, E)).astype(np.float32)),
                         dev((rng.standard_normal(E) * 0.1).astype(np.float32)), dev(lists), w(El, 64, d), w(El, 64, d), w(El, d, 64),
                         local_slot=dev(ls), E_local=El)
    finite = rng.standard_normal((T, d)).astype(np.float32)
    mixed = finite.copy()
    mixed[1::5, 0] = np.inf    # logits of both infinities
    mixed[3::7, 1] = np.nan    # NaN throughout
    for x in (finite, mixed):
        x = dev(x, dtype)
        layer.perm.fill_(-1)
        layer.forward(x)
        idx, gates, _ = c2r.route(x, layer.Wg, layer.bias, K, layer.collab_idx)
        counts, offsets, perm, inv, rows = c2r.permute(x, idx, E, layer.local_slot, El)
        assert torch.equal(layer.idx, idx) and torch.equal(layer.gates.view(torch.int32), gates.view(torch.int32))
        assert torch.equal(layer.counts, counts) and torch.equal(layer.offsets, offsets) and torch.equal(layer.inv_perm, inv)
        n = int(offsets[-1])
        assert torch.equal(layer.perm[:n], perm[:n]) and bool((layer.perm[n:] == -1).all())
        if layer.x_perm is not None:
            assert torch.equal(layer.x_perm[:n].view(torch.int16 if dtype == "bf16" else torch.int32), rows[:n].view(torch.int16 if dtype == "bf16" else torch.int32))
        if x.isfinite().all():
            assert bool(gates.isfinite().all()) and bool((idx >= 0).all())
            assert len(torch.unique(idx[:, 0])) >= min(T, E) // 2 and int((counts > 0).sum()) >= min(T * K * El // E, El) // 2


# the expert FFN of such a batch: every gate/up workgroup selects for itself, and its rows and their places are what it found.  One to 16 tokens,
# on either side of 2304 workgroups (72 and 76 column blocks of 32 rows), of 32 assignments and of 8 tokens beside a shared expert
@pytest.mark.parametrize("T,E,K,El,F,Fs", [
    (1, 60, 4, 60, 704, 0), (1, 60, 4, 60, 704, 1408), (3, 60, 4, 60, 64, 320), (7, 60, 4, 15, 128, 0), (2, 60, 4, 4, 64, 64), (8, 60, 4, 60, 704, 1408), (8, 60, 4, 60, 1152, 0),
    (8, 60, 4, 60, 1216, 0), (16, 16, 2, 16, 704, 0), (9, 32, 3, 32, 128, 320), (11, 20, 3, 20, 128, 0), (8, 32, 4, 32, 128, 320), (5, 20, 4, 20, 72, 0)])
def test_expert_ffn_of_the_smallest_batches(c2r, T, E, K, El, F, Fs):
    rng = np.random.default_rng(T + E + F)
    d = 128
    w = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), "bf16")
    ls = None
    if El < E:
        ls = np.full(E, -1, dtype=np.int32)
        ls[rng.permutation(E)[:El]] = rng.permutation(El).astype(np.int32)
    lists = np.stack([rng.permutation(np.delete(np.arange(E), e))[:K + 3] for e in range(E)]).astype(np.int32)
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, w(d, E).float(), None, dev(lists), w(El, F, d), w(El, F, d), w(El, d, F), local_slot=dev(ls),
                         E_local=El, shared=(w(1, Fs, d), w(1, Fs, d), w(1, d, Fs)) if Fs else None)
    assert layer.fuse_shared == bool(Fs) and layer.x_perm is None
    for _ in range(3):
        x = w(T, d)
        results = []
        for kw in ({"trace": {}}, {}):
            for t in (layer.y, layer.y_perm, layer.y_shared, layer.h, layer.__dict__.get("h_shared"), layer.__dict__.get("ws_ffn")):
                if t is not None:
                    t.view(torch.uint8).fill_(255)
            y = layer.forward(x, **kw).clone()
            n = int(layer.offsets[-1])
            results.append((y, layer.y_perm[:n].clone(), layer.idx.clone()) + ((layer.y_shared.clone(),) if Fs else ()))
        assert bool(results[0][0].isfinite().all()) and all(torch.equal(a, b) for a, b in zip(*results))


# K = 1 takes lists of no entries (Tc >= K - 1); the array then holds nothing that may be read, also where it is not NULL.  (The pointer
# lies inside an allocation here.)  Batches of the two routers, and the one-launch selection and index of the layer call.
@pytest.mark.parametrize("T,E,d,dtype", [(1, 60, 256, "bf16"), (70, 8, 64, "f32"), (12289, 5, 264, "f32")])
def test_lists_without_entries(c2r, orc, T, E, d, dtype):
    rng = np.random.default_rng(T + E)
    x = rng.standard_normal((T, d)).astype(np.float32)
    x = wl.round_bf16(x) if dtype == "bf16" else x
    Wg = rng.standard_normal((d, E)).astype(np.float32)
    xd, Wd, lists = dev(x, dtype), dev(Wg), torch.full((64,), 3, dtype=torch.int32, device="cuda")
    idx, gates = torch.empty((T, 1), dtype=torch.int32, device="cuda"), torch.empty((T, 1), dtype=torch.float32, device="cuda")
    dt = c2r.BF16 if dtype == "bf16" else c2r.F32
    ws = torch.empty(max(256, c2r.workspace_bytes(c2r.STAGE_ROUTE, T, d, E, 1, 0, dt)), dtype=torch.uint8, device="cuda")
    empty = lists.data_ptr() + 128
    assert c2r.lib().c2r_route(xd.data_ptr(), dt, Wd.data_ptr(), None, T, d, E, 1, empty, 0, idx.data_ptr(), gates.data_ptr(), None,
                               ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == c2r.OK
    torch.cuda.synchronize()
    ri, rg = orc.route(orc.logits_canon_f32(x, Wg, None), 1)
    assert np.array_equal(host(idx), ri) and np.array_equal(host(gates), rg.astype(np.float32))
    w = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), dtype)
    layer = c2r.C2RLayer(T, d, E, 1, 64, xd.dtype, Wd, None, None, w(E, 64, d), w(E, 64, d), w(E, d, 64))
    y = layer.forward(xd).clone()
    fields = list(layer._LAYER.unpack(layer._args()))
    assert fields[6] == 0 and fields[12] == 0                          # Tc, collab_idx
    fields[12] = empty
    layer.idx.fill_(-7)
    assert c2r.lib().c2r_layer_forward(layer._LAYER.pack(*fields), xd.data_ptr(), torch.cuda.current_stream().cuda_stream) == c2r.OK
    torch.cuda.synchronize()
    assert np.array_equal(host(layer.idx), ri) and torch.equal(layer.y, y)


# selection with sixteen tokens per workgroup: remainders of a tile, lists shorter and longer than a thread requests ahead, more slots
# than a token has lanes, special values, and the first batch that goes back to the 64-token kernel
@pytest.mark.parametrize("T,E,K,Tc", [(1, 64, 4, 16), (65, 60, 4, 16), (79, 64, 16, 63), (80, 64, 17, 40), (33, 63, 40, 62), (100, 5, 1, 3),
                                      (129, 17, 2, 17), (8192, 36, 4, 9), (8193, 36, 4, 9)])
def test_small_selection_against_oracle(c2r, orc, T, E, K, Tc):
    rng = np.random.default_rng(T + E * K)
    x = rng.standard_normal((T, 64)).astype(np.float32)
    Wg = np.round(rng.standard_normal((64, E)) * 2).astype(np.float32) / 4
    bias = rng.standard_normal(E).astype(np.float32)
    if E > 8:
        bias[[2, 7]] = np.nan, -np.inf
    # Tc entries with the expert itself and a duplicate among them where the slots leave room; out-of-range ones only for the GPU
    lists = np.stack([rng.permutation(np.delete(np.arange(E), e))[np.arange(Tc) % (E - 1)] for e in range(E)]).astype(np.int32)
    if Tc - 2 >= K - 1:
        lists[:, 1], lists[:, Tc - 1] = lists[:, 0], np.arange(E)
    padded = np.concatenate([np.full((E, 1), -1), lists, np.full((E, 1), E + 1)], axis=1).astype(np.int32)
    for cl, gl in ((None, None), (lists, padded)):
        idx, gates, logits = c2r.route(dev(x), dev(Wg), dev(bias), K, None if gl is None else dev(gl), want_logits=True)
        ri, rg = orc.route(host(logits), K, cl)
        assert np.array_equal(host(idx), ri)
        np.testing.assert_allclose(host(gates), rg, rtol=GATE_RTOL, atol=1e-37)
