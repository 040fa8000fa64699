"""C2RLayer.forward in one native call (c2r_layer_forward) gives what the same stages give one by one, in every form the
layer takes: gather fused or not, padded widths, shared expert riding in the routed launches, beside them, or in full
precision."""
import numpy as np
import pytest
import torch

from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,T,d,E,K,F,Fs,local,kw", [
    ("bf16", 70, 128, 12, 4, 192, 320, False, {}), ("bf16", 300, 64, 8, 2, 128, 64, True, {}),
    ("bf16", 33, 128, 8, 3, 64, 128, False, {"fuse_shared": False}),
    ("bf16", 33, 128, 8, 3, 64, 128, False, {"fuse_gather": False}),
    ("bf16", 40, 64, 16, 4, 88, 0, False, {}), ("bf16", 40, 64, 16, 4, 88, 72, True, {}),
    ("bf16", 9, 72, 5, 2, 64, 0, False, {}), ("f32", 65, 64, 8, 2, 96, 0, False, {}), ("f32", 10, 64, 7, 2, 32, 64, True, {})])
def test_one_call_equals_the_stages(dtype, T, d, E, K, F, Fs, local, kw):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T * 7 + F)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    w = lambda *sh: dev((rng.standard_normal(sh) * 0.05).astype(np.float32), dtype)
    El, ls = E, None
    if local:
        El = E // 2
        ls = np.full(E, -1, dtype=np.int32)
        ls[np.sort(rng.permutation(E)[:El])] = np.arange(El, dtype=np.int32)
    collab = np.stack([rng.permutation([j for j in range(E) if j != i])[:K + 1] for i in range(E)]).astype(np.int32)
    shared = (w(1, Fs, d), w(1, Fs, d), w(1, d, Fs)) if Fs else None
    layer = c2r.C2RLayer(T, d, E, K, F, tdt, dev(rng.standard_normal((d, E)).astype(np.float32)), None, dev(collab),
                         w(El, F, d), w(El, F, d), w(El, d, F), local_slot=dev(ls), E_local=El, shared=shared, **kw)
    x = dev(rng.standard_normal((T, d)).astype(np.float32), dtype)
    y = layer.forward(x).clone()
    got = [t.clone() for t in (layer.idx, layer.gates, layer.counts, layer.offsets, layer.inv_perm)]
    layer.y.zero_()
    y2 = layer.forward(x, trace={})                    # a trace goes stage by stage
    torch.cuda.synchronize()
    assert y.any() and torch.equal(y, y2)
    for a, b in zip(got, (layer.idx, layer.gates, layer.counts, layer.offsets, layer.inv_perm)):
        assert torch.equal(a, b)


def test_one_call_rejects_what_the_stages_reject():
    from paper_2504_01337_amd import c2r
    z = lambda *sh: torch.zeros(sh, dtype=torch.float32, device="cuda")
    layer = c2r.C2RLayer(4, 16, 4, 3, 8, torch.float32, z(16, 4), None, torch.zeros((4, 1), dtype=torch.int32, device="cuda"),
                         z(4, 8, 16), z(4, 8, 16), z(4, 16, 8))
    with pytest.raises(c2r.C2RError):                  # a list shorter than K - 1
        layer.forward(z(4, 16))
    layer.collab_idx = None
    with pytest.raises(AssertionError):
        layer.forward(z(5, 16))
    layer.w = (z(4, 8, 16), z(4, 8, 16), z(4, 8, 16))
    with pytest.raises(AssertionError):
        layer.forward(z(4, 16))


# fuse_shared asks for the shared expert to ride in the routed launches; in a form that has none to ride in (rows scattered, or h in the
# workspace) it still has to be computed
@pytest.mark.parametrize("dtype,F,Fs,kw", [("bf16", 64, 128, {"fuse_gather": False}), ("bf16", 88, 72, {}), ("bf16", 88, 128, {}),
                                           ("f32", 32, 64, {})])
def test_a_shared_expert_that_cannot_ride_is_computed(dtype, F, Fs, kw):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(F + Fs)
    T, d, E, K = 33, 64, 8, 2
    w = lambda *sh: dev((rng.standard_normal(sh) * 0.05).astype(np.float32), dtype)
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16 if dtype == "bf16" else torch.float32, w(d, E).float(), None, None,
                         w(E, F, d), w(E, F, d), w(E, d, F), shared=(w(1, Fs, d), w(1, Fs, d), w(1, d, Fs)), **kw)
    x = w(T, d)
    y = layer.forward(x, trace={}).clone()             # stage by stage
    fields = list(layer._LAYER.unpack(layer._args()))
    assert fields[9] == 0 and fields[27] == 0          # fuse_shared, h
    fields[9] = 1
    layer.y_shared.fill_(5.0)
    layer.y.zero_()
    assert c2r.lib().c2r_layer_forward(layer._LAYER.pack(*fields), x.data_ptr(), torch.cuda.current_stream().cuda_stream) == c2r.OK
    torch.cuda.synchronize()
    assert torch.equal(layer.y, y)


# a device with one local expert and the shared one: two single groups, at sizes of every FFN kernel (few rows, both sides of their limits,
# between, tiles); the same bits as the shared expert on its own
@pytest.mark.parametrize("T", [1, 4, 5, 9, 33, 90, 700])
def test_one_local_expert_beside_a_shared_one(T):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T)
    d, E, K, F, Fs = 128, 6, 2, 64, 192
    w = lambda *sh: dev((rng.standard_normal(sh) * 0.05).astype(np.float32), "bf16")
    ls = dev(np.array([-1, -1, 0, -1, -1, -1], dtype=np.int32))
    args = (T, d, E, K, F, torch.bfloat16, w(d, E).float(), None, None, w(1, F, d), w(1, F, d), w(1, d, F))
    shared = (w(1, Fs, d), w(1, Fs, d), w(1, d, Fs))
    x = w(T, d)
    got = []
    for fuse in (True, False):
        layer = c2r.C2RLayer(*args, local_slot=ls, E_local=1, shared=shared, fuse_shared=fuse)
        assert layer.fuse_shared == fuse
        got.append(layer.forward(x).clone())
        assert torch.equal(layer.forward(x, trace={}), got[-1])
    torch.cuda.synchronize()
    assert got[0].any() and torch.equal(got[0], got[1])


# a batch without tokens: an empty y and zero counts where the stages take one; gather-fused forms refuse it, as their calls do
@pytest.mark.parametrize("dtype,kw,shared", [("f32", {}, False), ("f32", {}, True), ("bf16", {"fuse_gather": False}, True)])
def test_no_tokens(dtype, kw, shared):
    from paper_2504_01337_amd import c2r
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    d, E, F = 64, 4, 64
    w = lambda *sh: torch.ones(sh, dtype=tdt, device="cuda")
    layer = c2r.C2RLayer(0, d, E, 2, F, tdt, w(d, E).float(), None, None, w(E, F, d), w(E, F, d), w(E, d, F),
                         shared=(w(1, F, d), w(1, F, d), w(1, d, F)) if shared else None, **kw)
    layer.counts.fill_(-7)
    layer.offsets.fill_(-7)
    y = layer.forward(w(0, d))
    torch.cuda.synchronize()
    assert y.shape == (0, d) and not layer.counts.any() and not layer.offsets.any()


# what the stage that takes a riding shared expert accepts, the one call accepts too: weights without the leading 1 (F_shared = d there: the
# constructor reads F_shared from the second dimension)
def test_shared_weights_without_the_leading_dimension():
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(3)
    T, d, E, K, F = 20, 64, 4, 2, 64
    w = lambda *sh: dev((rng.standard_normal(sh) * 0.05).astype(np.float32), "bf16")
    shared = (w(d, d), w(d, d), w(d, d))
    args = (T, d, E, K, F, torch.bfloat16, w(d, E).float(), None, None, w(E, F, d), w(E, F, d), w(E, d, F))
    flat, full = c2r.C2RLayer(*args, shared=shared), c2r.C2RLayer(*args, shared=tuple(t[None] for t in shared))
    assert flat.fuse_shared and full.fuse_shared
    x = w(T, d)
    assert torch.equal(flat.forward(x), full.forward(x)) and torch.equal(flat.forward(x), flat.forward(x, trace={}))


# an error of a later stage comes after the earlier stages: the router ahead of a bad index, the gate/up pass ahead of a bad down pass; batches
# of every form in which stages share a launch
@pytest.mark.parametrize("T,E,dtype,Fs", [(3, 20, "bf16", 0), (3, 20, "bf16", 64), (20, 20, "bf16", 0), (100, 8, "f32", 0), (100, 8, "bf16", 128), (2000, 8, "bf16", 0)])
def test_an_error_of_a_later_stage(T, E, dtype, Fs):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T)
    d, K, F = 64, 2, 64
    w = lambda *sh: dev((rng.standard_normal(sh) * 0.05).astype(np.float32), dtype)
    shared = (w(1, Fs, d), w(1, Fs, d), w(1, d, Fs)) if Fs else None
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16 if dtype == "bf16" else torch.float32, w(d, E).float(), None, None,
                         w(E, F, d), w(E, F, d), w(E, d, F), shared=shared)
    x = w(T, d)
    layer.forward(x)
    idx, gates, inv = layer.idx.clone(), layer.gates.clone(), layer.inv_perm.clone()
    h = None if layer.h is None else layer.h.clone()

    def call(field, value):
        fields = list(layer._LAYER.unpack(layer._args()))
        fields[field] = value
        for t in (layer.idx, layer.gates, layer.inv_perm, layer.h):
            if t is not None:
                t.fill_(-7)
        rc = c2r.lib().c2r_layer_forward(layer._LAYER.pack(*fields), x.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return rc

    assert call(37, 0) == c2r.ERR_WORKSPACE            # ws_permute_bytes
    assert torch.equal(layer.idx, idx) and torch.equal(layer.gates, gates) and bool((layer.inv_perm == -7).all())
    assert call(36, 0) == c2r.ERR_WORKSPACE            # ws_route_bytes
    assert bool((layer.idx == -7).all())
    if h is not None:
        assert call(16, 0) == c2r.ERR_INVALID_ARG      # w_down
        assert torch.equal(layer.idx, idx) and torch.equal(layer.inv_perm, inv) and torch.equal(layer.h, h)
