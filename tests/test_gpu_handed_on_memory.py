"""Stages that run in order may hand memory on: one scratch for all of them, a result in the place of an input that is done with.  A call
that does several stages' work in one launch gives the same bits there as with memory of its own for everything."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# fields of c2r_layer
X_PERM, H, Y_PERM, Y_SHARED, WS_ROUTE, WS_PERMUTE, WS_FFN = 26, 27, 28, 31, 32, 33, 34
PERM = 24


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


def _layer(c2r, T, d, E, K, F, dtype=torch.bfloat16, Fs=0, seed=0, **kw):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d + E + F + seed)
    w = lambda *s: torch.randn(s, generator=gen, device="cuda").mul_(0.05).to(dtype)
    lists = np.stack([np.random.default_rng(e).permutation(np.delete(np.arange(E), e))[:K + 1] for e in range(E)]).astype(np.int32)
    shared = (w(1, Fs, d), w(1, Fs, d), w(1, d, Fs)) if Fs else None
    layer = c2r.C2RLayer(T, d, E, K, F, dtype, w(d, E).float(), None, torch.from_numpy(lists).cuda(), w(E, F, d), w(E, F, d), w(E, d, F),
                         shared=shared, **kw)
    return layer, w(T, d)


def _forward(c2r, layer, x, places):
    """The layer call with some of its pointers replaced; y."""
    fields = list(layer._LAYER.unpack(layer._args()))
    for k, p in places.items():
        assert fields[k] != 0
        fields[k] = p
    layer.y.fill_(float("nan"))
    assert c2r.lib().c2r_layer_forward(layer._LAYER.pack(*fields), x.data_ptr(), torch.cuda.current_stream().cuda_stream) == c2r.OK
    return layer.y


def _memory(*tensors):
    return torch.full((max(t.numel() * t.element_size() for t in tensors),), 255, dtype=torch.uint8, device="cuda")


# selection and index at the start of the gate/up pass (up to 16 tokens): the chunk results that it reads where h goes, in more than a round
# of workgroups; h of the layer and of the workspace, a shared expert beside; the first batch that is selected before
@pytest.mark.parametrize("T,d,E,K,F,Fs", [(1, 256, 8, 2, 64, 0), (5, 1024, 20, 4, 704, 0), (5, 1024, 20, 4, 712, 0), (6, 512, 60, 4, 704, 1408),
                                          (16, 256, 16, 2, 704, 0), (17, 256, 32, 1, 704, 0)])
def test_scratch_of_the_router_where_h_goes(c2r, T, d, E, K, F, Fs):
    layer, x = _layer(c2r, T, d, E, K, F, Fs=Fs)
    ref = layer.forward(x).clone()
    own = layer.h if F % 64 == 0 else layer.ws_ffn
    for _ in range(3):
        m = _memory(own, layer.ws_route, layer.ws_perm).data_ptr()
        places = {WS_ROUTE: m, WS_PERMUTE: m, (H if F % 64 == 0 else WS_FFN): m}
        assert torch.equal(_forward(c2r, layer, x, places), ref)
    m = _memory(layer.perm, layer.ws_route).data_ptr()
    assert torch.equal(_forward(c2r, layer, x, {WS_ROUTE: m, PERM: m}), ref)


# selection, index and row scatter in one launch (few experts): the chunk results that it reads where the rows or the index go; 65 tokens and up
# without rows; batches that one workgroup selects for, and the first that no launch does it all for
@pytest.mark.parametrize("T,d,E,K,F,kw", [(20, 256, 8, 2, 64, {"fuse_gather": False}), (512, 256, 8, 2, 64, {"fuse_gather": False}),
                                          (1000, 128, 16, 4, 64, {"fuse_gather": False}), (1024, 64, 16, 3, 72, {"fuse_gather": False}),
                                          (1025, 64, 16, 3, 72, {"fuse_gather": False}), (128, 256, 16, 4, 64, {})])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_scratch_of_the_router_where_the_rows_go(c2r, T, d, E, K, F, kw, dtype):
    layer, x = _layer(c2r, T, d, E, K, F, dtype, **kw)
    ref = layer.forward(x).clone()
    for field, own in ((X_PERM, layer.x_perm), (PERM, layer.perm)):
        if own is None:
            continue
        for _ in range(3):
            m = _memory(own, layer.ws_route).data_ptr()
            assert torch.equal(_forward(c2r, layer, x, {WS_ROUTE: m, field: m}), ref)


# both FFN passes in one launch: results in the place of what the first pass reads.  Sizes on either side of the rule for one launch.
@pytest.mark.parametrize("T,Fs", [(200, 1408), (1300, 2560), (2500, 1024)])
def test_results_in_the_place_of_x(c2r, T, Fs):
    layer, x = _layer(c2r, T, 128, 16, 4, 832, Fs=Fs)
    assert layer.fuse_shared
    ref, y_perm = layer.forward(x).clone(), layer.y_perm.clone()
    for _ in range(3):
        xs = x.clone()
        assert torch.equal(_forward(c2r, layer, xs, {Y_SHARED: xs.data_ptr()}), ref)
    m = _memory(layer.y_perm)                          # x at the end of y_perm
    for _ in range(3):
        xs = m[m.numel() - x.numel() * 2:].view(torch.bfloat16).view(x.shape)
        xs.copy_(x)
        layer.y_perm.fill_(7.0)
        assert torch.equal(_forward(c2r, layer, xs, {Y_PERM: m.data_ptr()}), ref)
        assert torch.equal(m.view(torch.bfloat16).view(y_perm.shape), y_perm)
    # one scratch for every stage that has one
    n = _memory(layer.ws_route, layer.ws_perm).data_ptr()
    assert torch.equal(_forward(c2r, layer, x, {WS_ROUTE: n, WS_PERMUTE: n}), ref)


# the expert FFN alone: y_perm over x where rows are gathered (partly and whole), in the place of x_perm where they are not, and over a part of it
@pytest.mark.parametrize("sizes,F", [([30, 0, 70], 448), ([700, 600, 33, 257], 2560), ([1500], 7744)])
def test_expert_ffn_over_its_input(c2r, sizes, F):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(F)
    d, E, K, n = 128, len(sizes), 2, sum(sizes)
    w = [torch.randn(s, generator=gen, device="cuda").mul_(0.05).bfloat16() for s in ((E, F, d), (E, F, d), (E, d, F))]
    T = (n + K - 1) // K
    x = torch.randn((T, d), generator=gen, device="cuda").bfloat16()
    perm = torch.randperm(T * K, generator=gen, device="cuda").to(torch.int32)[:n].contiguous()
    offsets = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int32, device="cuda")
    ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, n, d, E, 1, F, c2r.BF16), dtype=torch.uint8, device="cuda")
    x_perm = x[(perm // K).long()].contiguous()
    ref = c2r.expert_ffn(x_perm, offsets, *w).clone()
    for _ in range(3):
        for shift in (0, 16, n - T):                   # rows of y_perm before x
            m = torch.full((n + T + 16, d), 7.0, dtype=torch.bfloat16, device="cuda")
            xs, y = m[shift:shift + T], m[:n]
            xs.copy_(x)
            ws.fill_(255)
            c2r.expert_ffn_gather(xs, perm, K, offsets, *w, ws=ws, out=y)
            assert torch.equal(y, ref)
        xs = x_perm.clone()
        assert torch.equal(c2r.expert_ffn(xs, offsets, *w, ws=ws, out=xs), ref)
        m = torch.full((n + 300, d), 7.0, dtype=torch.bfloat16, device="cuda")
        m[300:].copy_(x_perm)
        assert torch.equal(c2r.expert_ffn(m[300:], offsets, *w, ws=ws, out=m[:n]), ref)


# the dispatch index with send_row in the place of topk_idx, on either side of the rule for one launch
@pytest.mark.parametrize("T,K,n_dev", [(1, 4, 4), (1000, 4, 4), (1000, 3, 60), (4096, 2, 3), (4097, 2, 3), (8192, 4, 8), (700, 6, 5)])
def test_dispatch_index_over_its_input(c2r, T, K, n_dev):
    rng = np.random.default_rng(T)
    E = 60
    idx = torch.from_numpy(np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)).cuda()
    devmap = torch.from_numpy(rng.integers(-1, n_dev, size=E).astype(np.int32)).cuda()
    counts, offsets, token, row = c2r.dedup_dispatch(idx, E, devmap, n_dev)
    ws = torch.empty(max(256, c2r.workspace_bytes(c2r.STAGE_DEDUP_DISPATCH, T, 0, n_dev, K, 0, c2r.F32)), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        both, c, o, t = idx.clone(), torch.empty_like(counts), torch.empty_like(offsets), torch.full_like(token, -1)
        p = lambda v: v.data_ptr()
        assert c2r.lib().c2r_dedup_dispatch(p(both), T, K, E, p(devmap), n_dev, p(c), p(o), p(t), p(both), p(ws), ws.numel(),
                                            torch.cuda.current_stream().cuda_stream) == c2r.OK
        assert torch.equal(c, counts) and torch.equal(o, offsets) and torch.equal(t, token) and torch.equal(both.view(-1), row.view(-1))
