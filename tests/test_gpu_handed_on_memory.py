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
