"""Selection from stored logits: tokens that the keyed chain cannot decide (values that differ in the bits the column replaces, ties,
NaNs, infinities) among ones that it can, subnormal values, partial groups of 64 tokens."""
import numpy as np
import pytest

from helpers import GATE_RTOL, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,K,lists", [(64, 64, 4, True), (1000, 60, 4, False), (130, 16, 3, True), (67, 36, 4, True), (65, 48, 2, False),
                                         (3, 4, 4, False), (5000, 60, 4, True)])
def test_close_tied_special_and_subnormal_logits(orc, T, E, K, lists):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    l = rng.standard_normal((T, E)).astype(np.float32)
    kind = rng.integers(0, 8, size=T)
    b = l.view(np.int32)
    close = kind == 1                                        # a few bit patterns apart, both signs
    b[close] = np.float32(1.5).view(np.int32) + rng.integers(0, 130, size=(int(close.sum()), E)).astype(np.int32)
    l[close & (rng.random(T) < 0.5)] *= -1
    l[kind == 2] = rng.integers(-1, 2, size=(int((kind == 2).sum()), E))                   # ties, zeros of both signs
    l[kind == 2] *= np.where(rng.random((int((kind == 2).sum()), E)) < 0.5, -1, 1).astype(np.float32)
    sub = kind == 3                                          # subnormals
    b[sub] = rng.integers(0, 1 << 20, size=(int(sub.sum()), E)).astype(np.int32) | (rng.integers(0, 2, size=(int(sub.sum()), E)) << 31).astype(np.int32)
    for k, v in ((4, np.nan), (5, np.inf), (6, -np.inf)):
        l[(kind == k)[:, None] & (rng.random((T, E)) < 0.3)] = v
    ci = None
    if lists:
        ci = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, E // 4)] for e in range(E)]).astype(np.int32)
    idx, gates = c2r.route_from_logits(dev(l), K, None if ci is None else dev(ci))
    ri, rg = orc.route(l, K, ci)
    assert np.array_equal(host(idx), ri)
    np.testing.assert_allclose(host(gates), rg, rtol=GATE_RTOL, atol=1e-37)
    if K > 1:
        C = dev(np.zeros((E, E), dtype=np.int32))
        c2r.profile_from_logits(dev(l), K, C, None if ci is None else dev(ci))
        assert np.array_equal(host(C), orc.coactivation(ri, E))
