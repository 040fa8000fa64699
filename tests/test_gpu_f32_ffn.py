"""Full-precision expert FFN: the tile shapes of ffn_f32.hip against the oracle and against each other.  They add in the same
order, and which one runs follows from the rows allotted, so a larger allotment has to give the same bits."""
import numpy as np
import pytest
import torch

from helpers import TOL, dev, host, max_rel_err

pytestmark = pytest.mark.gpu


# contraction lengths that end inside a 16-, 32- and 64-wide group of k (8, 24, 40, 72, 136, 520) and that do not; widths that end
# inside a 16-, 32-, 64- and 128-wide column block; groups of 1, 15 to 17, 31 to 33, 127 to 129 and no rows.  The last two: some 4000
# rows and a contraction of 512 and more
@pytest.mark.parametrize("d,F,sizes,spare", [
    (8, 8, [1], 0), (24, 40, [15, 16, 17, 0, 1], 3), (72, 136, [31, 32, 33, 127, 128, 129], 0), (64, 512, [40] * 8, 0),
    (520, 264, [300, 0, 2, 61], 0), (256, 512, [128] * 8, 0), (1032, 72, [600, 700], 0), (256, 512, [900, 33, 0, 1000, 511, 513, 1, 1042], 0),
    (264, 520, [15, 1500, 17, 800, 0, 1200, 64, 404], 0)])
def test_f32_rows_against_oracle_and_between_kernels(orc, d, F, sizes, spare):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(d + F)
    E = len(sizes)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(offsets[-1])
    x = rng.standard_normal((n, d)).astype(np.float32)
    w = [(rng.standard_normal(s) * 0.1).astype(np.float32) for s in ((E, F, d), (E, F, d), (E, d, F))]
    wd = [dev(a) for a in w]
    got = []
    for cap in (n + spare, 256 * 128 + n):                  # (64-row tiles wherever the width holds three column blocks)
        xa = torch.full((cap, d), float("nan"), device="cuda")
        xa[:n] = dev(x)
        h = torch.full((cap, F), 77.0, device="cuda")
        y = torch.full((cap, d), 123.0, device="cuda")
        c2r.expert_ffn_gate_up(xa, dev(offsets), wd[0], wd[1], h)
        c2r.expert_ffn_down(h, dev(offsets), wd[2], y)
        torch.cuda.synchronize()
        assert torch.all(y[n:] == 123.0) and torch.all(h[n:] == 77.0)
        got.append(y[:n])
    assert torch.equal(got[0], got[1])
    ref = orc.expert_ffn_rows(x, np.repeat(np.arange(E), sizes).astype(np.int32), *w)
    assert max_rel_err(host(got[0]), ref) <= TOL["f32"]


# edges of the 32- and 64-row tiles, column blocks of 32 and 64, contractions of one to four 32-wide slices and a ragged last one
@pytest.mark.parametrize("d,F,sizes", [(64, 32, [63, 64, 65]), (96, 72, [95, 96, 97, 31, 32, 33]), (104, 128, [1, 0, 62, 66]), (32, 96, [129, 2])])
def test_f32_tile_edges_between_allotments(orc, d, F, sizes):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(d * F)
    E, n = len(sizes), sum(sizes)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    x = rng.standard_normal((n, d)).astype(np.float32)
    w = [(rng.standard_normal(s) * 0.1).astype(np.float32) for s in ((E, F, d), (E, F, d), (E, d, F))]
    wd = [dev(a) for a in w]
    got = []
    for cap in (n, 64 * 1280 + n, 32 * 1025 + n):  # the small tiles, the 64-row tiles, and the small ones' shallower ring
        xa = torch.zeros((cap, d), device="cuda")
        xa[:n] = dev(x)
        y = torch.full((cap, d), 5.0, device="cuda")
        c2r.expert_ffn(xa, dev(offsets), *wd, out=y)
        assert torch.all(y[n:] == 5.0)
        got.append(y[:n])
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
    ref = orc.expert_ffn_rows(x, np.repeat(np.arange(E), sizes).astype(np.int32), *w)
    assert max_rel_err(host(got[0]), ref) <= TOL["f32"]
