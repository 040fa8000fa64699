"""GPU parity of the expert FFN for batches of few rows (ffn_skinny.hip; passes of more rows than its limits already run in
ffn_mid.hip)."""
import numpy as np
import pytest
import torch

from paper_2504_01337_amd import workloads as wl
from helpers import dev, ffn_kernel, host, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


def _weights(rng, E, d, F):
    return [wl.round_bf16((rng.standard_normal(s) * 0.05).astype(np.float32)) for s in ((E, F, d), (E, F, d), (E, d, F))]


# batches on both sides of the limits: fragment edges (15, 16, 17, 32, 33, 48, 49 rows), 63, 64 and 65 rows, empty groups, 64
# groups, more rows allotted than used; contraction lengths of 1, 2, 3, 5, 8, 11 and 22 64-wide units (waves without any, remainders of a
# burst), widths that are no multiple of 64 (k tail and padding columns) and of 16 (column tail)
@pytest.mark.parametrize("d,F,sizes,spare", [
    (64, 64, [1], 0), (64, 64, [1, 0, 3], 0), (128, 192, [15, 16, 17, 0, 32, 33, 48, 49], 0),
    (192, 88, [63, 64, 65, 1], 5), (320, 688, [4, 0, 0, 2], 0), (2048, 136, [20, 0, 7], 100),
    (512, 1408, [2, 9], 0), (704, 72, [4] * 64, 0), (64, 1400, [64, 2], 0)])
def test_few_rows_against_oracle(c2r, orc, d, F, sizes, spare):
    rng = np.random.default_rng(d + F)
    E = len(sizes)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(offsets[-1])
    cap = n + spare
    assert cap <= (64 if E == 1 else 256)
    x = wl.round_bf16(rng.standard_normal((cap, d)).astype(np.float32))
    wg, wu, wd = _weights(rng, E, d, F)
    y = torch.full((cap, d), 123.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, cap, d, E, 1, F, c2r.BF16),), 255, dtype=torch.uint8,
                    device="cuda")                                       # stale scratch: NaNs as bf16
    c2r.expert_ffn(dev(x, "bf16"), dev(offsets), dev(wg, "bf16"), dev(wu, "bf16"), dev(wd, "bf16"), ws=ws, out=y)
    torch.cuda.synchronize()
    ref = orc.expert_ffn_rows(x[:n], np.repeat(np.arange(E), sizes).astype(np.int32), wg, wu, wd)
    assert max_rel_err(host(y)[:n], ref) <= 1e-2
    assert np.all(host(y)[n:] == 123.0)


@pytest.mark.parametrize("E,K,T,d,F,Fs", [(60, 4, 1, 128, 192, 448), (60, 4, 64, 2048, 64, 320), (7, 2, 33, 64, 64, 64),
                                          (8, 1, 200, 64, 128, 192), (16, 8, 40, 128, 64, 128),   # more rows than few
                                          # few rows for the routed groups alone, not beside this shared expert
                                          (60, 1, 9, 128, 192, 448), (60, 1, 33, 64, 64, 128), (60, 4, 33, 64, 64, 128),
                                          # and the other way round
                                          (16, 8, 5, 128, 64, 128), (40, 6, 30, 64, 64, 192)])
def test_few_rows_entry_points_agree_bit_for_bit(c2r, E, K, T, d, F, Fs):
    rng = np.random.default_rng(E * 1000 + T)
    idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)
    x = dev(rng.standard_normal((T, d)).astype(np.float32), "bf16")
    wg, wu, wd = (dev(a, "bf16") for a in _weights(rng, E, d, F))
    sg, su, sd = (dev(a, "bf16") for a in _weights(rng, 1, d, Fs))
    counts, offsets, perm, inv, x_perm = c2r.permute(x, dev(idx), E)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    h = [torch.zeros(T * K, F, **bf) for _ in range(3)]
    y = [torch.zeros(T * K, d, **bf) for _ in range(3)]
    hs = [torch.zeros(T, Fs, **bf) for _ in range(2)]
    ys = [torch.zeros(T, d, **bf) for _ in range(2)]
    off_s = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    c2r.expert_ffn_gate_up(x_perm, offsets, wg, wu, h[0])
    c2r.expert_ffn_gate_up_gather(x, perm, K, offsets, wg, wu, h[1])
    c2r.expert_ffn_gate_up(x, off_s, sg, su, hs[0])
    c2r.expert_ffn_gate_up_with_shared(x, perm, K, offsets, wg, wu, h[2], sg, su, hs[1])
    c2r.expert_ffn_down(h[0], offsets, wd, y[0])
    c2r.expert_ffn(x_perm, offsets, wg, wu, wd, out=y[1])
    c2r.expert_ffn_down(hs[0], off_s, sd, ys[0])
    c2r.expert_ffn_down_with_shared(h[2], offsets, wd, y[2], hs[1], sd, ys[1])
    torch.cuda.synchronize()
    assert torch.equal(h[0], h[1]) and torch.equal(h[0], h[2]) and torch.equal(hs[0], hs[1])
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2]) and torch.equal(ys[0], ys[1])
    assert h[0].any() and y[0].any() and ys[0].any()


def _both_allotments(c2r, d, F, sizes, x, w, poison=0.0):
    """The rows of sizes allotted as they are and in a large buffer (the tile kernel): y of each."""
    E, n = len(sizes), sum(sizes)
    assert {ffn_kernel(0, E, 600 * E + n, F), ffn_kernel(1, E, 600 * E + n, d)} == {"tile"}
    offsets = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    got = []
    for cap in (n, 600 * E + n):
        xa = torch.full((cap, d), poison, dtype=torch.bfloat16, device="cuda")
        xa[:n] = x
        y = torch.full((cap, d), 123.0, dtype=torch.bfloat16, device="cuda")
        ws = torch.full((c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, cap, d, E, 1, F, c2r.BF16),), 255, dtype=torch.uint8,
                        device="cuda")
        c2r.expert_ffn(xa, offsets, *w, ws=ws, out=y)
        torch.cuda.synchronize()
        assert torch.all(y[n:] == 123.0)
        got.append(y[:n])
    return got


# The sums are the tile kernel's, so a row has the same bits whatever is allotted around it.  Both passes few rows: one and
# two 16-row fragments (15, 16, 17, 31, 32 rows of a group), a single group of 1 to 8.  The down pass alone: 33 to 64 rows, several
# 64-row chunks (65, 130), a single group up to its limit, 40 and 64 groups; with 16 groups the four-waves-per-SIMD form meets
# groups of more than one fragment.  Contractions of 1 to 88 units, ends inside a unit, bursts that come out even and not.
@pytest.mark.parametrize("both,d,F,sizes", [
    (True, 64, 64, [1]), (True, 320, 88, [8]), (True, 704, 72, [1, 0, 3]), (True, 2048, 1408, [17, 15] + [0] * 14),
    (True, 512, 688, [0, 16, 1, 7] + [0] * 16), (True, 4032, 136, [1, 31] + [0] * 14), (True, 192, 5632, [32] + [0] * 15),
    (False, 128, 5632, [9]), (False, 192, 88, [16]), (False, 64, 1400, [17]), (False, 64, 192, [32]),
    (False, 128, 192, [15, 16, 17, 0, 32, 33]), (False, 64, 1400, [63, 64, 1]), (False, 192, 688, [65, 0, 2]),
    (False, 64, 320, [130, 9]), (False, 320, 704, [3] * 40), (False, 128, 136, [1] * 64), (False, 64, 1408, [65, 33, 20] + [0] * 13)])
def test_few_rows_have_the_bits_of_any_allotment(c2r, orc, both, d, F, sizes):
    rng = np.random.default_rng(d * 5 + F)
    E, n = len(sizes), sum(sizes)
    assert [ffn_kernel(0, E, n, F), ffn_kernel(1, E, n, d)] == ["few" if both else "mid", "few"]
    x = wl.round_bf16(rng.standard_normal((n, d)).astype(np.float32))
    w = _weights(rng, E, d, F)
    few, many = _both_allotments(c2r, d, F, sizes, dev(x, "bf16"), [dev(a, "bf16") for a in w], float("nan"))
    assert torch.equal(few, many)
    ref = orc.expert_ffn_rows(x, np.repeat(np.arange(E), sizes).astype(np.int32), *w)
    assert max_rel_err(host(few), ref) <= 1e-2


# A row or a weight that is not finite spoils what it meets and nothing else, exactly where the tile kernel has it: an activation row,
# weight rows of either pass, the last column of a contraction that ends inside a unit (its neighbours there are padding)
@pytest.mark.parametrize("kind", ["row inf", "row nan", "gate inf", "up nan", "down first", "down last"])
@pytest.mark.parametrize("which,d,F,sizes", [("few", 128, 136, [9, 2, 5, 1, 0, 3, 0, 2, 1, 0, 0, 1, 0, 0, 0, 4]), ("few", 64, 200, [5]),
                                             ("mid", 64, 88, [60, 53, 63]), ("mid", 192, 72, [90])])
def test_values_that_are_not_finite(c2r, kind, which, d, F, sizes):
    rng = np.random.default_rng(d + F)
    E, n = len(sizes), sum(sizes)
    assert [ffn_kernel(0, E, n, F), ffn_kernel(1, E, n, d)] == [which, which]
    x = rng.standard_normal((n, d)).astype(np.float32)
    w = _weights(rng, E, d, F)
    at = {"row inf": (x, (n // 2, 3), np.inf), "row nan": (x, (n // 2, d - 1), np.nan), "gate inf": (w[0], (0, 3, 5), np.inf),
          "up nan": (w[1], (E - 1, F - 1, 0), np.nan), "down first": (w[2], (0, 7, 0), np.inf),
          "down last": (w[2], (E - 1, d - 1, F - 1), -np.inf)}[kind]
    at[0][at[1]] = at[2]
    small, many = _both_allotments(c2r, d, F, sizes, dev(x, "bf16"), [dev(a, "bf16") for a in w])
    bad = torch.isnan(small)
    assert torch.equal(bad, torch.isnan(many)) and torch.equal(small[~bad], many[~bad])
    spoilt = int((~torch.isfinite(small)).sum())
    assert spoilt > 0 and (spoilt < small.numel() or (E == 1 and kind in ("gate inf", "up nan")))  # (one group: every row meets those)
