"""GPU parity of the expert FFN for batches of few rows (ffn_skinny.hip; gate/up passes of more than 32 routed rows or more
than 8 rows of a single group already run in ffn_mid.hip)."""
import numpy as np
import pytest
import torch

from paper_2504_01337_amd import workloads as wl
from helpers import dev, host, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


def _weights(rng, E, d, F):
    return [wl.round_bf16((rng.standard_normal(s) * 0.05).astype(np.float32)) for s in ((E, F, d), (E, F, d), (E, d, F))]


# fragment edges (15, 16, 17, 32, 33, 48, 49 rows), chunk edges (63, 64, 65 rows), empty groups, 64 groups, more rows
# allotted than used; contraction lengths of 1, 2, 3, 5, 8, 11 and 22 64-wide units (waves without any, remainders of a
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
                                          (8, 1, 200, 64, 128, 192),      # routed few rows, shared not: two launches
                                          (16, 8, 40, 128, 64, 128)])     # and the other way round
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
