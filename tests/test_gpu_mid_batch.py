"""GPU parity of the expert FFN kernel for batches between decoding and prefill (ffn_mid.hip).  It sums in the tile kernel's
order, and which of the two runs follows from the rows ALLOTTED, so the same rows in a larger allotment have to give the same
bits; the oracle bar is the one of every bf16 pass (tests/helpers.py)."""
import numpy as np
import pytest
import torch

from paper_2504_01337_amd import workloads as wl
from helpers import TOL, dev, ffn_kernel, ffn_two_problems, host, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


# edges of the 32-, 64- and 128-row tiles and of their 16-row fragments, groups of several tiles, empty groups, one group
# only, fewer tiles than workgroups and tiles of a single 64-wide k-slice (a workgroup crosses several in its first ring);
# k tails and padding columns (88, 688, 1400), column tails (72, 136), rows past the allotment's use
# (first column: the passes that run in this kernel; in the others, and where the rule has moved on, the tile kernel runs twice)
@pytest.mark.parametrize("mid,d,F,sizes,spare", [
    ("both", 64, 64, [90], 0), ("down", 64, 64, [200], 0), ("both", 64, 72, [31, 32, 33, 0, 15, 16, 17, 1], 60),
    ("both", 192, 88, [63, 64, 65, 129, 0, 1], 5), ("both", 320, 688, [127, 128, 48, 0], 20), ("both", 704, 136, [5] * 60, 0),
    ("gate/up", 64, 1400, [97, 300, 2], 0), ("none", 512, 192, [250, 1, 255], 0),
    # several chunks of a group in every tile height: 128 rows, 64, and 32 (a single group; 60 groups of which one holds most)
    ("both", 512, 192, [160, 1, 105], 0), ("both", 128, 320, [100, 33, 40, 0], 0), ("both", 192, 136, [64], 0), ("both", 64, 704, [33], 0),
    ("both", 128, 64, [90] + [1] * 59, 100), ("both", 64, 128, [178, 1], 0)])
def test_mid_rows_against_oracle_and_tile_kernel(c2r, orc, mid, d, F, sizes, spare):
    rng = np.random.default_rng(d * 3 + F)
    E = len(sizes)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(offsets[-1])
    assert [ffn_kernel(0, E, n + spare, F), ffn_kernel(1, E, n + spare, d)] == [
        "mid" if mid in ("both", "gate/up") else "tile", "mid" if mid in ("both", "down") else "tile"]
    assert {ffn_kernel(0, E, 600 * E + n, F), ffn_kernel(1, E, 600 * E + n, d)} == {"tile"}
    x = wl.round_bf16(rng.standard_normal((n, d)).astype(np.float32))
    wg, wu, wd = [wl.round_bf16((rng.standard_normal(s) * 0.05).astype(np.float32)) for s in ((E, F, d), (E, F, d), (E, d, F))]
    w = [dev(a, "bf16") for a in (wg, wu, wd)]
    got = []
    for cap in (n + spare, 600 * E + n):
        xa = torch.full((cap, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        xa[:n] = dev(x, "bf16")
        y = torch.full((cap, d), 123.0, dtype=torch.bfloat16, device="cuda")
        ws = torch.full((c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, cap, d, E, 1, F, c2r.BF16),), 255, dtype=torch.uint8,
                        device="cuda")                                    # stale scratch: NaNs as bf16
        c2r.expert_ffn(xa, dev(offsets), *w, ws=ws, out=y)
        torch.cuda.synchronize()
        assert torch.all(y[n:] == 123.0)
        got.append(y[:n])
    assert torch.equal(got[0], got[1])
    ref = orc.expert_ffn_rows(x, np.repeat(np.arange(E), sizes).astype(np.int32), wg, wu, wd)
    assert max_rel_err(host(got[0]), ref) <= TOL["bf16"]


# the gathered first pass (row numbers held in LDS: up to 4096 of them), alone and with a shared expert riding along
@pytest.mark.parametrize("E,K,T,d,F,Fs", [(60, 4, 70, 128, 64, 320), (60, 4, 250, 64, 64, 128), (40, 4, 1024, 64, 64, 64),
                                          (40, 4, 1025, 64, 64, 64), (1, 1, 100, 64, 128, 64)])
def test_mid_entry_points_agree_bit_for_bit(c2r, E, K, T, d, F, Fs):
    rng = np.random.default_rng(E * 1000 + T)
    idx = np.stack([rng.permutation(E)[:K] for _ in range(T)]).astype(np.int32)
    r = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), "bf16")
    x, wg, wu, wd = r(T, d), r(E, F, d), r(E, F, d), r(E, d, F)
    sg, su, sd = r(1, Fs, d), r(1, Fs, d), r(1, d, Fs)
    counts, offsets, perm, inv, x_perm = c2r.permute(x, dev(idx), E)
    z = lambda rows, cols: torch.zeros(rows, cols, dtype=torch.bfloat16, device="cuda")
    h, y, hs, ys = [z(T * K, F) for _ in range(3)], [z(T * K, d) for _ in range(2)], [z(T, Fs) for _ in range(2)], [z(T, d) for _ in range(2)]
    off_s = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    c2r.expert_ffn_gate_up(x_perm, offsets, wg, wu, h[0])
    c2r.expert_ffn_gate_up_gather(x, perm, K, offsets, wg, wu, h[1])
    c2r.expert_ffn_gate_up(x, off_s, sg, su, hs[0])
    c2r.expert_ffn_down(h[0], offsets, wd, y[0])
    c2r.expert_ffn_down(hs[0], off_s, sd, ys[0])
    if E > 1:
        c2r.expert_ffn_gate_up_with_shared(x, perm, K, offsets, wg, wu, h[2], sg, su, hs[1])
        c2r.expert_ffn_down_with_shared(h[2], offsets, wd, y[1], hs[1], sd, ys[1])
        assert torch.equal(h[0], h[2]) and torch.equal(hs[0], hs[1])
        assert torch.equal(y[0], y[1]) and torch.equal(ys[0], ys[1])
    assert torch.equal(h[0], h[1]) and h[0].any() and y[0].any() and ys[0].any()


# the tile kernel cuts a single group with a long contraction into 64-row (d 2048: up to 1280 rows), 128-row or 256-row tiles:
# alone and beside routed groups it gives the bits of any other cut
@pytest.mark.parametrize("T", [513, 639, 1025, 1280, 1281, 1793])
def test_lower_tiles_of_a_single_group_change_no_bits(c2r, T):
    rng = np.random.default_rng(T)
    d, F, Fs, E, K = 2048, 64, 192, 6, 2
    r = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), "bf16")
    h, hs, wd, sd = r(T * K, F), r(T, Fs), r(E, d, F), r(1, d, Fs)
    offsets = torch.tensor(np.linspace(0, T * K, E + 1).round().astype(np.int32), device="cuda")
    z = lambda rows: torch.zeros(rows, d, dtype=torch.bfloat16, device="cuda")
    y, ys, alone, tall, y2 = z(T * K), z(T), z(T), z(3000), z(T * K)
    c2r.expert_ffn_down_with_shared(h, offsets, wd, y, hs, sd, ys)
    off = lambda n: torch.tensor([0, n], dtype=torch.int32, device="cuda")
    c2r.expert_ffn_down(hs, off(T), sd, alone)
    c2r.expert_ffn_down(torch.cat([hs, torch.zeros(3000 - T, Fs, dtype=torch.bfloat16, device="cuda")]), off(T), sd, tall)
    c2r.expert_ffn_down(h, offsets, wd, y2)
    torch.cuda.synchronize()
    assert ys.any() and torch.equal(ys, alone) and torch.equal(ys, tall[:T]) and not tall[T:].any()
    assert torch.equal(y, y2)
    ref = hs.double() @ sd[0].double().t()
    assert ((ys.double() - ref).abs().max() / ref.abs().max()).item() <= TOL["bf16"]


# two problems in one launch, tiles of their own heights and workgroups of their own: routed groups even, skewed, one holding all and
# none holding any; single groups of one to eight chunks, short and long beside the routed ones.  up, down: the rows of the routed and of the
# shared tiles of that pass, or the other kernel that takes it
@pytest.mark.parametrize("T,E,d,F,Fs,sizes,cap,up,down", [
    (20, 10, 128, 64, 1024, [8] * 10, 80, (64, 32), "few"), (131, 60, 192, 128, 64, [100, 70] + [6] * 58, 524, (64, 64), (64, 64)),
    (179, 30, 64, 704, 320, [0] * 29 + [716], 716, (64, 64), (64, 64)), (70, 12, 704, 64, 64, [0] * 12, 280, (64, 64), (64, 32)),
    (500, 60, 64, 192, 1408, [400, 129, 65] + [24] * 57, 2000, "tile", (64, 64)), (65, 40, 256, 320, 64, [65, 0, 33, 1] * 10, 990, (64, 64), (64, 32)),
    (16, 60, 128, 1408, 320, [3, 0, 1] * 16 + [0] * 12, 64, (32, 32), "few"), (100, 60, 192, 320, 704, [2] * 60, 240, (32, 64), (32, 32)),
    (150, 60, 704, 64, 320, [33, 0, 1] + [3] * 57, 240, (32, 64), (32, 64)), (179, 8, 128, 192, 320, [140, 0, 129, 1, 260, 100, 86, 0], 716, (128, 64), (128, 64)),
    (200, 8, 256, 64, 704, [129, 70, 0, 1, 48, 60, 60, 32], 400, "tile", (128, 64)), (64, 4, 64, 320, 128, [200, 129, 0, 183], 512, (128, 32), "tile")])
def test_mid_two_problems_against_each_alone(c2r, T, E, d, F, Fs, sizes, cap, up, down):
    assert (ffn_two_problems(0, E, cap, T), ffn_two_problems(1, E, cap, T)) == (up, down)
    rng = np.random.default_rng(T * E)
    n = sum(sizes)
    r = lambda *s: dev((rng.standard_normal(s) * 0.1).astype(np.float32), "bf16")
    z = lambda rows, cols: torch.zeros(rows, cols, dtype=torch.bfloat16, device="cuda")
    offsets = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    x, wg, wu, wd, sg, su, sd = r(T, d), r(E, F, d), r(E, F, d), r(E, d, F), r(1, Fs, d), r(1, Fs, d), r(1, d, Fs)
    perm = dev(rng.integers(0, T * 4, size=max(n, 1)).astype(np.int32))
    h, y, hs, ys = z(cap, F), z(cap, d), z(T, Fs), z(T, d)
    full = torch.zeros(cap, dtype=torch.int32, device="cuda")
    full[:n] = perm[:n]
    c2r.expert_ffn_gate_up_with_shared(x, full, 4, offsets, wg, wu, h, sg, su, hs)
    c2r.expert_ffn_down_with_shared(h, offsets, wd, y, hs, sd, ys)
    big = 600 * E + n                               # allotments of the tile kernel
    xa, h2, y2 = z(big, d), z(big, F), z(big, d)
    xa[:n] = x[torch.div(full[:n], 4, rounding_mode="floor").long()]
    c2r.expert_ffn_gate_up(xa, offsets, wg, wu, h2)
    c2r.expert_ffn_down(h2, offsets, wd, y2)
    xs, hs2, ys2 = z(3000, d), z(3000, Fs), z(3000, d)
    xs[:T] = x
    off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    c2r.expert_ffn_gate_up(xs, off, sg, su, hs2)
    c2r.expert_ffn_down(hs2, off, sd, ys2)
    assert torch.equal(h[:n], h2[:n]) and torch.equal(y[:n], y2[:n]) and not h[n:].any() and not y[n:].any()
    assert hs.any() and torch.equal(hs, hs2[:T]) and torch.equal(ys, ys2[:T])


# The longest walk of the gate/up pass follows from the experts in use, 22 of 60 with 44 column blocks each beside the shared expert's 176: 1144
# items for 512 workgroups.  Two walks of three on one CU, where no CU needs more than five items, made this pass 18 % slower than with
# 20 experts (59 and 70 us); with the longer walks on CUs of their own it is 5 % (59 and 62), the weights being 9 % more.
def test_mid_walks_of_a_few_more_experts():
    from paper_2504_01337_amd import c2r
    T, K, E, d, F, Fs = 24, 4, 60, 2048, 1408, 5632
    r = lambda *s: torch.randn(s, device="cuda", dtype=torch.bfloat16) * 0.02
    x, wg, wu, sg, su = r(T, d), r(E, F, d), r(E, F, d), r(1, Fs, d), r(1, Fs, d)
    h, hs = r(T * K, F), r(T, Fs)
    perm = torch.arange(T * K, dtype=torch.int32, device="cuda")
    assert ffn_two_problems(0, E, T * K, T) == (32, 32)

    def offsets(used, first):  # 96 rows of `used` experts from `first` on
        n = np.zeros(E, dtype=np.int64)
        n[first:first + used] = np.diff(np.linspace(0, T * K, used + 1).round())
        return dev(np.concatenate([[0], np.cumsum(n)]).astype(np.int32))

    best = {}
    for used in (20, 22):
        offs = [offsets(used, first) for first in (0, 30)]  # (in turn, so that the weights come from memory)
        times = []
        for _ in range(20):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for i in range(8):
                c2r.expert_ffn_gate_up_with_shared(x, perm, K, offs[i & 1], wg, wu, h, sg, su, hs)
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best[used] = min(times)
    assert best[22] < 1.11 * best[20]
