"""Router of large batches on the matrix pipe: the stream of sub-tiles that runs on across the 256-wide chunks, in both forms (chunk
results summed in registers, or stored one by one), logits bit-exact in the declared order."""
import numpy as np
import pytest

from paper_2504_01337_amd import workloads as wl
from helpers import GATE_RTOL, dev, host, select_limit

pytestmark = pytest.mark.gpu


# summed in registers (from 25025 tokens on, 32705 with up to 32 experts): whole chunks, a ragged last one, one expert block and two; stored: one
# chunk per workgroup and two (an even and an odd number of chunks, a ragged last one), the remainders of tokens and experts
@pytest.mark.parametrize("T,E,d,dtype", [
    (32768, 60, 512, "bf16"), (32705, 33, 520, "bf16"), (32769, 20, 768, "f32"), (40001, 64, 264, "f32"),
    (12353, 60, 776, "bf16"), (16400, 40, 1024, "bf16"), (16383, 61, 1100 // 8 * 8, "f32"), (16390, 18, 1288, "bf16"),
    (12289, 17, 256, "bf16"),
    # stored, tiles of 32 experts: a pipeline per chunk, whole chunks and a ragged last one
    (12290, 16, 776, "bf16"), (8193, 31, 1032, "f32"), (6200, 24, 2048, "bf16"),
    # 64-token workgroups of half the experts per wave (the third and the fifth half round)
    (33001, 60, 776, "bf16"), (65700, 34, 512, "bf16"), (36000, 61, 520, "f32"),
    # the last and the first batches of the rules: chunks stored / summed, workgroups of 128 / 64 tokens
    (25024, 60, 520, "bf16"), (25025, 60, 520, "bf16"), (32704, 20, 520, "bf16"), (32705, 20, 520, "bf16"),
    (32768, 33, 512, "bf16"), (32769, 33, 512, "bf16"), (49152, 36, 512, "bf16"), (49153, 36, 512, "bf16")])
def test_large_route_logits_bit_exact(orc, T, E, d, dtype):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E + d)
    x = rng.standard_normal((T, d)).astype(np.float32) * np.exp2(rng.integers(-6, 7, size=(T, 1))).astype(np.float32)
    x = wl.round_bf16(x) if dtype == "bf16" else x
    Wg = rng.standard_normal((d, E)).astype(np.float32)
    bias = rng.standard_normal(E).astype(np.float32)
    idx, _, logits = c2r.route(dev(x, dtype), dev(Wg), dev(bias), 4, None, want_logits=True)
    ref = orc.logits_canon_f32(x, Wg, bias)
    assert np.array_equal(host(logits), ref)
    assert np.array_equal(host(idx), orc.route(ref, 4)[0])


# selection from one chunk result per token, past 8192 tokens: ties and values a few bit patterns apart (small integers and a router
# whose columns are nearly alike), NaN and infinite logits, lists and none, fewer slots than four, partial tiles of 64 tokens
@pytest.mark.parametrize("T,E,K,dtype", [(8193, 60, 4, "bf16"), (9000, 64, 4, "f32"), (8200, 17, 3, "bf16"), (8256, 36, 1, "f32"),
                                         (8300, 12, 2, "bf16"), (8250, 4, 4, "f32")])
def test_large_selection_from_one_chunk(orc, T, E, K, dtype):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    x = rng.integers(-2, 3, size=(T, 64)).astype(np.float32)
    x[::3] = wl.round_bf16(rng.standard_normal((len(x[::3]), 64)).astype(np.float32))
    Wg = np.repeat(rng.standard_normal((64, 1)), E, axis=1) * (1 + 1e-6 * rng.integers(0, 9, size=(1, E)))
    Wg[:, ::2] = rng.integers(-2, 3, size=Wg[:, ::2].shape)
    Wg = Wg.astype(np.float32)
    x[5], x[77] = np.inf, np.nan
    for bias in (None, np.where(rng.random(E) < 0.1, np.float32(-np.inf), rng.standard_normal(E)).astype(np.float32)):
        lists = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, E // 3)] for e in range(E)]).astype(np.int32)
        if E > 8:
            lists[3, 0] = lists[3, 1]
        for cl in (None, lists):
            gl = None if cl is None else np.concatenate([np.full((E, 1), -1, np.int32), cl, np.full((E, 1), E, np.int32)], axis=1)
            idx, gates, logits = c2r.route(dev(x, dtype), dev(Wg), None if bias is None else dev(bias), K,
                                           None if gl is None else dev(gl), want_logits=True)
            ri, rg = orc.route(host(logits), K, cl)
            assert np.array_equal(host(idx), ri)
            # logits of up to some hundred apart: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero
            np.testing.assert_allclose(host(gates), rg, rtol=114 / 34 * GATE_RTOL, atol=1e-37)


# selection from several chunk results, by sixteen lanes per token and by four (the sizes on either side of the rule: 16 and 32 experts; 2048, 4096
# and 8192 tokens; 2 and 8 slots), few slots, five to eight and more; lists of more than sixteen entries with the expert itself, duplicates and
# entries out of range; ties, NaN and infinite logits
@pytest.mark.parametrize("T,E,K,d", [
    (65, 8, 8, 1032), (300, 16, 5, 776), (300, 16, 16, 520), (2048, 20, 4, 520), (2049, 20, 4, 520), (2050, 32, 8, 264), (2050, 32, 9, 264),
    (4096, 60, 2, 776), (4097, 60, 2, 776), (4100, 33, 1, 264), (8192, 40, 3, 520), (8192, 17, 13, 264), (8193, 12, 9, 264), (8193, 60, 4, 776),
    (8200, 64, 17, 520), (8256, 61, 6, 520), (9000, 60, 8, 776), (9000, 36, 5, 264), (16400, 60, 4, 776)])
def test_selection_from_several_chunks(orc, T, E, K, d):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E + K)
    x = rng.integers(-2, 3, size=(T, d)).astype(np.float32)
    x[::3] = rng.standard_normal((len(x[::3]), d)).astype(np.float32)
    x[::7, 8:] = 0.0
    x[5], x[44] = np.inf, np.nan
    Wg = rng.integers(-2, 3, size=(d, E)).astype(np.float32)
    Wg[::5] = 0.03 * rng.standard_normal(Wg[::5].shape)
    bias = np.where(rng.random(E) < 0.1, np.float32(-np.inf), rng.integers(-2, 3, size=E)).astype(np.float32)
    cl = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, min(E - 1, 18))] for e in range(E)]).astype(np.int32)
    gl = np.concatenate([np.full((E, 1), -1), cl[:, :1], cl, np.arange(E)[:, None], np.full((E, 1), E)], axis=1).astype(np.int32)
    for b in (None, bias):
        for c, g in ((None, None), (cl, gl)):
            idx, gates, logits = c2r.route(dev(x), dev(Wg), None if b is None else dev(b), K, None if g is None else dev(g), want_logits=True)
            ri, rg = orc.route(host(logits), K, c)
            assert np.array_equal(host(idx), ri)
            # logits of up to some hundred apart: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero (and, for K up to
            # 17, nine more roundings of the sum)
            np.testing.assert_allclose(host(gates), rg, rtol=123 / 34 * GATE_RTOL, atol=1e-37)


# undecided tokens in groups of 64 (none, a few that the wave scans together, one more, all): rows of zeros, rows with equal logits of either sign,
# an expert masked by -infinity, NaN; a partial last group
@pytest.mark.parametrize("E,K", [(60, 4), (64, 4), (36, 3), (16, 2), (8, 4), (5, 4)])
def test_large_selection_of_undecided_tokens(orc, E, K):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(E * K)
    T, d = 64 * 130 - 17, 64
    x = rng.standard_normal((T, d)).astype(np.float32)
    Wg = (0.25 * rng.standard_normal((d, E))).astype(np.float32)  # (logits of deviation 2: kept ones differ by less than GATE_RTOL's 24)
    Wg[0] = 1.0
    few = [0, 1, 2, E // 8, E // 8 + 1, 20, 64]
    for g in range(130):
        for t in g * 64 + rng.permutation(64)[:few[g % len(few)]]:
            if t < T:
                x[t] = 0.0
                if g % 3:
                    x[t, 0] = [1.5, -2.25, 1.1, np.nan][rng.integers(0, 4)]   # (1.1: its low bits are not zero)
    masked = np.zeros(E, dtype=np.float32)
    masked[E // 2] = -np.inf
    for bias in (None, masked):
        idx, gates, logits = c2r.route(dev(x), dev(Wg), None if bias is None else dev(bias), K, want_logits=True)
        ri, rg = orc.route(host(logits), K)
        assert np.array_equal(host(idx), ri)
        np.testing.assert_allclose(host(gates), rg, rtol=GATE_RTOL, atol=1e-37)


# a batch of padding (rows of zeros) takes the time of any other (3.5 times it with one undecided token after the other), and so does a router
# with an expert masked by -infinity
def test_large_selection_of_padding_costs_no_multiple():
    import torch
    from paper_2504_01337_amd import c2r
    T, E, d = 65536, 60, 64
    x, Wg = torch.randn((T, d), device="cuda"), torch.randn((d, E), device="cuda")
    bias = torch.zeros(E, device="cuda")
    masked = bias.clone()
    masked[7] = float("-inf")
    best = []
    for a, b in ((x, bias), (torch.zeros_like(x), bias), (x, masked)):
        times = []
        for _ in range(12):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(8):
                c2r.route(a, Wg, b, 4)
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best.append(min(times))
    assert max(best[1:]) < 2 * best[0]


# One token more than a round of the chip's workgroups costs the busiest CU one more chunk: 1.00 times the time of 8192 tokens with 16 experts of
# d 4096 (34.2 us; 42.2 against 32.7 when chunks went in pairs wherever that left a workgroup per CU), 1.24 times with 60 of d 2048 (33.9 and
# 41.8 us, 49.7 in pairs)
@pytest.mark.parametrize("E,d,most", [(16, 4096, 1.15), (60, 2048, 1.36)])
def test_large_route_of_one_more_token(E, d, most):
    import torch
    from paper_2504_01337_amd import c2r
    Wg = torch.randn((d, E), device="cuda")
    best = []
    for T in (8192, 8193):
        x = torch.randn((T, d), device="cuda", dtype=torch.bfloat16)
        ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_ROUTE, T, d, E, 4, 0, c2r.BF16), dtype=torch.uint8, device="cuda")
        out = torch.empty((T, 4), dtype=torch.int32, device="cuda"), torch.empty((T, 4), device="cuda")
        times = []
        for _ in range(20):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(8):
                c2r.route(x, Wg, None, 4, ws=ws, out=out)
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best.append(min(times))
    assert best[1] < most * best[0]


# selection by the waves that have the sums in registers (no logits asked for, up to four slots): two blocks of 32 experts and one, the first and a
# ragged number of tokens, one slot to four; lists with the expert itself, duplicates and entries out of range, short ones and none; ties,
# logits of equal upper bits, NaN and infinite ones, rows of zeros one by one and in numbers, experts masked by -infinity; outputs that
# stand in the place of the input's memory or are not aligned, which take the two launches
@pytest.mark.parametrize("T,E,K,d,dtype", [(25025, 60, 4, 520, "bf16"), (32768, 64, 4, 512, "bf16"), (25100, 33, 3, 264, "f32"), (32705, 20, 4, 512, "bf16"),
                                           (32721, 32, 2, 264, "f32"), (25030, 61, 1, 512, "bf16"), (50000, 36, 4, 512, "bf16"), (32710, 17, 4, 520, "bf16")])
def test_selection_beside_the_sums(orc, T, E, K, d, dtype):
    import torch
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    x = rng.integers(-2, 3, size=(T, d)).astype(np.float32)
    x[::3] = wl.round_bf16(rng.standard_normal((len(x[::3]), d)).astype(np.float32))
    x[::11, 8:] = 0.0
    x[1000:1040], x[64 * 200 + 5], x[5], x[77], x[T - 1] = 0.0, 0.0, np.inf, np.nan, np.inf
    Wg = rng.integers(-2, 3, size=(d, E)).astype(np.float32)
    Wg[::5] = 0.03 * rng.standard_normal(Wg[::5].shape)
    Wg[:, 1] = Wg[:, 0] * np.float32(1 + 2.0 ** -22)
    bias = np.where(rng.random(E) < 0.1, np.float32(-np.inf), rng.integers(-2, 3, size=E)).astype(np.float32)
    cl = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, E // 3)] for e in range(E)]).astype(np.int32)
    gl = np.concatenate([np.full((E, 1), -1), cl[:, :1], cl, np.arange(E)[:, None], np.full((E, 1), E)], axis=1).astype(np.int32)
    short = np.full((E, 4), -1, dtype=np.int32)
    short[:, 0] = (np.arange(E) + 1) % E
    xd, wd = dev(x, dtype), dev(Wg)
    for b in (None, bias):
        bd = None if b is None else dev(b)
        for c, g in ((None, None), (cl, gl), (None, short)):
            gd = None if g is None else dev(g)
            two = c2r.route(xd, wd, bd, K, gd, want_logits=True)  # (the two launches; the oracle takes no lists that are too short)
            ri, rg = (host(two[0]), host(two[1])) if g is short else orc.route(host(two[2]), K, c)
            apart = torch.empty(T * K + 1, dtype=torch.int32, device="cuda"), torch.empty(T * K + 1, device="cuda")
            for out in (None, tuple(a[1:].view(T, K) for a in apart)):
                idx, gates, _ = c2r.route(xd, wd, bd, K, gd, out=out)
                assert np.array_equal(host(idx), ri)
                # (logits up to some hundred apart: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero)
                np.testing.assert_allclose(host(gates), rg, rtol=114 / 34 * GATE_RTOL, atol=1e-37)
    x2 = xd.clone()
    idx = x2.view(-1).view(torch.int32)[:T * K].view(T, K)
    got = c2r.route(x2, wd, None, K, None, out=(idx, torch.empty((T, K), device="cuda")))
    assert np.array_equal(host(got[0]), orc.route(host(c2r.route(xd, wd, None, K, want_logits=True)[2]), K)[0])


# experts masked by -infinity in the same selection: one, every second, all but two, all; by the type's lowest value; lists of any experts and, for half
# of the experts, of masked ones alone (what is left to choose is then masked itself); rows of zeros among the others, a NaN and an infinity
@pytest.mark.parametrize("T,E,K,d,dtype", [(25025, 60, 4, 512, "bf16"), (25100, 33, 3, 264, "f32"), (32705, 20, 2, 512, "bf16"), (32721, 32, 4, 264, "f32"),
                                           (25030, 64, 1, 264, "bf16")])
def test_masked_experts_beside_the_sums(orc, T, E, K, d, dtype):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    x = wl.round_bf16(rng.standard_normal((T, d)).astype(np.float32))
    x[1000:1100], x[::97], x[5, 3], x[77, 0] = 0.0, 0.0, np.inf, np.nan
    Wg = (0.25 * rng.standard_normal((d, E))).astype(np.float32)
    order = rng.permutation(E)
    xd, wd = dev(x, dtype), dev(Wg)
    for out, value in ((order[:1], -np.inf), (order[::2], -np.inf), (order[2:], -np.inf), (order, -np.inf), (order[::2], np.finfo(np.float32).min)):
        bias = rng.standard_normal(E).astype(np.float32)
        bias[out] = value
        lists = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, E // 3)] for e in range(E)]).astype(np.int32)
        n = max(K - 1, 1)
        gone = np.stack([rng.permutation(out[out != e] if e % 2 and len(out) > n else np.delete(np.arange(E), e))[:n] for e in range(E)]).astype(np.int32)
        for cl in (None, lists, gone):
            bd, cd = dev(bias), None if cl is None else dev(cl)
            ri, rg = orc.route(host(c2r.route(xd, wd, bd, K, cd, want_logits=True)[2]), K, cl)
            idx, gates, _ = c2r.route(xd, wd, bd, K, cd)
            assert np.array_equal(host(idx), ri)
            # (logits up to some hundred apart: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero)
            np.testing.assert_allclose(host(gates), rg, rtol=114 / 34 * GATE_RTOL, atol=1e-37)


# ... which costs what any other batch does (1.3 times it, 8 us of 28, with every token scanned by the literal rule), and so do rows of zeros
@pytest.mark.parametrize("lists", [False, True])
def test_masked_experts_beside_the_sums_cost_no_more(lists):
    import torch
    from paper_2504_01337_amd import c2r
    T, E, d = 32768, 60, 512
    x, Wg = torch.randn((T, d), device="cuda", dtype=torch.bfloat16), torch.randn((d, E), device="cuda")
    plain = torch.zeros(E, device="cuda")
    masked = plain.clone()
    masked[7] = float("-inf")
    cl = dev(np.stack([np.random.default_rng(e).permutation(np.delete(np.arange(E), e))[:16] for e in range(E)]).astype(np.int32)) if lists else None
    ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_ROUTE, T, d, E, 4, 0, c2r.BF16), dtype=torch.uint8, device="cuda")
    out = torch.empty((T, 4), dtype=torch.int32, device="cuda"), torch.empty((T, 4), device="cuda")
    best = []
    for a, bias in ((x, plain), (x, masked), (torch.zeros_like(x), plain)):
        times = []
        for _ in range(20):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(8):
                c2r.route(a, Wg, bias, 4, cl, ws=ws, out=out)
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best.append(min(times))
    assert max(best[1:]) < 1.15 * best[0]


# ... and from some number of tokens on they do not: the last and the first batches of the rules (without lists, with as many experts as a wave
# selects from or fewer; with lists and short rows)
UP_TO, MOST, NARROW = select_limit("UP_TO"), select_limit("MOST_UP_TO"), select_limit("NARROW_UP_TO")


@pytest.mark.parametrize("T,E,K,lists", [(UP_TO, 20, 4, False), (UP_TO + 1, 20, 4, False), (UP_TO, 56, 2, False), (UP_TO + 1, 28, 3, False), (MOST, 29, 4, False),
                                         (MOST + 1, 29, 4, False), (MOST, 57, 4, False), (MOST + 1, 60, 1, False), (NARROW, 9, 4, True),
                                         (NARROW + 1, 9, 4, True), (NARROW + 1, 33, 4, True), (NARROW + 1, 30, 2, True)])
def test_selection_beside_the_sums_up_to_a_batch(orc, T, E, K, lists):
    from paper_2504_01337_amd import c2r
    rng = np.random.default_rng(T + E)
    x = rng.standard_normal((T, 264), dtype=np.float32)
    x[:64], x[T - 40:T - 30], x[7, 3] = 0.0, 0.0, np.inf
    xd, Wg = dev(x, "bf16"), dev((0.25 * rng.standard_normal((264, E))).astype(np.float32))
    bias = rng.standard_normal(E).astype(np.float32)
    bias[E // 2] = -np.inf
    cl = np.stack([rng.permutation(np.delete(np.arange(E), e))[:max(K, E // 3)] for e in range(E)]).astype(np.int32) if lists else None
    for b in (None, dev(bias)):
        cd = None if cl is None else dev(cl)
        ri, rg = orc.route(host(c2r.route(xd, Wg, b, K, cd, want_logits=True)[2]), K, cl)
        idx, gates, _ = c2r.route(xd, Wg, b, K, cd)
        assert np.array_equal(host(idx), ri)
        # (logits up to some hundred apart: the bound of GATE_RTOL with |a_s| up to 104, where a gate is flushed to zero)
        np.testing.assert_allclose(host(gates), rg, rtol=114 / 34 * GATE_RTOL, atol=1e-37)


# A batch of many rounds costs no more than in two launches, which results that stand in the place of the last rows take (10^6 tokens of 9 experts
# 231 us; 278 with a selection at the end of every round)
def test_large_route_costs_no_more_than_in_two_launches():
    import torch
    from paper_2504_01337_amd import c2r
    T, E, d = 1000000, 9, 264
    x, Wg, bias = torch.randn((T, d), device="cuda", dtype=torch.bfloat16), torch.randn((d, E), device="cuda"), torch.randn(E, device="cuda")
    ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_ROUTE, T, d, E, 4, 0, c2r.BF16), dtype=torch.uint8, device="cuda")
    gates = torch.empty((T, 4), device="cuda")
    best = []
    for idx in (x.view(-1).view(torch.int32)[-T * 4:].view(T, 4), torch.empty((T, 4), dtype=torch.int32, device="cuda")):
        times = []
        for _ in range(12):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(4):
                c2r.route(x, Wg, bias, 4, ws=ws, out=(idx, gates))
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best.append(min(times))
    assert best[1] < 1.1 * best[0]
