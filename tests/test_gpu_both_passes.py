"""The expert FFN's two passes in one launch (ffn_bf16_dma.hip) against the same passes in a launch each: the same tiles, so the same
bits.  Several times over the same buffers: the launch's counters have to be clear again, and h is rewritten while it is in caches."""
import numpy as np
import pytest
import torch

from helpers import dev, ffn_both_limit, ffn_kernel, ffn_shared_schedule, ffn_tiles, ffn_tiles_limit

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def c2r():
    from paper_2504_01337_amd import c2r as m
    m.lib()
    return m


def _weights(rng, *shapes):
    return [dev((rng.standard_normal(s) * 0.05).astype(np.float32), "bf16") for s in shapes]


# full, short and tiny tiles and empty groups; one group; fewer M-tiles than XCDs; rows not all in use; a column tail (d 192); one
# slice (64); as many M-tiles as there are counters (1024) and one more (two launches); N-tiles enough for the rule to take one launch
@pytest.mark.parametrize("d,F,sizes,cap", [
    (64, 2560, [256, 257, 511, 129, 128, 64, 65, 1, 0, 1000], 2600), (64, 8192, [3000, 0, 1], 3001), (192, 7744, [700], 800), (512, 8192, [300, 299], 599),
    (2048, 1408, [796, 624, 464, 341, 136, 63, 7, 0], 3400), (128, 448, [900] * 15, 13500), (64, 64, [131000, 130000], 1022 * 256),
    (64, 64, [131000, 130500], 1023 * 256)])
def test_routed_groups(c2r, d, F, sizes, cap):
    rng = np.random.default_rng(d + F)
    E, n, K = len(sizes), sum(sizes), 2
    assert ffn_kernel(0, E, cap, F) == ffn_kernel(1, E, cap, d) == "tile" and ffn_tiles(E, cap, F) >= ffn_tiles_limit()
    T = (cap + K - 1) // K
    x = dev(rng.standard_normal((T, d)).astype(np.float32), "bf16")
    perm = dev(np.concatenate([rng.permutation(T * K)[:n], np.full(cap - n, -1)]).astype(np.int32))
    offsets = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    wg, wu, wd = _weights(rng, (E, F, d), (E, F, d), (E, d, F))
    h, y = (torch.full((cap, c), 7.0, dtype=torch.bfloat16, device="cuda") for c in (F, d))
    c2r.expert_ffn_gate_up_gather(x, perm, K, offsets, wg, wu, h)
    c2r.expert_ffn_down(h, offsets, wd, y)
    ws = torch.full((c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, cap, d, E, 1, F, c2r.BF16),), 255, dtype=torch.uint8, device="cuda")
    for _ in range(4):
        got = torch.full((cap, d), 7.0, dtype=torch.bfloat16, device="cuda")
        ws.fill_(255)  # (NaNs: a row of h that is read before it is there shows)
        c2r.expert_ffn_gather(x, perm, K, offsets, wg, wu, wd, ws=ws, out=got)
        assert torch.equal(got, y)


# a shared expert beside the routed groups, through the layer call: every row of it and of the routed experts
@pytest.mark.parametrize("T,d,F,Fs", [(1300, 128, 832, 2560), (2500, 256, 448, 1024), (5000, 64, 192, 64)])
def test_layer_with_shared_expert(c2r, T, d, F, Fs):
    rng = np.random.default_rng(T)
    E, K = 16, 4
    assert ffn_tiles(E, T * K, F) + ffn_tiles(1, T, Fs) >= ffn_tiles_limit()
    x = dev(rng.standard_normal((T, d)).astype(np.float32), "bf16")
    Wg = dev((rng.standard_normal((d, E)) * 0.05 + np.linspace(0, 0.1, E)).astype(np.float32))
    collab = dev(np.stack([np.delete(np.arange(E), e) for e in range(E)]).astype(np.int32))
    weights = _weights(rng, (E, F, d), (E, F, d), (E, d, F))
    shared = _weights(rng, (1, Fs, d), (1, Fs, d), (1, d, Fs))
    a, b = (c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, Wg, None, collab, *weights, shared=tuple(shared), fuse_shared=f) for f in (True, False))
    assert a.fuse_shared and not b.fuse_shared
    ref = b.forward(x).clone()
    for _ in range(4):
        a.h.fill_(float("nan"))
        a.h_shared.fill_(float("nan"))
        assert torch.equal(a.forward(x), ref)
        assert torch.equal(a.y_perm, b.y_perm) and torch.equal(a.y_shared, b.y_shared)


BESIDE, EARLY, LONG, LONGEST = (ffn_both_limit(n) for n in ("BESIDE", "EARLY_UP_TO", "EARLY_LONG_UP_TO", "EARLY_LONGEST_UP_TO"))


# the layer call on either side of the rules that give a pass to this kernel or that: rows of a shared expert (its down tiles early), 125 likely
# rows per expert, 4096 rows allotted to a device with a part of the experts.  The same bits as stage by stage, where every pass chooses by the
# rows allotted.
@pytest.mark.parametrize("T,E,El,K,Fs", [(LONG, 60, 60, 4, 2176), (LONG + 1, 60, 60, 4, 2176),
                                         (390, 60, 60, 4, 192), (391, 60, 60, 4, 192), (501, 16, 16, 4, 0), (504, 16, 16, 4, 0), (600, 16, 16, 4, 0),
                                         (1000, 60, 15, 4, 0), (1024, 60, 15, 4, 0), (1025, 60, 15, 4, 0), (2100, 60, 15, 4, 0), (15500, 60, 15, 4, 0),
                                         (16384, 60, 15, 4, 0), (17000, 60, 15, 4, 0), (300, 64, 1, 4, 0)])
def test_layer_at_the_limits_of_the_kernels(c2r, T, E, El, K, Fs):
    rng = np.random.default_rng(T + E)
    d, F = 128, 704
    x = dev(rng.standard_normal((T, d)).astype(np.float32), "bf16")
    Wg = dev((rng.standard_normal((d, E)) * 0.05 + np.linspace(0, 0.1, E)).astype(np.float32))
    slots = None
    if El < E:
        slots = np.full(E, -1, dtype=np.int32)
        slots[rng.permutation(E)[:El]] = np.arange(El)
        slots = dev(slots)
    shared = tuple(_weights(rng, (1, Fs, d), (1, Fs, d), (1, d, Fs))) if Fs else None
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, Wg, None, None, *_weights(rng, (El, F, d), (El, F, d), (El, d, F)), local_slot=slots, E_local=El,
                         shared=shared)
    ref = layer.forward(x, trace={}).clone()
    for _ in range(3):
        layer.h.fill_(float("nan"))
        assert torch.equal(layer.forward(x), ref)


# widths that are no whole slices: the first pass keeps the padding columns of h at zero in its workspace.  Zero weights there in launches of
# their own give the same sums.
@pytest.mark.parametrize("d,F,sizes,cap", [(128, 688, [900, 513, 130, 0, 64, 1] * 4, 6500), (64, 2568, [700, 257, 33, 1000], 2000), (192, 7688, [700], 800)])
def test_padded_widths(c2r, d, F, sizes, cap):
    rng = np.random.default_rng(d + F)
    E, n, K, Fp = len(sizes), sum(sizes), 2, -(-F // 64) * 64
    assert Fp > F and ffn_kernel(0, E, cap, Fp) == ffn_kernel(1, E, cap, d) == "tile" and ffn_tiles(E, cap, Fp) >= ffn_tiles_limit()
    T = (cap + K - 1) // K
    x = dev(rng.standard_normal((T, d)).astype(np.float32), "bf16")
    perm = dev(np.concatenate([rng.permutation(T * K)[:n], np.full(cap - n, -1)]).astype(np.int32))
    offsets = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))
    wg, wu, wd = _weights(rng, (E, F, d), (E, F, d), (E, d, F))
    pad = lambda w, dim: torch.cat([w, torch.zeros([Fp - F if i == dim else s for i, s in enumerate(w.shape)], dtype=w.dtype, device="cuda")], dim).contiguous()
    h, y = (torch.full((cap, c), 7.0, dtype=torch.bfloat16, device="cuda") for c in (Fp, d))
    c2r.expert_ffn_gate_up_gather(x, perm, K, offsets, pad(wg, 1), pad(wu, 1), h)
    c2r.expert_ffn_down(h, offsets, pad(wd, 2), y)
    x_perm = torch.zeros((cap, d), dtype=torch.bfloat16, device="cuda")
    x_perm[:n] = x[(perm[:n] // K).long()]
    ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, cap, d, E, 1, F, c2r.BF16), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        for call in (lambda o: c2r.expert_ffn_gather(x, perm, K, offsets, wg, wu, wd, ws=ws, out=o),
                     lambda o: c2r.expert_ffn(x_perm, offsets, wg, wu, wd, ws=ws, out=o)):
            got = torch.full((cap, d), 7.0, dtype=torch.bfloat16, device="cuda")
            ws.fill_(255)
            assert torch.equal(call(got), y)


# two layers on two streams: a tile of either waits only for workgroups of its own launch that run
def test_beside_another_launch(c2r):
    layers, xs, refs = [], [], []
    for seed, (T, d, F, Fs) in enumerate([(1300, 128, 832, 2560), (3000, 256, 448, 1024)]):
        rng = np.random.default_rng(seed)
        E, K = 16, 4
        assert ffn_tiles(E, T * K, F) + ffn_tiles(1, T, Fs) >= ffn_tiles_limit()
        Wg = dev((rng.standard_normal((d, E)) * 0.05 + np.linspace(0, 0.1, E)).astype(np.float32))
        layers.append(c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, Wg, None, None, *_weights(rng, (E, F, d), (E, F, d), (E, d, F)),
                                   shared=tuple(_weights(rng, (1, Fs, d), (1, Fs, d), (1, d, Fs)))))
        xs.append(dev(rng.standard_normal((T, d)).astype(np.float32), "bf16"))
        refs.append(layers[-1].forward(xs[-1]).clone())
    streams = [torch.cuda.Stream() for _ in layers]
    outs = [[torch.empty_like(r) for _ in range(12)] for r in refs]
    torch.cuda.synchronize()
    for i in range(12):
        for layer, x, stream, out in zip(layers, xs, streams, outs):
            with torch.cuda.stream(stream):
                out[i].copy_(layer.forward(x))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for out, ref in zip(outs, refs) for o in out)


# a shared expert's down tiles ahead of routed gate/up tiles: the last rows of the rule for long contractions and the first beyond it, a down pass cut
# to 64 rows, nothing but the shared expert's in a list's first round; and such layers as take a launch per pass or the down tiles late; two
# layers on two streams, each of whose waits must end by workgroups of its own launch
@pytest.mark.parametrize("T,E,d,F,Fs", [(LONG, 60, 128, 704, 2176), (LONG + 1, 60, 128, 704, 2176), (512, 2, 64, 2048, 16448),
                                        (257, 60, 128, 704, 2816), (420, 60, 2048, 320, 5632), (640, 60, 256, 1408, 1024), (641, 60, 256, 1408, 1024),
                                        (300, 60, 128, 1408, 64), (512, 16, 192, 192, 16448), (257, 2, 64, 11264, 8192)])
def test_shared_expert_down_tiles_early(c2r, T, E, d, F, Fs):
    K = min(E, 4)
    assert ffn_tiles(E, T * K, F) + ffn_tiles(1, T, Fs) >= ffn_tiles_limit() and ffn_kernel(0, 1, T, Fs) == "tile"
    layers, xs, refs = [], [], []
    for seed in (T, T + 1):
        rng = np.random.default_rng(seed)
        xs.append(dev(rng.standard_normal((T, d)).astype(np.float32), "bf16"))
        Wg = dev((rng.standard_normal((d, E)) * 0.05 + np.linspace(0, 0.1, E)).astype(np.float32))
        weights, shared = _weights(rng, (E, F, d), (E, F, d), (E, d, F)), tuple(_weights(rng, (1, Fs, d), (1, Fs, d), (1, d, Fs)))
        a, b = (c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, Wg, None, None, *weights, shared=shared, fuse_shared=f) for f in (True, False))
        layers.append(a)
        refs.append(b.forward(xs[-1]).clone())
        for _ in range(3):
            a.h.fill_(float("nan"))
            a.h_shared.fill_(float("nan"))
            assert torch.equal(a.forward(xs[-1]), refs[-1])
            assert torch.equal(a.y_perm, b.y_perm) and torch.equal(a.y_shared, b.y_shared)
    streams = [torch.cuda.Stream() for _ in layers]
    outs = [[torch.empty_like(r) for _ in range(8)] for r in refs]
    torch.cuda.synchronize()
    for i in range(8):
        for layer, x, stream, out in zip(layers, xs, streams, outs):
            with torch.cuda.stream(stream):
                out[i].copy_(layer.forward(x))
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for out, ref in zip(outs, refs) for o in out)


# the rules for as many rows of a shared expert as ffn_mid's down pass takes: the last rows and the first (a launch per pass or one; the down tiles
# early or late, for a shared contraction of under three times the routed one, of three and of more than four), one expert and one step of the shared
# contraction more or
# less (down tiles, k-slices), a narrow model; 64-row down tiles and whole ones, one column tile of gate/up.  The same bits as in launches of their own.
@pytest.mark.parametrize("T,E,d,F,Fs,schedule", [
    (BESIDE, 60, 1280, 704, 2048, "two"), (BESIDE + 1, 60, 1280, 704, 2048, "early"), (EARLY, 60, 1280, 704, 2048, "early"), (EARLY + 1, 60, 1280, 704, 2048, "late"),
    (EARLY + 1, 60, 1280, 704, 2112, "early"), (511, 60, 1280, 704, 2112, "early"), (300, 60, 1280, 1408, 64, "early"),
    (LONG, 60, 128, 704, 2816, "early"), (LONG + 1, 60, 128, 704, 2816, "late"), (LONGEST, 60, 128, 704, 2880, "early"), (LONGEST + 1, 60, 128, 704, 2880, "late"),
    (257, 52, 1024, 704, 704, "early"), (257, 50, 1024, 704, 704, "two"), (300, 60, 1280, 704, 2816, "early"), (300, 60, 1280, 704, 2880, "two"),
    (300, 60, 128, 704, 2816, "two")])
def test_schedules_beside_a_shared_expert(c2r, T, E, d, F, Fs, schedule):
    assert ffn_shared_schedule(T, E, 4, d, F, Fs) == schedule
    g = torch.Generator(device="cuda")
    g.manual_seed(T + Fs)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.05)
    weights, shared = [normal(E, F, d), normal(E, F, d), normal(E, d, F)], (normal(1, Fs, d), normal(1, Fs, d), normal(1, d, Fs))
    x, Wg = normal(T, d).mul_(20), torch.randn((d, E), generator=g, device="cuda")
    a, b = (c2r.C2RLayer(T, d, E, 4, F, torch.bfloat16, Wg, None, None, *weights, shared=shared, fuse_shared=f) for f in (True, False))
    ref = b.forward(x).clone()
    for _ in range(4):
        a.h.fill_(float("nan"))
        a.h_shared.fill_(float("nan"))
        assert torch.equal(a.forward(x), ref)
        assert torch.equal(a.y_perm, b.y_perm) and torch.equal(a.y_shared, b.y_shared)


# A narrow model's layer takes no longer than its two passes and the stages around them (62 us; 86 with both passes in one launch, whose few
# down tiles are chains that nothing runs beside)
def test_narrow_model_costs_no_more_than_its_passes(c2r):
    T, E, K, d, F, Fs = 363, 8, 1, 512, 4096, 2048
    normal = lambda *shape: torch.randn(shape, device="cuda", dtype=torch.bfloat16)
    weights, shared = (normal(E, F, d), normal(E, F, d), normal(E, d, F)), (normal(1, Fs, d), normal(1, Fs, d), normal(1, d, Fs))
    x, Wg = normal(T, d), torch.randn((d, E), device="cuda")
    layer = c2r.C2RLayer(T, d, E, K, F, torch.bfloat16, Wg, None, None, *weights, shared=shared)
    layer.forward(x)
    idx = layer.idx.clone()
    _, offsets, perm, _ = c2r.permute(None, idx, E)[:4]
    h, hs = torch.empty((T * K, F), dtype=torch.bfloat16, device="cuda"), torch.empty((T, Fs), dtype=torch.bfloat16, device="cuda")
    y, ys = torch.empty((T * K, d), dtype=torch.bfloat16, device="cuda"), torch.empty((T, d), dtype=torch.bfloat16, device="cuda")

    def passes():
        c2r.expert_ffn_gate_up_with_shared(x, perm, K, offsets, weights[0], weights[1], h, shared[0], shared[1], hs)
        c2r.expert_ffn_down_with_shared(h, offsets, weights[2], y, hs, shared[2], ys)

    best = []
    for call in (passes, lambda: layer.forward(x)):
        times = []
        for _ in range(12):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(16):
                call()
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end) / 16 * 1e3)
        best.append(min(times))
    assert best[1] < 1.15 * (best[0] + 20), best


# one group alone: both passes in one launch (more items in ffn_mid's down pass than workgroups: 511 rows of d 4160) and a launch each (as many: d 4096)
@pytest.mark.parametrize("d", [4096, 4160])
def test_lone_group_at_the_limit_of_the_down_pass(c2r, d):
    T, F = 511, 11520
    assert ffn_kernel(0, 1, T, F) == "tile" and ffn_kernel(1, 1, T, d) == "mid" and ffn_tiles(1, T, F) >= ffn_tiles_limit()
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    wg, wu, wd = (torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02) for s in ((1, F, d), (1, F, d), (1, d, F)))
    x = torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    offsets = dev(np.array([0, T], dtype=np.int32))
    h = torch.empty((T, F), dtype=torch.bfloat16, device="cuda")
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    c2r.expert_ffn_gate_up(x, offsets, wg, wu, h)
    c2r.expert_ffn_down(h, offsets, wd, y)
    for _ in range(3):
        assert torch.equal(c2r.expert_ffn(x, offsets, wg, wu, wd), y)


# One call takes no longer than its two passes by themselves where one group's down pass gives every workgroup of ffn_mid one item at most (300
# rows of d 2048, F 12288: 107 us either way; 149 in one launch of the tile kernel, whose 40 down tiles are a chain of 192 slices each)
def test_lone_group_costs_no_more_than_its_passes(c2r):
    T, d, F = 300, 2048, 12288
    wg, wu, wd = (torch.randn(s, device="cuda", dtype=torch.bfloat16) for s in ((1, F, d), (1, F, d), (1, d, F)))
    x, y = torch.randn((T, d), device="cuda", dtype=torch.bfloat16), torch.empty((T, d), device="cuda", dtype=torch.bfloat16)
    h, offsets = torch.empty((T, F), device="cuda", dtype=torch.bfloat16), dev(np.array([0, T], dtype=np.int32))
    ws = torch.empty(c2r.workspace_bytes(c2r.STAGE_EXPERT_FFN, T, d, 1, 1, F, c2r.BF16), dtype=torch.uint8, device="cuda")

    def passes():
        c2r.expert_ffn_gate_up(x, offsets, wg, wu, h)
        c2r.expert_ffn_down(h, offsets, wd, y)

    best = []
    for call in (passes, lambda: c2r.expert_ffn(x, offsets, wg, wu, wd, ws=ws, out=y)):
        times = []
        for _ in range(12):
            beg, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            beg.record()
            for _ in range(8):
                call()
            end.record()
            torch.cuda.synchronize()
            times.append(beg.elapsed_time(end))
        best.append(min(times))
    assert best[1] < 1.15 * best[0]
