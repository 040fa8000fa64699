"""Shared plumbing of the GPU parity tests: host<->device copies and the
oracle-side pipeline.  No arithmetic of the method lives here."""
import os
import re

import numpy as np
import torch

from paper_2504_01337_amd import workloads as wl


def dev(a, dtype="f32"):
    """numpy -> cuda tensor in the given storage dtype (values already representable)."""
    if a is None:
        return None
    t = torch.from_numpy(np.ascontiguousarray(a))
    if t.dtype == torch.float32 and dtype == "bf16":
        t = t.to(torch.bfloat16)
    return t.cuda()


def host(t):
    if t is None:
        return None
    t = t.detach()
    if t.dtype == torch.bfloat16:
        t = t.to(torch.float32)
    return t.cpu().numpy()


def max_rel_err(got, ref):
    """max |got - ref| / max |ref| : the error measure of the layer-output bar."""
    ref = np.asarray(ref, dtype=np.float64)
    got = np.asarray(got, dtype=np.float64)
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300))


# Relative tolerance of the fp32 gates against the oracle's fp64 gates (both from the same fp32
# logits).  A gate is exp(a_s) / sum_s' exp(a_s') with a_s = l_s - l_0 <= 0.  In fp32: a_s is one
# rounded subtraction (relative 2^-24, so exp(a_s) moves by |a_s| 2^-24 relatively), the exponential
# is good to 2 ulp, the sum of K <= 8 positive terms to (K - 1) roundings, the division to 1 ulp:
# (|a_s| + 2 + 7 + 1) 2^-24 in all.  A gate that is not flushed to zero has |a_s| < 88 in
# principle, but the workloads' logits differ by less than 24 inside a token's kept set, which
# gives (24 + 10) 2^-24 = 2.0e-6.  (1e-6 would hold only for |a_s| < 7.)
GATE_RTOL = 2e-6


def share_outside(got, ref, tol):
    """Second error measure of the layer-output bar: the share of elements whose error exceeds
    tol * (|ref| + rms(ref)), so that rows that are small next to the batch maximum count too."""
    ref = np.asarray(ref, dtype=np.float64)
    got = np.asarray(got, dtype=np.float64)
    rms = float(np.sqrt(np.mean(ref * ref)))
    return float(np.mean(np.abs(got - ref) > tol * (np.abs(ref) + rms)))


TOL = {"f32": 1e-5, "bf16": 1e-2}
# Share of elements allowed outside tol * (|ref| + rms): none in fp32.  In bf16 every output is
# rounded to 8 significant bits three times on the way (h, y_perm, y): an element's error is
# a few times 2^-9 of the magnitude of the TERMS it sums, which for an element that is itself
# near zero is a few times 2^-9 * rms, i.e. inside 1e-2 * rms but not by a wide margin, so a
# small share of elements is allowed to land outside.
SHARE_OUTSIDE_MAX = {"f32": 0.0, "bf16": 1e-4}     # measured at full size: 6e-8 .. 1e-5
# Every token's row on its own scale: max |d| over the row / max |ref| over the row.  Measured at
# full size 7.6e-3 (bf16), 1.5e-6 (fp32): a wrong row (a tile of the ragged map written to the
# wrong place, a missing term of the combine) is off by order 1.
ROW_TOL = {"f32": 1e-5, "bf16": 1.5e-2}


class OracleLayer:
    """The oracle's view of one workload: profiling -> lists -> routing -> dispatch."""

    def __init__(self, orc, w, x=None, x_prof=None):
        self.w = w
        self.Wg, self.bias = wl.router(w)
        self.x = wl.hidden(w) if x is None else x
        if w.T_profile:
            self.x_prof = wl.hidden(w, w.T_profile, stream=1) if x_prof is None else x_prof
        else:
            self.x_prof = self.x
        lp = orc.logits_canon_f32(self.x_prof, self.Wg, self.bias)
        self.idx_prof, _ = orc.route(lp, w.K)
        self.C = orc.coactivation(self.idx_prof, w.E)
        self.collab = orc.collaborators(self.C, w.Tc)
        self.logits = lp if self.x_prof is self.x else orc.logits_canon_f32(self.x, self.Wg, self.bias)
        self.idx, self.gates = orc.route(self.logits, w.K, self.collab)
        self.local_slot = wl.local_slot(w)
        self.counts, self.offsets, self.perm, self.inv_perm = orc.permute(
            self.idx, w.E, self.local_slot, w.n_local)


def _csrc(name):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    with open(os.path.join(root, "paper_2504_01337_amd", "csrc", name)) as f:
        return f.read()


def ffn_kernel(which, E, A_cap, N):
    """Which kernel a bf16 expert-FFN pass over one problem takes ("few": ffn_skinny.hip, "mid", "tile"): pass 0 (gate/up) or 1
    (down), E groups with A_cap rows allotted, N output columns.  The limits are read from the sources, so that a test whose
    sizes a changed limit moves to another kernel fails instead of testing that one twice."""
    src = _csrc("ffn_skinny.hip")
    lim = {k: int(re.search(r"\bSKINNY_%s = (\d+)" % k, src).group(1))
           for k in ("UP_ROWS", "UP_PER_GROUP", "UP_SINGLE", "DOWN_ROWS", "DOWN_SINGLE")}
    tiles = min(E, A_cap) * -(-N // 64)
    if E == 1:
        few = A_cap <= lim["DOWN_SINGLE" if which else "UP_SINGLE"]
    elif which == 0:
        few = A_cap <= min(lim["UP_ROWS"], lim["UP_PER_GROUP"] * E)
    else:
        few = A_cap <= lim["DOWN_ROWS"] and (A_cap <= E or tiles < 1024) and (A_cap <= 16 * E or tiles <= 128)
    if few:
        return "few"
    most = _mid_limits("SINGLE" if E == 1 else "RAGGED")[which]
    return "mid" if (A_cap if E == 1 else A_cap // E) <= most[-1] else "tile"


def ffn_tiles(E, rows, F):
    """Likely gate/up tiles of a problem, by which the launcher decides whether both passes are one launch (ffn_bf16_dma.hip)."""
    return (-(-rows // 256) if E == 1 else rows // 256 + min(E, rows) // 2) * -(-F // 128)


def ffn_both_limit(name):
    """A limit of the rules by which one launch takes both passes (BOTH_*, ffn_bf16_dma.hip)."""
    return int(re.search(r"\bBOTH_%s = (\d+)" % name, _csrc("ffn_bf16_dma.hip")).group(1))


def select_limit(name):
    """A number of tokens up to which the router's waves of large batches select as well (SELECT_*, route.hip)."""
    return int(re.search(r"\bSELECT_%s = (\d+)" % name, _csrc("route.hip")).group(1))


def ffn_tiles_limit():
    return ffn_both_limit("TILES")


def ffn_shared_schedule(T, E, K, d, F, Fs):
    """The FFN of a layer call whose gate/up pass and shared expert the tile kernel takes: "two" launches, or one with the shared expert's
    down tiles "late" or "early" (both_in_tiles, both_fills and ffn_down_early, ffn_bf16_dma.hip)."""
    up = lambda a, b: -(-a // b)
    mtiles, cols = T * K // 256 + min(E, T * K) // 2, up(d, 256)
    rows = 256 if Fs < 2 * F else {0: 64, 1: 128, 2: 256}[(up(T, 256) * cols > 40) + (up(T, 256) * cols >= 64)]
    routed, shared = mtiles * cols, up(T, rows) * cols
    gate_up = mtiles * up(F, 128) + up(T, 256) * up(Fs, 128)
    slices = gate_up * up(d, 64) + routed * up(F, 64) + shared * up(Fs, 64)
    fills = routed + shared >= ffn_both_limit("DOWN_TILES") and 10 * slices >= 7 * 256 * up(max(F, Fs), 64)
    mid = T <= _mid_limits("SINGLE")[1][1] and T * K // E <= _mid_limits("RAGGED")[1][2]
    if gate_up < ffn_tiles_limit() or mid and (T <= ffn_both_limit("BESIDE") or not fills):
        return "two"
    limit = "EARLY_LONGEST_UP_TO" if Fs > 4 * F else "EARLY_LONG_UP_TO" if Fs >= 3 * F else "EARLY_UP_TO"
    return "early" if T <= ffn_both_limit(limit) else "late"


def _mid_limits(side):
    """Most rows of every tile height of ffn_mid.hip, per pass (side: RAGGED, per group, or SINGLE)."""
    table = re.search(r"\bMID_%s_UP_TO\[2\]\[\d\] = \{([{}\d, ]+)\}" % side, _csrc("ffn_mid.hip")).group(1)
    return [[int(v) for v in re.findall(r"\d+", t)] for t in re.findall(r"\{([\d, ]+)\}", table + "}")]


def ffn_two_problems(which, E, A_cap, T):
    """The same for a pass over E routed groups and a shared expert's T rows: the kernel, or, for ffn_mid.hip, the rows of the routed
    and of the shared tiles."""
    src, mid = _csrc("ffn_skinny.hip"), _csrc("ffn_mid.hip")
    lim = {k: int(re.search(r"\bSKINNY_%s = (\d+)" % k, src).group(1))
           for k in ("UP_ROWS", "UP_PER_GROUP", "UP_SINGLE", "DOWN_BESIDE", "DOWN_SINGLE")}
    if which == 0 and T <= lim["UP_SINGLE"] and A_cap <= min(lim["UP_ROWS"], lim["UP_PER_GROUP"] * E):
        return "few"
    if which == 1 and T <= lim["DOWN_SINGLE"] and A_cap <= lim["DOWN_BESIDE"]:
        return "few"
    ragged, single, mean = _mid_limits("RAGGED")[which], _mid_limits("SINGLE")[which], A_cap // E
    if mean > ragged[2] or T > single[1]:
        return "tile"
    low = int(re.search(r"\bMID_LOW_BESIDE = (\d+)", mid).group(1))
    return 32 if mean <= low else 64 if mean <= ragged[1] else 128, 32 if T <= single[0] else 64
