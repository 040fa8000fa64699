"""Router of large batches on the matrix pipe: the stream of sub-tiles that runs on across the 256-wide chunks, in both forms (chunk
results summed in registers, or stored one by one), logits bit-exact in the declared order."""
import numpy as np
import pytest

from paper_2504_01337_amd import workloads as wl
from helpers import dev, host

pytestmark = pytest.mark.gpu


# summed in registers (from 25057 tokens on, 32737 with up to 32 experts): whole chunks, a ragged last one, one expert block and two; stored: one
# chunk per workgroup and two (an even and an odd number of chunks, a ragged last one), the remainders of tokens and experts
@pytest.mark.parametrize("T,E,d,dtype", [
    (32768, 60, 512, "bf16"), (32705, 33, 520, "bf16"), (32769, 20, 768, "f32"), (40001, 64, 264, "f32"),
    (12353, 60, 776, "bf16"), (16400, 40, 1024, "bf16"), (16383, 61, 1100 // 8 * 8, "f32"), (16390, 18, 1288, "bf16"),
    (12289, 17, 256, "bf16"),
    # 64-token workgroups of half the experts per wave (the third and the fifth half round), and the first batches on either side of
    # the rules
    (33001, 60, 776, "bf16"), (49153, 36, 512, "bf16"), (65700, 34, 512, "bf16"), (36000, 61, 520, "f32"), (25089, 60, 520, "bf16"), (25000, 60, 520, "bf16")])
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
