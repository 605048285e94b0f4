"""GPU tests of the short convolution's two block lengths against the oracle (MI355X only).

Launches of fewer than 1,024 workgroups of 8 tokens take blocks of 4 tokens (widths up
to 5); both sides of the limit, partial blocks, tails shorter than the carried rows.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2609_18935_amd as tu
from gpu_cases import DEV, bits_of, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tu.lib()


@pytest.mark.parametrize("W,C,T", [(5, 16, 3), (5, 16, 4), (4, 2056, 5), (5, 8192, 2045), (5, 8192, 2053), (6, 64, 9),
                                   (3, 8192, 2049)])
def test_block_lengths(W, C, T):
    print(f"[case] short conv W={W} C={C} T={T}", flush=True)
    st, x, w = synth.gen_conv_inputs(17, T, C, W)
    ref_y, _, ref_s = oracle.short_conv_continue(st, x, w)
    s, out = to_dev_bf16(st), torch.full((T, C), float("nan"), dtype=torch.bfloat16, device=DEV)
    tu.short_conv_continue(s, to_dev_bf16(x), to_dev_bf16(w), out)
    torch.cuda.synchronize()
    # one bf16 ulp (at most 2^-7 of the value) plus the fp32 sum's own error: W products and
    # sums, each within 2^-24 of the sum of magnitudes (SiLU's slope stays below 1.1); among
    # millions of outputs some cancel to values whose bf16 ulp is below that
    _, y_abs, _ = oracle.short_conv_continue(st & 0x7FFF, x & 0x7FFF, w & 0x7FFF, activation="none")
    got, ref = synth.bf16_bits_to_f32(bits_of(out)).astype(np.float64), synth.bf16_bits_to_f32(ref_y).astype(np.float64)
    assert np.all(np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 1.1 * W * 2.0 ** -23 * y_abs)
    assert np.count_nonzero(bits_of(out) != ref_y) <= 1e-3 * ref_y.size
    assert np.array_equal(bits_of(s), ref_s)
