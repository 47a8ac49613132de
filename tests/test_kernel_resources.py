"""Registers of kernels whose speed hangs on the wavefronts a unit holds."""
import re

from kernel_resources import kernels
from paper_2505_19342_amd import binding as B


def registers(pattern):
    found = {n: k[".vgpr_count"] for n, k in kernels(B.LIB_PATH).items() if re.search(pattern, n)}     # of either kind
    assert found, pattern
    return found


def test_fp32_attention_leaves_room_for_three_wavefronts():
    """512 registers per lane and SIMD, in steps of 8.  12 heads of 256 over 100 causal rows: 31.6 us with one wavefront, 12.5 with three."""
    for name, n in registers("attn_f32_kernel").items():
        assert n <= 168, (name, n)
