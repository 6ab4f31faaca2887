"""GPU parity where the split of the work over workgroups can go wrong: remainders of the item lists.

Bars as in test_gpu_parity (bf16 inputs, fp32 accumulation, bf16 output).
"""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_parity import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("Hkv", [1, 2, 4, 8, 3])
@pytest.mark.parametrize("P,E", [([40], [257]), ([0, 100, 7], [513, 1, 300]), ([64, 64], [300, 300])])
def test_items_dealt_out_over_the_xcds(H, Hkv, P, E):
    """Numbers of items that no number of XCDs divides, with several XCDs to a KV head and with one."""
    w = W.make_uniform("items", 51, len(P), 3 * Hkv, Hkv, P, E)
    want = oracle.attention_of(w)
    for splits in (1, 3):
        _check(H.gpu_attention(w, num_splits=splits), want, f"Hkv={Hkv} P={P} E={E} splits={splits}")
