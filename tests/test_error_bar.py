"""The bar of long rows sees a lost partial result and an output of zeros, which a fixed one does not."""
import dataclasses

import numpy as np
import pytest

import oracle
from error_bar import OF_RMS, worst_of_rms
from workloads import AttnShape, make_batch


@pytest.mark.parametrize("kv,fixed", [("bf16", 2e-2), ("fp8", 6e-2)])
def test_a_lost_partial_of_a_long_row_is_over_the_bar(kv, fixed):
    b = make_batch(AttnShape(8, 1, 128, "bf16", kv), [1], [3073], seed=91, value_mult=0.5)
    ref, _, _ = oracle.run_batch(b)
    lost = dataclasses.replace(b, ctx_lens=b.ctx_lens - 128, k_prefix=b.k_prefix[128:], v_prefix=b.v_prefix[128:])   # 8 pages of 193
    wrong, _, _ = oracle.run_batch(lost)
    assert worst_of_rms(wrong, ref) > 2 * OF_RMS and worst_of_rms(0 * ref, ref) > 10 * OF_RMS
    assert np.max(np.abs(wrong - ref)) < fixed
