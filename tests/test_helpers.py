"""The comparison that the GPU parity tests rest on."""
import numpy as np
import pytest

from helpers import logits_error


def test_logits_error_does_not_pass_over_a_nan():
    want = np.ones((1, 2, 3, 4), np.float32)
    got = want.copy()
    assert logits_error(got, want, [2]) == (0.0, 0.0)
    got[0, 1, 2, 0] = np.nan          # an idle row
    assert logits_error(got, want, [2]) == (0.0, 0.0)
    got[0, 1, 1, 3] = np.nan
    with pytest.raises(AssertionError):
        logits_error(got, want, [2])
