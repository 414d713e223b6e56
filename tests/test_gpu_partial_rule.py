"""Partial contraction on both sides of the rule that groups its tensor pairs by the transforms and spectra it saves:
two pairs of two assignments each (singly), three pairs (grouped), one pair with all of the free modes."""
import pytest

from test_gpu_partial_groups import test_entries as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p, free, m, dtype", [
    (3, {0: [2], 2: [2]}, 1024, "float32"), (3, {0: [2], 2: [3]}, 256, "float64"), (3, {0: [5]}, 64, "float32"),
    (6, {0: [2], 3: [2]}, 256, "float32"), (6, {0: [4]}, 512, "bfloat16")])
def test_rule(p, free, m, dtype):
    check(p, free, m, dtype)
