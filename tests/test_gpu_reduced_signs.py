"""The bare reduced solver hands out the eigenvectors it always has, signs
included, at the edges of its reductions' forms (the golden file's writer says
what the values are)."""
import importlib.util
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
_spec = importlib.util.spec_from_file_location("make_reduced_vectors", os.path.join(GOLDEN, "make_reduced_vectors.py"))
maker = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(maker)


@pytest.mark.parametrize("n", maker.SIZES)
def test_first_entries(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    i = maker.SIZES.index(n)
    re, im = np.loadtxt(maker.OUT)[:, 2 * i:2 * i + 2].T
    # the same arithmetic: no tolerance
    np.testing.assert_array_equal(maker.first_entries(n), re + 1j * im)
