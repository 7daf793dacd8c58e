"""Even and odd cooling / heating pairs at L <= 16, both legs of a pair in one workgroup, at
the sizes the other tests leave out: sites that do not fill the workgroup (L = 6, 10, 14),
one, two and four of a thread; same oracle comparisons and tolerances."""
import pytest

from tests import test_gpu_coolheat as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [6, 10, 12, 14])
@pytest.mark.parametrize("pairing", [1, 2])
def test_pairs_fp32(L, pairing):
    base.test_coolheat_parity_fp32(L, pairing)


@pytest.mark.parametrize("L", [8, 10, 14])
@pytest.mark.parametrize("pairing", [1, 2])
def test_pairs_fp64(L, pairing):
    base.test_coolheat_parity_fp64(L, pairing)
