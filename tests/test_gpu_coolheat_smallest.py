"""Cooling / heating at L = 2, the smallest lattice, whose legs are the generic ones in every
pair order (several even or odd pairs per chain among them); same oracle comparisons and
tolerances as at the other sizes."""
import pytest

from tests import test_gpu_coolheat as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairing", [0, 1, 2])
def test_smallest_lattice_fp64(pairing):
    base.test_coolheat_parity_fp64(2, pairing)


@pytest.mark.parametrize("pairing", [1, 2])
def test_smallest_lattice_fp32(pairing):
    base.test_coolheat_parity_fp32(2, pairing)
