"""Measurement beyond L = 32, where a pair of replicas is read in slices: against the oracle,
and fused with the sweep (two and three chains) against sweep and measurement apart."""
import pytest

from tests import test_gpu_parity as parity
from tests import test_gpu_sweep_measure as fused

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L", [("fp32", 34), ("fp64", 34), ("fp32", 40)])
def test_sliced_measure_against_oracle(prec, L):
    parity.test_measure_parity(prec, L)


@pytest.mark.parametrize("prec,L,C", [("fp32", 34, 2), ("fp64", 36, 3)])
def test_sliced_measure_after_sweeps(prec, L, C):
    fused.test_sweep_measure_equals_sweep_then_measure(prec, L, C, 2)
