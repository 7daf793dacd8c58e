"""The measurement that finishes a streaming sweep's energies (hsg_sweep_measure where the
sweep streams and the pairs of replicas are read whole, L = 18 .. 32, or a single chain)
against the sweep's own finishing pass and a measurement behind it: sizes and calls that
stream by default."""
import pytest

from tests import test_gpu_sweep_measure as fused

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L,C,n_sweeps", [("fp64", 20, 1, 1), ("fp64", 20, 2, 2), ("fp64", 20, 3, 1),
                                               ("fp32", 24, 2, 1), ("fp32", 28, 3, 1), ("fp32", 34, 1, 2)])
def test_measure_finishes_streaming_sweeps(prec, L, C, n_sweeps):
    fused.test_sweep_measure_equals_sweep_then_measure(prec, L, C, n_sweeps)
