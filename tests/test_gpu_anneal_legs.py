"""Annealing legs beyond L = 16 against the oracle (rules: gpu_pair.anneal_and_check), in the
register-resident kernel, which takes binary32 L = 18 .. 22 and, with enough overrelaxation
lattice sweeps, binary32 L = 24 and binary64 L = 18, and in the streaming kernels, which take
the others: forward and adjoint order, with and without heat-bath (binary32 legs without one
renormalise), pairs with K = 0 among them."""
import numpy as np
import pytest

from gpu_pair import anneal_and_check, make_pair
from oracle import hsgref

pytestmark = pytest.mark.gpu
SEED = 0x100642470A17


def _legs(prec, L, S, K, n_hb, n_or):
    betas = hsgref.geometric_betas(1.0, 1.5, 5)
    K = np.array(K, dtype=np.int32)
    for parity in (0, 1):
        gpu, ref = make_pair(L, S, 2, betas, SEED + L + parity, prec=prec, K_max=2)
        n_dec, n_cmp, _ = anneal_and_check(gpu, ref, parity, K, None, n_hb, n_or,
                                           what="legs L=%d %s %d+%d parity %d" % (L, prec, n_hb, n_or, parity))
        assert n_cmp >= n_dec // 2
        gpu.check()


@pytest.mark.parametrize("prec,L,n_hb,n_or", [
    ("fp32", 18, 0, 1), ("fp32", 18, 0, 2), ("fp32", 18, 1, 3),  # 0 + 1: renormalisation and energy in one lattice sweep
    ("fp32", 20, 0, 2), ("fp32", 20, 1, 3),
    ("fp32", 22, 0, 1), ("fp32", 22, 0, 2), ("fp32", 22, 1, 3),
    ("fp32", 24, 0, 2), ("fp32", 24, 1, 3),
    ("fp64", 18, 0, 2), ("fp64", 18, 1, 3), ("fp64", 18, 2, 6),
])
def test_column_legs(prec, L, n_hb, n_or):
    _legs(prec, L, 1, [1, 0, 1, 1], n_hb, n_or)


@pytest.mark.parametrize("prec,L,n_hb,n_or", [
    ("fp32", 24, 1, 0), ("fp32", 24, 1, 2),  # (the compositions next to those above)
    ("fp64", 18, 1, 2), ("fp64", 18, 0, 1),
    ("fp32", 26, 1, 0), ("fp32", 26, 1, 3), ("fp32", 28, 1, 0), ("fp32", 28, 1, 3),
    ("fp32", 34, 1, 0), ("fp32", 34, 1, 3),  # a size without an instance of its own
])
def test_streaming_legs(prec, L, n_hb, n_or):
    _legs(prec, L, 1, [1, 0, 2, 1] if n_or == 0 else [1, 0, 1, 1], n_hb, n_or)
