"""The register-resident sweeps (binary32 L = 18 .. 32, binary64 L = 16 and 18; the default
path where they are the faster kernel) against the streaming / LDS-resident kernels on the
same state: spins and counters bit for bit, energies within the rounding of a binary64 sum
taken in another order (N terms of size ~1: a few N 2^-53); and their annealing legs
against the oracle."""
import numpy as np
import pytest
import torch

import paper_1006_4247_amd as hsg
from gpu_pair import anneal_and_check, make_pair
from oracle import hsgref

pytestmark = pytest.mark.gpu
SIZES = [("fp32", 18), ("fp32", 20), ("fp32", 22), ("fp32", 24), ("fp32", 26), ("fp64", 16), ("fp64", 18)]
SEED = 0x100642470C20


def _ensemble(prec, L):
    e = hsg.Ensemble(L, 2, 3, hsg.geometric_betas(1.0, 8.0, 6), SEED + L, precision=prec)  # 36 slots
    e.init_couplings()
    e.init_spins()
    return e


@pytest.mark.parametrize("prec,L", SIZES)
# forward order with and without each kind; the energy in an overrelaxation and in a
# heat-bath half-sweep; renormalising sweeps; several sweeps, one energy
@pytest.mark.parametrize("n,n_hb,n_or", [(1, 1, 3), (2, 2, 5), (2, 0, 4), (4, 1, 0), (5, 0, 1)])
def test_column_equals_other_kernels(prec, L, n, n_hb, n_or):
    a, b = _ensemble(prec, L), _ensemble(prec, L)
    for _ in range(2):
        a.sweep(n, n_hb, n_or)
        b.sweep(n, n_hb, n_or, tuning={"path": 3 if L <= 16 else 2})
    torch.cuda.synchronize()
    assert torch.equal(a.spins, b.spins)
    assert torch.equal(a.sweep_ctr, b.sweep_ctr)
    assert float((a.energy - b.energy).abs().max()) <= 8 * L ** 3 * 2.0 ** -53
    a.check()


@pytest.mark.parametrize("prec,L", [s for s in SIZES if s[1] > 16])
def test_column_annealing_legs(prec, L):
    """Pairs with K = 0, 1 and 2 mixed, both parities, heat-bath legs (which do not amplify
    rounding)."""
    betas = hsgref.geometric_betas(1.0, 1.5, 5)
    K = np.array([1, 0, 2, 1], dtype=np.int32)
    for parity in (0, 1):
        gpu, ref = make_pair(L, 1, 2, betas, SEED + 9 + parity, prec=prec, K_max=2)
        n_dec, n_cmp, _ = anneal_and_check(gpu, ref, parity, K, None, 1, 0, what="legs L=%d %s" % (L, prec))
        assert n_cmp >= n_dec // 2
        gpu.check()


@pytest.mark.parametrize("L", [28, 30, 32])
# one energy after several sweeps, several heat-baths, and the fewest sweeps that take the
# path with 96 slots; 48 slots take it for longer calls
@pytest.mark.parametrize("S,n,n_hb,n_or", [(4, 1, 1, 3), (4, 2, 2, 1), (2, 1, 1, 19)])
def test_whole_columns_equal_other_kernels(L, S, n, n_hb, n_or):
    es = []
    for tuning in (None, {"path": 2}):
        e = hsg.Ensemble(L, S, 3, hsg.geometric_betas(1.0, 8.0, 8), SEED + L, precision="fp32")
        e.init_couplings()
        e.init_spins()
        for _ in range(2):
            e.sweep(n, n_hb, n_or, tuning=tuning)
        e.check()
        es.append(e)
    a, b = es
    assert torch.equal(a.spins, b.spins)
    assert torch.equal(a.sweep_ctr, b.sweep_ctr)
    # the same terms in two orders: no term passes through more than L + 6 + 8 additions here
    # and 16 + 6 + 4 + L^3 / 256 there, each of which rounds a partial sum of at most the sum
    # of |J| (a bond's |s . s'| is at most 1)
    adds = (L + 14) + (26 + L ** 3 / 256)
    bound = adds * 2.0 ** -53 * a.couplings.double().abs().sum(dim=tuple(range(1, a.couplings.dim())))
    assert bool(((a.energy - b.energy).abs().amax(dim=(1, 2)) <= bound).all())
