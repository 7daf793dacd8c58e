"""The register-resident sweeps (binary32 L = 18 .. 32, binary64 L = 18) and the streaming
ones, between which the default path chooses by the size of the ensemble and the length of
the call, leave the same energies bit for bit: an ensemble swept in shards, or in several
calls, takes the exchange decisions of the whole."""
import pytest
import torch

import paper_1006_4247_amd as hsg

pytestmark = pytest.mark.gpu
SIZES = [("fp32", 18), ("fp32", 20), ("fp32", 22), ("fp32", 24), ("fp32", 26), ("fp64", 18)]
WHOLE = [("fp32", 28), ("fp32", 30), ("fp32", 32)]
SEED = 0x100642470E17


def _ensemble(prec, L, S, C, R):
    e = hsg.Ensemble(L, S, C, hsg.geometric_betas(1.0, 8.0, R), SEED + L, precision=prec)
    e.init_couplings()
    e.init_spins()
    return e


def _same(a, b):
    torch.cuda.synchronize()
    assert torch.equal(a.spins, b.spins)
    assert torch.equal(a.energy, b.energy)
    a.check()
    b.check()


# the energy taken in an overrelaxation, a renormalising and a heat-bath half-sweep
@pytest.mark.parametrize("prec,L", SIZES)
@pytest.mark.parametrize("S,n,n_hb,n_or", [(2, 2, 1, 10), (2, 2, 0, 8), (10, 4, 1, 0)])
def test_energy_bits(prec, L, S, n, n_hb, n_or):
    a, b = _ensemble(prec, L, S, 4, 6), _ensemble(prec, L, S, 4, 6)
    a.sweep(n, n_hb, n_or)
    b.sweep(n, n_hb, n_or, tuning={"path": 2})
    _same(a, b)


@pytest.mark.parametrize("prec,L", WHOLE)
@pytest.mark.parametrize("n,n_hb,n_or", [(2, 1, 10), (1, 2, 8)])
def test_energy_bits_whole_columns(prec, L, n, n_hb, n_or):
    a, b = _ensemble(prec, L, 4, 3, 8), _ensemble(prec, L, 4, 3, 8)
    a.sweep(n, n_hb, n_or)
    b.sweep(n, n_hb, n_or, tuning={"path": 2})
    _same(a, b)


@pytest.mark.parametrize("prec,L", SIZES + WHOLE)
def test_energy_of_shard_and_of_shorter_calls(prec, L):
    whole = _ensemble(prec, L, 8, 2, 8)  # 128 slots
    shard = _ensemble(prec, L, 1, 2, 8)  # its first sample
    steps = _ensemble(prec, L, 8, 2, 8)
    for _ in range(2):
        whole.sweep(4, 1, 3)
        shard.sweep(4, 1, 3)
        for _ in range(4):
            steps.sweep_measure(1, 1, 3)
    _same(whole, steps)
    assert torch.equal(whole.energy[:1], shard.energy)
    assert torch.equal(whole.spins[:1], shard.spins)
