"""Calls that do without an ensemble's scratch leave it as it is, whatever it holds."""
import numpy as np
import pytest
import torch

import paper_1006_4247_amd as hsg
from gpu_pair import compare_ints, make_pair
from oracle import hsgref

pytestmark = pytest.mark.gpu
SEED = 0x100642475C


def _mark(e):
    e.scratch.copy_(torch.arange(e.scratch.numel(), device=e.device) % 251)
    return e.scratch.clone()


@pytest.mark.parametrize("prec,L,C", [("fp32", 34, 2), ("fp64", 34, 3), ("fp32", 20, 2)])
def test_measure_leaves_the_scratch(prec, L, C):
    e = hsg.Ensemble(L, 2, C, hsg.geometric_betas(1.0, 4.0, 3), SEED + L, precision=prec)
    e.init_couplings()
    e.init_spins()
    before = _mark(e)
    Q, chi, _ = [t.clone() for t in e.measure()]
    torch.cuda.synchronize()
    assert torch.equal(e.scratch, before)
    e.desc.scratch = None
    Q0, chi0, _ = e.measure()
    torch.cuda.synchronize()
    assert torch.equal(Q, Q0) and torch.equal(chi, chi0)


@pytest.mark.parametrize("L,S", [(18, 2), (20, 40)])  # one launch per pair; two
def test_decimate_leaves_a_misaligned_scratch(L, S):
    """All pairs with a scratch 16 bytes past its alignment: the pass without one, in binary64
    against the oracle at the tolerances of the other exchange tests."""
    gpu, ref = make_pair(L, S, 1, hsgref.geometric_betas(1.0, 1.1, 4), SEED + L, prec="fp64")
    before = _mark(gpu)
    gpu.desc.scratch = gpu.scratch.data_ptr() + 16
    w = gpu.decimate_swap(0)
    lnA, role = ref.decimate_swap(0)
    torch.cuda.synchronize()
    assert torch.equal(gpu.scratch, before)
    assert np.max(np.abs(w.cpu().numpy()[..., 0] - lnA)) <= 1e-10 * max(1.0, np.abs(lnA).max())
    st = compare_ints(gpu, ref, "misaligned scratch L=%d" % L)
    assert np.max(np.abs(st["spins"] - ref.spins)) <= 1e-12
    assert np.max(np.abs(st["energy"] - ref.energy)) <= 1e-9
    gpu.check()
