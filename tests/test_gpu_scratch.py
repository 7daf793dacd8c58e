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
