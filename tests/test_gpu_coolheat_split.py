"""The ascending cooling / heating pass at L > 16, whose heating legs run first and whose
accepted configurations stay in their candidate buffers until the pass ends, against the
oracle in binary64 (the tolerances of the other binary64 exchange tests): a single pair,
runs of accepted and of rejected pairs, slices with a remainder, few sites and several
rounds of sites per workgroup, and several calls on the state a call left."""
import numpy as np
import pytest
import torch

from gpu_pair import compare_ints, make_pair
from oracle import hsgref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,S,C,R,eps", [
    (18, 1, 1, 2, 0.01),    # one pair; 11 slices of 265 or 266 sites
    (18, 1, 2, 14, 0.004),  # long runs of accepted pairs
    (18, 30, 2, 3, 0.01),   # 60 chains, 9 slices of 324
    (20, 3, 1, 9, 0.01),
    (34, 1, 1, 4, 0.004),   # 64 slices of 307, a remainder of 51 to a thread's second site
])
def test_split_pass_against_oracle(L, S, C, R, eps):
    gpu, ref = make_pair(L, S, C, hsgref.geometric_betas(0.5, 0.5 * 1.12 ** (R - 1), R), 0x5C01 + L + R, prec="fp64")
    for call in range(3):
        w = gpu.coolheat_swap(eps, 0)
        _, ld = ref.coolheat_swap(eps, 0)
        torch.cuda.synchronize()
        what = "L=%d S=%d C=%d R=%d call %d" % (L, S, C, R, call)
        assert np.max(np.abs(w.cpu().numpy() - ld)) <= 1e-9 * max(1.0, np.abs(ld).max()), what
        st = compare_ints(gpu, ref, what)
        assert np.max(np.abs(st["spins"] - ref.spins)) <= 1e-12, what
        assert np.max(np.abs(st["energy"] - ref.energy)) <= 1e-9, what
    if S * C * (R - 1) >= 8:
        assert 0 < ref.stats[..., 1].sum() < ref.stats[..., 0].sum()
    gpu.check()
