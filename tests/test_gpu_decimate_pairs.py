"""The ascending decimated pass at L > 16 with few chains, which draws both configurations
before a pair is decided and copies at its end, against the oracle in binary64 (the
tolerances of the other binary64 exchange tests): a single pair, runs of accepted and of
rejected pairs, slices with a remainder and with a second round of sites, and the numbers
of chains on both sides of the rule that takes it."""
import numpy as np
import pytest
import torch

from gpu_pair import compare_ints, make_pair
from oracle import hsgref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,S,C,R", [
    (18, 1, 1, 2),   # one pair; 11 slices of 265 or 266 sites
    (18, 1, 2, 14),
    (18, 22, 1, 3),  # the most chains that take it ...
    (18, 23, 1, 3),  # ... and the fewest that do not
    (20, 3, 1, 9),
    (34, 1, 1, 4),   # 64 slices of 307
])
def test_pair_pass_against_oracle(L, S, C, R):
    gpu, ref = make_pair(L, S, C, hsgref.geometric_betas(1.0, 1.03 ** (R - 1), R), 0xDEC0 + L + R, prec="fp64")
    for call in range(3):
        w = gpu.decimate_swap(0)
        lnA, role = ref.decimate_swap(0)
        torch.cuda.synchronize()
        wg = w.cpu().numpy()
        what = "L=%d S=%d C=%d R=%d call %d" % (L, S, C, R, call)
        assert np.max(np.abs(wg[..., 0] - lnA)) <= 1e-10 * max(1.0, np.abs(lnA).max()), what
        assert np.array_equal(wg[..., 1].astype(int), role), what
        st = compare_ints(gpu, ref, what)
        assert np.max(np.abs(st["spins"] - ref.spins)) <= 1e-12, what
        assert np.max(np.abs(st["energy"] - ref.energy)) <= 1e-9, what
    if S * C * (R - 1) >= 8:
        assert 0 < ref.stats[..., 1].sum() < ref.stats[..., 0].sum()
    gpu.check()
