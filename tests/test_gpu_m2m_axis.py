"""Upward pass of orders 7 and 8: levels on both sides of the two M2M forms' dividing line, against the oracle."""
import pytest

import oracle
from helpers import rel_err
from paper_2006_14952_amd import inputs


@pytest.mark.gpu
@pytest.mark.parametrize("p", [7, 8])
@pytest.mark.parametrize("n,n_crit", [(9, 8), (600, 5), (12000, 8), (30000, 3)])
def test_orders_7_and_8(n, n_crit, p):
    """One parent; a few a level, with 1 to 8 children; some 1,500 parents on one level; 4,096."""
    import torch

    import paper_2006_14952_amd as hf
    pos, m = inputs.uniform(n, inputs.rng_for(661, n))
    prm = hf.params(r_s=0.05, r_cut=0.2, theta=0.5, p=p, n_crit=n_crit)
    d = [torch.tensor(a, device="cuda") for a in (pos, m)]
    got = hf.Tree().build(*d, prm).short_range(prm).cpu().numpy()
    ref = oracle.fmm(pos, m, oracle.make_params(rs=0.05, rcut=0.2, theta=0.5, p=p, ncrit=n_crit)).acc
    assert rel_err(got, ref).max() < 1e-9
    # FP32: the level-by-level sums are those of the FP64 form; its own bar as for the other orders
    p32 = hf.copy_params(prm, precision=1)
    g32 = hf.Tree().build(*d, p32).short_range(p32).cpu().numpy()
    assert rel_err(g32, got).mean() < 1e-4
