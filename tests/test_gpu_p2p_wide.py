"""Sink leaves computed by a workgroup of several waves: FP32 bits as by one wave, FP64 as the oracle."""
import numpy as np
import pytest

import oracle
from helpers import rel_err
from paper_2006_14952_amd import inputs


def _cluster_beside_wide_leaves(n, seed, sigma):
    """A tight cluster and a few dozen particles around it, whose large leaves list the whole cluster."""
    rng = inputs.rng_for(641, seed)
    c = np.array([0.26, 0.27, 0.24])
    pos = np.concatenate([c + sigma * rng.standard_normal((n, 3)), rng.random((40, 3)) * 0.5])
    return np.mod(pos, 1.0), np.full(n + 40, 1.0 / n)


def _tree(pos, m, prm):
    import torch

    import paper_2006_14952_amd as hf
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), prm)
    acc = t.short_range(prm)
    st = t.stats()
    entries = np.unique(t.interactions("p2p")[:, 0], return_counts=True)[1].max()
    return acc, st, int(entries)


def _line(st):
    return max(st["n_p2p"] // 4096 // 4, 4 * (st["n_p2p"] // st["n_leaves"]), 256)


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_crit,tile,split", [(6000, 3, 0, 0), (20000, 12, 0, 0), (20000, 12, 0, 1), (30000, 40, 16, 0),
                                                 (30000, 90, 64, 0), (40000, 1, 0, 0)])
def test_fp32_bits_do_not_depend_on_the_waves_of_a_leaf(n, n_crit, tile, split):
    """Schedule 3 launches P2P level by level, one wave per leaf; fixed-order sums elsewhere."""
    import torch

    import paper_2006_14952_amd as hf
    pos, m = _cluster_beside_wide_leaves(n, n_crit, 0.01)
    kw = dict(r_s=0.06, r_cut=0.27, theta=0.9, p=3, n_crit=n_crit, precision=1, deterministic=1, p2p_chunk=tile, split=split)
    wide, st, entries = _tree(pos, m, hf.params(schedule=1, **kw))
    one, st3, _ = _tree(pos, m, hf.params(schedule=3, **kw))
    assert entries >= _line(st), (entries, _line(st))  # some leaf goes to a workgroup
    assert torch.equal(wide, one)
    assert st["p2p_pairs"] == st3["p2p_pairs"] and st["p2p_evaluated"] == st3["p2p_evaluated"]


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_crit,ratio", [(6000, 3, 4.5), (20000, 12, 5.0), (20000, 12, 7.0), (40000, 1, 4.5)])
def test_fp64_matches_the_oracle(n, n_crit, ratio):
    import paper_2006_14952_amd as hf
    pos, m = _cluster_beside_wide_leaves(n, n_crit, 0.01)
    prm = hf.params(r_s=0.27 / ratio, r_cut=0.27, theta=0.9, p=3, n_crit=n_crit)
    acc, st, entries = _tree(pos, m, prm)
    assert entries >= _line(st), (entries, _line(st))
    ref = oracle.fmm(pos, m, oracle.make_params(rs=prm.r_s, rcut=prm.r_cut, theta=0.9, p=3, ncrit=n_crit))
    assert st["p2p_pairs"] == ref.stats["p2p_pairs"]
    assert rel_err(acc.cpu().numpy(), ref.acc).max() < 1e-9
