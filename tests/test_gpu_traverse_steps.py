"""Traversal steps: the whole-number acceptance criterion on both sides of its range, and stacks
longer than their LDS part, as identical lists with the oracle's."""
import numpy as np
import pytest

import oracle
from helpers import rel_err, same_lists
from paper_2006_14952_amd import inputs


def _check(pos, m, **kw):
    import torch

    import paper_2006_14952_amd as hf
    prm = hf.params(p=2, **kw)
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), prm)
    got = t.short_range(prm).cpu().numpy()
    ref = oracle.fmm(pos, m, oracle.make_params(box=prm.box, rs=prm.r_s, rcut=prm.r_cut, theta=prm.theta, p=2,
                                                ncrit=prm.n_crit, mac_mode=prm.mac_mode))
    st = t.stats()
    assert st["n_m2l"] == ref.stats["n_m2l"] and st["n_p2p"] == ref.stats["n_p2p"]
    assert same_lists(t.interactions("p2p"), ref.lists("p2p")) and same_lists(t.interactions("m2l"), ref.lists("m2l"))
    assert rel_err(got, ref.acc).max() < 1e-9
    return st


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("box,cut,theta", [(1.0, 0.09, 0.5), (3.7, 0.31, 0.37), (1.0, 0.4999, 1.0), (0.01, 0.125, 0.25),
                                           (1.0, 0.0625, 0.6180339887)])
def test_lists_across_cutoffs_boxes_and_angles(box, cut, theta, mode):
    pos, m = inputs.clustered(4000, 3, inputs.rng_for(631))
    _check(pos * box, m, box=box, r_s=box * cut / 4.0, r_cut=box * cut, theta=theta, n_crit=12, mac_mode=mode)


@pytest.mark.gpu
@pytest.mark.parametrize("level", [9, 10, 11, 12])
def test_deepest_cells_around_the_whole_number_range(level):
    """r_cut = 0.49: r_cut / u = 0.98 2^level, past 4096 from level 13 of the cells on (pairs that part at
    `level` make cells there and one level below)."""
    rng = inputs.rng_for(632, level)
    c = (np.floor(rng.random((30, 3)) * 2 ** (level + 1)) + 0.5) / 2 ** (level + 1)
    pos = np.concatenate([rng.random((1500, 3)), c, c + 0.3 / 2 ** (level + 1), np.mod(c + 1.0 / 2 ** (level + 1), 1.0)])
    m = np.full(len(pos), 1.0 / len(pos))
    _check(pos, m, r_s=0.12, r_cut=0.49, theta=0.5, n_crit=1)


@pytest.mark.gpu
def test_stacks_longer_than_their_lds_part():
    """Leaves of one or two particles and a cutoff of 0.45: sinks inherit thousands of pairs."""
    pos, m = inputs.clustered(6000, 3, inputs.rng_for(633))
    st = _check(pos, m, r_s=0.11, r_cut=0.45, theta=0.3, n_crit=2)
    assert st["n_p2p"] / st["n_leaves"] > 1024
