"""Octree passes at the edges of their tiles and windows: counts, lists and forces against the oracle."""
import numpy as np
import pytest

import oracle
from helpers import rel_err, same_lists
from paper_2006_14952_amd import inputs

R_S, R_CUT = 0.05, 0.2


def _oracle(pos, m, n_crit):
    return oracle.fmm(pos, m, oracle.make_params(rs=R_S, rcut=R_CUT, theta=0.5, p=3, ncrit=n_crit))


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_crit", [(1, 1), (2, 1), (63, 3), (64, 64), (65, 64), (1024, 7), (1025, 16), (2047, 31),
                                      (3000, 511), (3000, 512), (3000, 513), (3000, 1023), (3000, 1024), (3000, 2999),
                                      (3000, 3000), (4097, 1)])
def test_one_box(n, n_crit):
    import torch

    import paper_2006_14952_amd as hf
    pos, m = inputs.clustered(n, 2, inputs.rng_for(621, n))
    prm = hf.params(r_s=R_S, r_cut=R_CUT, theta=0.5, p=3, n_crit=n_crit)
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), prm)
    got = t.short_range(prm).cpu().numpy()
    ref, st = _oracle(pos, m, n_crit), t.stats()
    assert (st["n_cells"], st["n_leaves"], st["max_level"]) == tuple(ref.stats[k] for k in ("ncell", "nleaf", "maxlevel"))
    assert same_lists(t.interactions("p2p"), ref.lists("p2p")) and same_lists(t.interactions("m2l"), ref.lists("m2l"))
    assert rel_err(got, ref.acc).max() < 1e-9


@pytest.mark.gpu
@pytest.mark.parametrize("n_crit", [5, 600])
@pytest.mark.parametrize("sizes", [(0, 7, 0, 0, 1500, 5, 6, 0), (1024, 0, 1024, 1), (3, 1, 2, 4, 5)])
def test_forest_with_empty_and_small_boxes(sizes, n_crit):
    import torch

    import paper_2006_14952_amd as hf
    boxes = [inputs.clustered(n, 2, inputs.rng_for(622, b)) if n else (np.zeros((0, 3)), np.zeros(0))
             for b, n in enumerate(sizes)]
    pos, m = (np.concatenate([b[k] for b in boxes]) for k in (0, 1))
    off = np.concatenate([[0], np.cumsum(sizes)])
    prm = hf.params(r_s=R_S, r_cut=R_CUT, theta=0.5, p=3, n_crit=n_crit)
    t = hf.Tree().build_batched(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), [prm] * len(sizes), off)
    got = t.short_range(prm).cpu().numpy()
    st = t.stats()
    refs = [_oracle(*b, n_crit) for b in boxes if len(b[1])]
    empty = sum(n == 0 for n in sizes)
    assert st["n_cells"] == sum(r.stats["ncell"] for r in refs) + empty
    assert st["n_leaves"] == sum(r.stats["nleaf"] for r in refs) + empty
    assert st["n_p2p"] == sum(r.stats["n_p2p"] for r in refs) and st["n_m2l"] == sum(r.stats["n_m2l"] for r in refs)
    ref = np.concatenate([r.acc for r in refs])
    assert rel_err(got, ref).max() < 1e-9
