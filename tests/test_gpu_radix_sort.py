"""Particle order of the tree build at the edges of the sort's forms, rounds and tiles."""
import numpy as np
import pytest

from paper_2006_14952_amd import inputs

SIZES = [1, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 9215, (1 << 17), (1 << 17) + 1,
         (1 << 20), (1 << 20) + 1]


def _build(pos, m, nbox, off):
    import torch

    import paper_2006_14952_amd as hf
    prm = hf.params(r_s=0.02, p=2, n_crit=24)
    d = [torch.tensor(a, device="cuda") for a in (pos, m)]
    t = hf.Tree()
    return (t.build(*d, prm) if nbox == 1 else t.build_batched(*d, [prm] * nbox, off)), prm


@pytest.mark.gpu
@pytest.mark.parametrize("nbox", [1, 3, 300])
@pytest.mark.parametrize("n", SIZES)
def test_order_does_not_depend_on_the_callers(n, nbox):
    """The sort is correct if a shuffled copy gives the same tree; one that lost, doubled or
    misplaced a particle gives other counts.  Boxes of a batch keep their own particles."""
    rng = inputs.rng_for(671, n)
    pos, m = inputs.clustered(n, 1 + n // 5000, rng)
    off = np.linspace(0, n, nbox + 1).astype(np.int64)
    perm = np.concatenate([off[b] + rng.permutation(int(off[b + 1] - off[b])) for b in range(nbox)])
    a, prm = _build(pos, m, nbox, off)
    b, _ = _build(pos[perm], m[perm], nbox, off)
    fa, fb = a.short_range(prm).cpu().numpy(), b.short_range(prm).cpu().numpy()
    sa, sb = a.stats(), b.stats()
    assert all(sa[k] == sb[k] for k in ("n_cells", "n_leaves", "max_level", "n_p2p", "n_m2l"))
    scale = np.sqrt((fa ** 2).sum(1).mean()) if n > 1 else 1.0
    assert np.abs(fa[perm] - fb).max() <= 1e-9 * max(scale, np.abs(fa).max())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [700, 1500, 4000, 8000, 20000, 200000])
def test_deep_trees_are_sorted_again_over_every_digit(n):
    """Particles that share their first 15 levels: the lowest two digits decide."""
    import oracle

    from helpers import rel_err
    rng = inputs.rng_for(672, n)
    pos, m = inputs.uniform(n, rng)
    pos[:600] = 0.3 + 2e-6 * rng.random((600, 3))
    t, prm = _build(pos, m, 1, None)
    assert t.stats()["max_level"] > 15
    got = t.short_range(prm).cpu().numpy()
    if n <= 20000:
        rs, rc = prm.r_s, prm.r_cut
        ref = oracle.fmm(pos, m, oracle.make_params(rs=rs, rcut=rc, theta=0.5, p=2, ncrit=24))
        assert rel_err(got, ref.acc).max() < 1e-9
