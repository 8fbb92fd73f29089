"""FP64 P2P: the fitted force laws, the box tests and the sink tiles against extended precision."""
import numpy as np
import pytest

from paper_2006_14952_amd import inputs

LD = np.longdouble


def _direct(pos, mass, r_s, r_cut, split):
    """Hard-cut minimum-image sum in extended precision, and a bound on FP64 rounding:
    every pair's weight good to 8 roundings of its Newtonian size, its separation to the
    rounding of coordinates of size 1 (wrapped images are not exact), the sum to its terms."""
    x, m = pos.astype(LD), mass.astype(LD)
    acc, bound = np.zeros_like(x), np.zeros(len(x))
    eps = np.finfo(np.float64).eps
    for i in range(len(x)):
        d = x[i] - x
        d -= np.round(d)
        r2 = (d * d).sum(1)
        k = (r2 > 0) & (r2 < LD(r_cut) ** 2)
        d, r2, mm = d[k], r2[k], m[k]
        r = np.sqrt(r2)
        if split:
            q = r / LD(r_cut)
            h = (1 - q) ** 2 * (1 + 2 * q + 3 * q * q + LD(1.5) * q ** 3)
        else:  # 1 - S u^3 with the series of S (its terms stay below e^v)
            u = r / (2 * LD(r_s))
            v, s, t = u * u, np.zeros_like(u), np.ones_like(u)
            for n in range(120):
                s += t / (2 * n + 3)
                t *= -v / (n + 1)
            h = 1 - 4 / np.sqrt(LD("3.14159265358979323846")) * s * u ** 3
        acc[i] = ((-mm * h / (r2 * r))[:, None] * d).sum(0)
        bound[i] = float((mm / r2 * (8 + 4 / r)).sum()) * eps * (1 + np.sqrt(max(k.sum(), 1)))
    return acc, bound


@pytest.mark.gpu
@pytest.mark.parametrize("ratio,split", [(1.0, 0), (4.5, 0), (4.52, 0), (5.0, 0), (5.001, 0), (6.5, 0), (4.5, 1)])
@pytest.mark.parametrize("n,n_crit,tile", [(1, 32, 0), (33, 64, 32), (700, 17, 16), (900, 65, 0), (640, 1000, 64)])
def test_direct_pairs(ratio, split, n, n_crit, tile):
    import torch

    import paper_2006_14952_amd as hf
    pos, mass = inputs.clustered(n, 3, inputs.rng_for(611, n))
    r_cut = 0.31
    prm = hf.params(r_s=r_cut / ratio, r_cut=r_cut, theta=1e-3, p=2, n_crit=n_crit, split=split, p2p_chunk=tile)
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"), prm)
    got = t.short_range(prm).cpu().numpy()
    st = t.stats()
    assert st["n_m2l"] == 0 and st["p2p_evaluated"] <= st["p2p_pairs"]
    ref, bound = _direct(pos, mass, r_cut / ratio, r_cut, split)
    err = np.sqrt(((got - ref) ** 2).sum(1)).astype(float)
    assert np.all(err <= bound), (err / np.maximum(bound, 1e-300)).max()


@pytest.mark.gpu
@pytest.mark.parametrize("r_cut", [1e-6, 1e-4, 2e-3])
def test_box_tests_keep_pairs_at_the_cutoff_of_a_wide_leaf(r_cut):
    """A leaf far wider than the cutoff, pairs just inside it: none is lost to the FP32 boxes."""
    import torch

    import paper_2006_14952_amd as hf
    rng = inputs.rng_for(612)
    a = rng.random((300, 3))
    u = rng.standard_normal((300, 3))
    b = a + (r_cut * (1 - 1e-9)) * u / np.linalg.norm(u, axis=1, keepdims=True)
    pos = np.mod(np.concatenate([a, b]), 1.0)
    mass = rng.random(600) + 0.5
    prm = hf.params(r_s=r_cut / 2, r_cut=r_cut, theta=1e-3, p=2, n_crit=80)
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"), prm)
    got = t.short_range(prm).cpu().numpy()
    ref, bound = _direct(pos, mass, r_cut / 2, r_cut, 0)
    assert np.count_nonzero((ref != 0).any(1)) >= 590
    err = np.sqrt(((got - ref) ** 2).sum(1)).astype(float)
    assert np.all(err <= bound), (err / np.maximum(bound, 1e-300)).max()
