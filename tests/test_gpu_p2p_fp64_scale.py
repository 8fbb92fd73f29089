"""FP64 forces in boxes of any size: lengths scaled by a power of two scale every force by an exact power of two."""
import numpy as np
import pytest

from paper_2006_14952_amd import inputs


def _forces(pos, mass, box, ratio, split):
    import torch

    import paper_2006_14952_amd as hf
    prm = hf.params(box=box, r_s=0.06 * box / ratio, r_cut=0.06 * box, theta=1e-9, p=2, n_crit=3, split=split,
                    deterministic=1)
    t = hf.Tree().build(torch.tensor(pos * box, device="cuda"), torch.tensor(mass, device="cuda"), prm)
    return t.short_range(prm).cpu().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("ratio,split", [(4.5, 0), (7.0, 0), (4.5, 1)])
@pytest.mark.parametrize("k", [-200, -110, -81, -72, -71, -70, -69, 60, 99, 101, 130, 200])
def test_any_box_gives_the_unit_boxes_forces(k, ratio, split):
    """r_cut = 0.06 box; at 2^-70 the box tests' squared gaps are a few of FP32's smallest steps."""
    pos, mass = inputs.uniform(20000, inputs.rng_for(613))
    one = _forces(pos, mass, 1.0, ratio, split)
    assert np.count_nonzero(one) > 50000
    got = np.ldexp(_forces(pos, mass, 2.0 ** k, ratio, split), 2 * k)
    if -80 <= k <= 100:
        assert np.array_equal(got, one), np.abs(got - one).max()
    else:  # FP32 boxes cannot hold these: no box tests, so some 90 terms a particle in another order
        assert np.abs(got - one).max() <= 90 * 2.0 ** -53 * np.abs(one).max()
