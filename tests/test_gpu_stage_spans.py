"""Stage spans of an evaluation whose costliest leaves have a P2P launch of their own."""
import pytest

from paper_2006_14952_amd import inputs


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
def test_the_launch_of_the_costliest_leaves_counts_as_p2p(precision):
    """Leaves of some 600 particles are walked in twenty passes, and so cost twenty times their list entries: every one
    has a workgroup.  No pair is accepted for M2L, so M2L's span is that of an empty stage."""
    import torch

    import paper_2006_14952_amd as hf
    pos, m = inputs.uniform(40000, inputs.rng_for(642))
    prm = hf.params(r_s=0.06, r_cut=0.27, theta=1e-9, p=3, n_crit=2000, precision=precision)
    t = hf.Tree().build(torch.tensor(pos, device="cuda"), torch.tensor(m, device="cuda"), prm)
    t.set_timing(True)
    for _ in range(3):
        t.short_range(prm)
    st = t.stats()
    assert st["n_leaves"] == 64 and st["n_m2l"] == 0
    assert 0 < st["t_m2l_ms"] < 0.2 * st["t_p2p_ms"], st
    assert st["t_p2p_ms"] <= st["t_total_ms"]
