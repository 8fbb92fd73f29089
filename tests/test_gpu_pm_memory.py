"""The mesh order of the particle-mesh calls is kept for reuse, but never at the cost of another buffer."""
import pytest

from paper_2006_14952_amd import inputs

N, MESH = 1 << 20, 64


def _close(a, b):
    assert float((a - b).norm()) < 1e-10 * float(b.norm())


@pytest.mark.gpu
def test_a_tree_takes_the_room_of_the_kept_order():
    """A bound that holds the meshes with the order, or with the tree, but not with both."""
    import torch

    import paper_2006_14952_amd as hf
    pos, m = (torch.tensor(a, device="cuda") for a in inputs.clustered(N, 40, inputs.rng_for(658)))
    prm = hf.params(r_s=1.25 / MESH, p=3, n_crit=48, precision=1)
    ref = hf.pm_long_range(pos, m, prm, MESH).clone()
    held = hf.memory_in_use()
    t = hf.Tree().build(pos, m, prm)
    want = t.short_range(prm).clone()
    torch.cuda.synchronize()
    tree = hf.memory_in_use() - held
    t.free()
    assert hf.memory_in_use() <= held
    hf.pm_long_range(pos, m, prm, MESH)
    try:
        hf.set_memory_limit(held + tree - 35 * N)  # the order is 70 bytes a particle at least
        t = hf.Tree().build(pos, m, prm)
        got = t.short_range(prm)
        torch.cuda.synchronize()
        assert float((got - want).abs().max()) <= 1e-5 * float(want.abs().max())
        _close(hf.pm_long_range(pos, m, prm, MESH), ref)  # with no room for the order
        t.free()
        _close(hf.pm_long_range(pos, m, prm, MESH), ref)
    finally:
        hf.set_memory_limit(0)


@pytest.mark.gpu
def test_a_bound_below_what_is_held_gives_the_order_back():
    import torch

    import paper_2006_14952_amd as hf
    pos, m = (torch.tensor(a, device="cuda") for a in inputs.clustered(N, 40, inputs.rng_for(658)))
    prm = hf.params(r_s=1.25 / MESH)
    ref = hf.pm_long_range(pos, m, prm, MESH).clone()
    held = hf.memory_in_use()
    try:
        hf.set_memory_limit(1)
        assert hf.memory_in_use() <= held - 56 * N
    finally:
        hf.set_memory_limit(0)
    _close(hf.pm_long_range(pos, m, prm, MESH), ref)
    torch.cuda.synchronize()
    assert hf.memory_in_use() >= 56 * N
