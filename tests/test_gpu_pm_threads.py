"""Mesh calls of several threads: they share the mesh part one after the other, and nothing else."""
import threading
import time

import numpy as np
import pytest

from paper_2006_14952_amd import inputs


def _box(n, seed, device="cuda"):
    import torch
    pos, m = inputs.uniform(n, inputs.rng_for(657, seed))
    return [torch.tensor(a, device=device) for a in (pos, m)]


@pytest.mark.gpu
def test_a_hybrid_steps_short_range_holds_no_other_threads_mesh_call():
    """Small mesh calls go on while another thread's hybrid step traverses its tree and evaluates P2P."""
    import torch

    import paper_2006_14952_amd as hf
    d, small = _box(200000, 1), _box(1000, 2)
    prm = hf.params(r_s=0.1 / 4.5, r_cut=0.1, theta=0.15, p=2, n_crit=4, precision=1)
    prm_small = hf.params(r_s=0.05)
    t, sa, sb = hf.Tree(), torch.cuda.Stream(), torch.cuda.Stream()
    acc, acc_small = torch.empty_like(d[0]), torch.empty_like(small[0])
    torch.cuda.synchronize()
    for _ in range(2):
        t.hybrid(*d, prm, 32, out=acc, stream=sa)
        hf.pm_long_range(*small, prm_small, 16, out=acc_small, stream=sb)
    torch.cuda.synchronize()
    calls, stop = [], threading.Event()

    def other():
        while not stop.is_set():
            t0 = time.perf_counter()
            hf.pm_long_range(*small, prm_small, 16, out=acc_small, stream=sb)
            calls.append((t0, time.perf_counter()))

    th = threading.Thread(target=other)
    th.start()
    time.sleep(0.05)
    share = []
    for _ in range(15):
        t0 = time.perf_counter()
        t.hybrid(*d, prm, 32, out=acc, stream=sa)
        sa.synchronize()
        t1 = time.perf_counter()
        time.sleep(0.02)
        inside = [min(b, t1) - max(a, t0) for a, b in calls if b > t0 and a < t1]
        share.append(max(inside) / (t1 - t0))
    stop.set()
    th.join()
    # a call that waits for the whole step takes some nine tenths of it
    assert np.median(share) < 0.7, share


@pytest.mark.gpu
def test_threads_on_one_mesh_get_their_own_forces():
    import torch

    import paper_2006_14952_amd as hf
    mesh, reps = 48, 8
    boxes = [_box(n, 10 + k) for k, n in enumerate((30000, 20000, 50000, 700))]
    prm = [hf.params(r_s=1.25 / mesh, p=3, n_crit=16, precision=p) for p in (0, 1, 1, 0)]
    trees, streams = [hf.Tree() for _ in range(3)], [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()

    def call(k):
        with torch.cuda.stream(streams[k]):
            if k < 3:
                return trees[k].hybrid(*boxes[k], prm[k], mesh, stream=streams[k])
            return hf.pm_long_range(*boxes[k], prm[k], mesh, stream=streams[k])

    alone = []
    for k in range(4):
        alone.append(call(k))
        torch.cuda.synchronize()
    got, errors = [[] for _ in range(4)], []

    def work(k):
        try:
            for _ in range(reps):
                got[k].append(call(k))
            streams[k].synchronize()
        except Exception as e:  # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for k in range(4):
        scale = float(alone[k].norm(dim=1).max())
        for a in got[k]:  # the atomics' order varies: the bounds the header gives, 1e-11 and 1e-5
            assert float((a - alone[k]).abs().max()) <= (1e-5 if prm[k].precision else 1e-11) * scale
