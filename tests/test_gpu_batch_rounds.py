"""A batch beyond the 2 GB of one round of pod_batch_assemble: copies of a set
of cells, enough for several rounds, against the set by itself (which the
parity tests pin to the oracle).  The same sums in another order of a few
hundred terms at most: 1e-12 of the largest entry."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


def test_several_rounds():
    s = wl.SETUP_CFG2
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    b = wl.make_batch(40, 5, s, n_min=100, n_max=250)
    nl, copies = b.nl, 90
    N, P = int(b.N), int(nl.n_pairs)
    K, PA = 6, 4
    rows = K * ((PA + 1) * (PA + 2) * (PA + 3) // 6 + PA + 1) * 8
    assert copies * (P * ((4 + 2 * K) * 8 + 4) + N * rows) > 2 * 2 ** 30   # at least two rounds
    say(f"[gpu] batch in several rounds: {copies * b.n_cfg} cells, {copies * N} atoms")
    one = pod.batch_assemble(m, pod.DeviceBatch.from_batch(b))
    off = np.concatenate([np.asarray(b.cfg_atom_off[:-1], np.int64) + k * N for k in range(copies)] + [[copies * N]])
    offs = np.concatenate([nl.offsets[:-1].astype(np.int64) + k * P for k in range(copies)] + [[copies * P]])
    j = (nl.nbr_j[None].astype(np.int64) + np.arange(copies)[:, None] * N).ravel()
    big = pod.DeviceBatch(off, np.tile(b.pos, (copies, 1)), np.tile(np.asarray(b.cells).reshape(-1, 9), (copies, 1)),
                          offs, j, np.tile(nl.shift, copies))
    out = pod.batch_assemble(m, big)
    for k in ("D", "G", "dGdR"):
        ref, got = one[k], out[k].view(copies, *one[k].shape)
        assert float((got - ref).abs().max()) <= 1e-12 * float(ref.abs().max()), k


def test_more_cells_than_a_launch_takes():
    """2^20 + 3 equal dimers, one column per chunk: more cells than a round has
    and more items than a launch has workgroups.  Every cell as the first."""
    s = wl.PodSetup(0.5, 5.0, 6, 4, 4, 0, 3, 0)
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    n = 2 ** 20 + 3
    say(f"[gpu] batch of {n} dimers")
    x = np.array([[0.1, 0.2, 0.3], [1.1, 2.0, 2.3]])
    cell = 40.0 * np.eye(3).reshape(1, 9)

    def batch(k):
        one = np.arange(2 * k).reshape(k, 2)
        return pod.DeviceBatch(2 * np.arange(k + 1), np.tile(x, (k, 1)), np.tile(cell, (k, 1)), np.arange(2 * k + 1),
                               one[:, ::-1].ravel(), np.zeros(2 * k, np.int32))

    ref = pod.batch_assemble(m, batch(1), tune=(1, 0, 0))
    out = pod.batch_assemble(m, batch(n), tune=(1, 0, 0))
    for k in ("D", "G", "dGdR"):
        assert float(ref[k].abs().max()) > 0.0
        got = out[k].view(n, *ref[k].shape)
        assert float((got - ref[k]).abs().max()) <= 1e-13 * float(ref[k].abs().max()), k
