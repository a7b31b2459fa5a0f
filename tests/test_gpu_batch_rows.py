"""The rows and chunks of the batched derivatives: every (cell, atom, column)
against the oracle at the sizes where the work items change shape -- cells of
1, 63, 64, 65 and 129 atoms (blocks of 64 atoms), models whose radial counts
differ per body order (radial indices without some of the columns), degrees
from 0 to 6 (every class of rows), chunks of one column up to all of them,
and a batch whose records need several rounds.

Tolerance: FP64 sums of at most a few thousand terms against an oracle in
another order, 1e-10 relative to the largest entry of a column."""
import numpy as np
import pytest
import torch

from gpu_common import colerr, oracle_params, relerr, say
from oracle import pod_oracle as po
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu

TOL = 1e-10


def _batch(sizes, setup, seed):
    rng = np.random.default_rng(seed)
    kinds, poss, cells, lists = [], [], [], []
    for n in sizes:
        kind = ["bcc", "fcc", "a15"][int(rng.integers(3))]
        pos, cell = wl.small_cell(kind, n, float(rng.uniform(0.9, 1.1)), 0.1, rng)
        kinds.append(kind)
        poss.append(pos)
        cells.append(cell)
        lists.append(wl.neighbor_list(pos, cell, setup.rcut))
    off = np.concatenate([[0], np.cumsum([len(p) for p in poss])])
    poff = np.concatenate([[0], np.cumsum([nl.n_pairs for nl in lists])])
    offsets = np.concatenate([[0]] + [nl.offsets[1:].astype(np.int64) + poff[c] for c, nl in enumerate(lists)])
    nbr_j = np.concatenate([nl.nbr_j.astype(np.int64) + off[c] for c, nl in enumerate(lists)])
    shift3 = np.concatenate([nl.shift3 for nl in lists]).astype(np.int32)
    nl = wl.NeighborList(offsets.astype(np.int32), nbr_j.astype(np.int32), shift3, wl.pack_shift(shift3))
    return wl.Batch(kinds, off.astype(np.int32), np.concatenate(poss), np.stack(cells), nl, setup)


def _check(setup, sizes, tunes, seed):
    op = oracle_params(setup)
    Q, _ = po.pod_basis(op)
    m = pod.PodModel(pod.setup_from_workload(setup), "f64", Q=Q[:, : op.K])
    b = _batch(sizes, setup, seed)
    refs = []
    for c in range(b.n_cfg):
        pos, cell, nl = b.config(c)
        args = (pos, cell, nl.offsets.astype(np.int64), nl.nbr_j, nl.shift3, op, Q)
        dG = po.global_descriptor_derivatives(*args)
        refs.append((po.descriptors_fast(*args), dG.reshape(-1, dG.shape[2])))
    db = pod.DeviceBatch.from_batch(b)
    for tune in tunes:
        say(f"[gpu] batch rows K=({setup.K2},{setup.K3},{setup.K4}) P=({setup.P3},{setup.P4}) tune={tune}")
        o = {k: v.cpu().numpy() for k, v in pod.batch_assemble(m, db, tune=tune).items()}
        D = np.concatenate([r[0] for r in refs])
        dG = np.concatenate([r[1] for r in refs])
        assert colerr(o["D"], D) < TOL
        assert relerr(o["G"], np.stack([r[0].sum(0) for r in refs])) < TOL
        assert np.all(o["dGdR"][:, 0] == 0.0)
        assert colerr(o["dGdR"], dG) < TOL


@pytest.mark.parametrize("K2, K3, K4, P3, P4", [
    (3, 0, 0, 0, 0),     # 2-body columns only
    (0, 3, 2, 1, 0),     # no 2-body column; D4 of degree 0
    (2, 4, 3, 2, 2),     # columns that differ by radial index
    (4, 2, 3, 4, 3),     # 4-body degree below the 3-body one
    (1, 2, 4, 1, 4),     # and above it
])
def test_rows_per_model(K2, K3, K4, P3, P4):
    _check(wl.PodSetup(0.5, 5.0, 6, K2, K3, K4, P3, P4), (2, 17, 65), (None, (1, 0, 64), (5, 3, 128)), 3)


@pytest.mark.parametrize("P3, P4", [(5, 2), (2, 5), (6, 6)])
def test_high_degree_rows(P3, P4):
    _check(wl.PodSetup(0.5, 4.0, 6, 2, 2, 2, P3, P4), (3, 20), (None, (4, 0, 0)), 4)


def test_block_edges():
    _check(wl.PodSetup(0.5, 4.0, 6, 2, 2, 2, 4, 4), (1, 63, 64, 65, 129), (None, (17, 0, 512)), 5)


def test_several_rounds():
    """40 million pairs of a 2/3-body model: more records than one round holds."""
    s = wl.PodSetup(0.5, 5.0, 6, 4, 4, 0, 3, 0)
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    b = _batch((40, 120, 200, 7), s, 6)
    reps = 4200
    N, P, M = b.N, b.nl.n_pairs, m.M
    assert reps * P * (4 + 2 * 4) * 8 > 2 << 30
    off = np.concatenate([b.cfg_atom_off[:-1] + r * N for r in range(reps)] + [[reps * N]])
    offsets = np.concatenate([b.nl.offsets[:-1].astype(np.int64) + r * P for r in range(reps)] + [[reps * P]])
    nbr_j = (b.nl.nbr_j[None, :].astype(np.int64) + np.arange(reps)[:, None] * N).ravel()
    say(f"[gpu] batch rounds cells={reps * b.n_cfg} atoms={reps * N} pairs={reps * P}")
    db = pod.DeviceBatch(off, np.tile(b.pos, (reps, 1)), np.tile(b.cells, (reps, 1, 1)), offsets, nbr_j,
                         np.tile(b.nl.shift, reps))
    one = pod.batch_assemble(m, pod.DeviceBatch.from_batch(b))
    got = pod.batch_assemble(m, db)
    for k, rows in (("D", N), ("G", b.n_cfg), ("dGdR", 3 * N)):
        ref = one[k].reshape(1, rows, M)
        err = (got[k].reshape(reps, rows, M) - ref).abs().max()
        assert float(err) < 1e-11 * float(ref.abs().max())
        del ref
    torch.cuda.empty_cache()
