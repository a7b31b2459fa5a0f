"""Order of the device neighbour list and the reverse-pair index, exactly.

The list's contract fixes the order of each atom's row: bins of the home cell
by (z, y, x) offset from the atom's own, the atoms of a bin by index.  The
reference walks the bins serially in that order (plain Python), so the rows
must be equal entry by entry, at cells from one bin (several images, more
segments than the search has lanes per atom) to many, with rows holding
fewer and more candidates than lanes.  Pairs within 1e-9 A of the radius
would be ambiguous; the seeds have none (asserted)."""
import numpy as np
import pytest

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu

S = wl.PodSetup(0.5, 5.0, 8, 4, 4, 4, 3, 3)


def _serial_list(pos, cell, rlist):
    inv = np.linalg.inv(cell)
    height = 1.0 / np.linalg.norm(inv, axis=0)
    nb = np.maximum(1, np.minimum(256, np.floor(height / rlist))).astype(int)
    ns = np.ceil(rlist * nb / height * (1.0 + 1e-12)).astype(int)
    frac = pos @ inv
    wrap = np.floor(frac).astype(int)
    bins = np.clip(((frac - wrap) * nb).astype(int), 0, nb - 1)
    home = pos - wrap @ cell
    members = {}
    for i, b in enumerate(map(tuple, bins)):
        members.setdefault(b, []).append(i)
    rows, near = [], np.inf
    for i in range(len(pos)):
        row = []
        for dz in range(-ns[2], ns[2] + 1):
            for dy in range(-ns[1], ns[1] + 1):
                for dx in range(-ns[0], ns[0] + 1):
                    b = bins[i] + (dx, dy, dz)
                    image = np.floor_divide(b, nb)
                    for j in members.get(tuple(b - image * nb), ()):
                        if j == i and not image.any():
                            continue
                        d = home[j] + image @ cell - home[i]
                        r = np.sqrt(d @ d)
                        near = min(near, abs(r - rlist))
                        if r < rlist:
                            row.append((j, *(image - wrap[j] + wrap[i])))
        rows.append(row)
    assert near > 1e-9
    return rows


@pytest.mark.parametrize("n, edges, rlist, spread", [
    (1, (3.0, 4.0, 5.5), 5.0, 0.0),          # one atom, one bin, only images
    (15, (6.0, 9.0, 11.0), 5.0, 0.0),        # a partial group of lanes; 1 to 2 bins a side
    (17, (5.2, 10.3, 16.0), 5.0, 30.0),      # atoms far outside the home cell
    (60, (26.0, 6.0, 3.2), 5.0, 0.0),        # five bins along x, thin along z
    (130, (11.0, 11.0, 11.0), 5.0, 5.0),     # dense: more candidates in a row of bins than lanes
    (33, (2.1, 12.0, 12.0), 6.0, 0.0),       # seven images along x: more segments than lanes
])
def test_rows_in_scan_order(n, edges, rlist, spread):
    say(f"[gpu] neighbour order n={n} edges={edges} rlist={rlist}")
    rng = np.random.default_rng(n)
    cell = np.diag(edges) + np.tril(rng.uniform(-0.3, 0.3, (3, 3)), -1)
    pos = rng.uniform(0, 1, (n, 3)) @ cell + np.round(rng.normal(0.0, spread / 10.0, (n, 3))) @ cell
    rows = _serial_list(pos, cell, rlist)
    m = pod.PodModel(pod.setup_from_workload(S), "f64")
    nb = pod.DeviceNeighbors.build(m, pos, cell, rlist)
    off, j, sh = (t.cpu().numpy() for t in (nb.offsets, nb.nbr_j, nb.shift))
    shift = np.stack([(sh >> (8 * d)).astype(np.int8) for d in range(3)], 1).astype(int)
    got = [[(int(j[p]), *map(int, shift[p])) for p in range(off[i], off[i + 1])] for i in range(n)]
    assert got == rows
    rev = nb.build_reverse(m).cpu().numpy()
    first = {}
    for i, row in enumerate(got):
        for k, e in enumerate(row):
            first.setdefault((i, *e), off[i] + k)
    want = [first[(e[0], i, -e[1], -e[2], -e[3])] for i, row in enumerate(got) for e in row]
    assert rev[:nb.P].tolist() == want
