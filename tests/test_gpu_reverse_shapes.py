"""The reverse-pair index at both launch shapes (on either side of 32,768
atoms): rows shorter and longer than the lanes of an atom, repeated entries
(the first one counts) and an entry without a reverse (-1, reported)."""
import numpy as np
import pytest

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 1213, 1214, 1300])
def test_reverse_index(copies):
    rng = np.random.default_rng(3)
    n = 27                                   # copies x 27 = 32,751 and 32,778 around the switch
    rows = [[] for _ in range(n)]
    for i in range(n):
        for _ in range(int(rng.integers(0, 60)) if i % 5 else 0):
            j, s = int(rng.integers(n)), tuple(int(v) for v in rng.integers(-2, 3, 3))
            rows[i].append((j, s))
            rows[j].append((i, tuple(-v for v in s)))
    rows[4].append((7, (3, 3, 3)))           # no reverse
    off = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
    say(f"[gpu] reverse index N={n * copies} rows {min(map(len, rows))}..{max(map(len, rows))}")
    first = {}
    for i, r in enumerate(rows):
        for k, (j, s) in enumerate(r):
            first.setdefault((i, j, s), int(off[i]) + k)
    want = np.array([first.get((j, i, tuple(-v for v in s)), -1) for i, r in enumerate(rows) for j, s in r])
    assert (want < 0).sum() == 1
    P = int(off[-1])
    j = np.array([e[0] for r in rows for e in r])
    sh = wl.pack_shift(np.array([e[1] for r in rows for e in r]))
    big = np.arange(copies)[:, None]
    nb = pod.DeviceNeighbors(np.concatenate([(off[:-1] + big * P).ravel(), [copies * P]]), (j + big * n).ravel(),
                             np.tile(sh, copies))
    m = pod.PodModel(pod.setup_from_workload(wl.SETUP_CFG1), "f64")
    rev = nb.build_reverse(m, check=False).cpu().numpy().reshape(copies, P)
    with pytest.raises(pod.PodError) as e:
        m.check()
    assert pod.ERRORS[e.value.code] == "POD_ENEIGH"
    assert np.array_equal(rev, np.where(want < 0, -1, want + big * P))
