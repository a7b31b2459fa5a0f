"""The library's own launch shape is the autotuner's first candidate, and picks
cached for other kernels are measured again."""
from paper_2212_14446_amd import autotune as at


def test_library_choice_comes_first():
    c = at.candidates()
    assert c[0] == (0, 0, 0)
    # nothing beats it by the margin: the library's choice stays
    assert at.tune("k", lambda x: 1.0 if x == (0, 0, 0) else 0.99, None) == (0, 0, 0)
    assert at.tune("k", lambda x: 1.0 if x == (0, 0, 0) else 0.9, None) == c[1]
    assert len(set(c)) == len(c)


def test_signature_names_the_kernels(monkeypatch):
    args = (3, [2, 10, 250], [20, 200, 6000], 103, 6, 4)
    a = at.signature(*args)
    monkeypatch.setattr(at, "KERNELS", at.KERNELS + 1)
    assert at.signature(*args) != a
