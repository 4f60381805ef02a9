"""Saved tuning tables of earlier candidate numbers: their entries keep their
shapes.  No GPU."""
import pytest

FIELDS = ("bm", "bn", "bk", "waves_m", "waves_n", "split_k", "prefetch")


@pytest.fixture
def li():
    from paper_2312_13170_amd import li as mod
    families = range(7)
    old = {(k, b): mod.li_tune_get(k, b) for k in families for b in range(64)}
    yield mod
    for (k, b), v in old.items():
        mod.li_tune_set(k, b, v)


# the candidates of version 1 that other shapes took the numbers of
VERSION_1 = {
    (1, 10): (128, 128, 32, 4, 4, 7, 2),
    (1, 20): (128, 128, 32, 4, 4, 0, 4),
    (1, 21): (64, 64, 32, 2, 2, 0, 2),
    (3, 9): (64, 64, 32, 2, 2, 4, 2),
    (3, 10): (64, 64, 32, 2, 2, 1, 3),
    (3, 14): (64, 64, 32, 2, 2, 0, 2),
    (3, 15): (128, 128, 32, 4, 4, 0, 4),
    (4, 0): (128, 128, 32, 2, 4, 1, 3),
    (4, 1): (64, 64, 32, 2, 2, 1, 3),
    (4, 2): (32, 32, 32, 1, 1, 1, 3),
    (5, 0): (128, 128, 32, 2, 4, 1, 3),
    (5, 1): (64, 64, 32, 2, 2, 1, 3),
    (5, 2): (32, 32, 32, 1, 1, 1, 3),
    # unchanged numbers
    (0, 44): (128, 128, 32, 4, 4, 1, 8),
    (1, 17): (64, 64, 32, 2, 2, 1, 4),
    (3, 6): (128, 128, 32, 4, 4, 7, 2),
    (6, 12): (256, 256, 64, 2, 4, 1, 3),
}


def shape(li, family, idx):
    c = li.li_tune_candidate(family, idx)
    return tuple(c[f] for f in FIELDS)


@pytest.mark.parametrize("header", ["# li tuning table (gfx950): kernel slot candidate\n", ""])
def test_version_1_entries_keep_their_shapes(li, tmp_path, header):
    path = tmp_path / "old.txt"
    slots = {key: 30 + i for i, key in enumerate(VERSION_1)}
    path.write_text(header + "".join("%d %d %d\n" % (k, b, i) for (k, i), b in slots.items()))
    li.li_tune_load(str(path))
    for (k, i), b in slots.items():
        assert shape(li, k, li.li_tune_get(k, b)) == VERSION_1[(k, i)], (k, i)


def test_present_numbers_survive_a_file(li, tmp_path):
    path = tmp_path / "new.txt"
    for (k, i) in VERSION_1:
        li.li_tune_set(k, 30 + i % 8, i)
    want = {(k, b): li.li_tune_get(k, b) for k in range(7) for b in range(64)}
    li.li_tune_save(str(path))
    for (k, b) in want:
        li.li_tune_set(k, b, -1)
    li.li_tune_load(str(path))
    assert {(k, b): li.li_tune_get(k, b) for (k, b) in want} == want


def test_unknown_version_is_refused(li, tmp_path):
    path = tmp_path / "next.txt"
    before = li.li_tune_get(1, 30)
    path.write_text("# li tuning table (gfx950) version 99: kernel slot candidate\n1 30 0\n")
    with pytest.raises(li.LiError):
        li.li_tune_load(str(path))
    assert li.li_tune_get(1, 30) == before


def test_default_search_keeps_the_rules(li):
    # the shipped table and the default search hold the same families, so that
    # a search does not write over the rules of the others
    import os
    from paper_2312_13170_amd import autotune
    assert autotune.parser().parse_args([]).only == "lp"
    table = os.path.join(os.path.dirname(autotune.__file__), "tune_gfx950.txt")
    lines = [l.split() for l in open(table) if l.strip() and not l.startswith("#")]
    assert {int(l[0]) for l in lines} == {li.LI_KERNEL_GEMM_LP, li.LI_KERNEL_GEMM_LP_SPLIT}
