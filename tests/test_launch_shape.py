"""CPU: the rules that give a launch its workgroups and vectors per lane."""
import ctypes

import pytest

import paper_0901_0638_amd as qm

FAMILIES = ["QM_SHAPE_" + f for f in ("STREAM", "STREAM32", "LIGHT32", "LIGHT64", "NQ32", "NQ64", "GU32", "GU64",
                                      "GEN32", "GEN64", "GT32", "GT64", "GH32", "GH64", "T32", "T64", "H32", "H64")]
CUS = 256


@pytest.fixture(autouse=True)
def no_overrides(monkeypatch):
    for name in FAMILIES + ["QM_UNROLL", "QM_BLOCKS_PER_CU"]:
        monkeypatch.delenv(name, raising=False)


def launch(family, nvec, table=0):
    blocks = ctypes.c_ulonglong()
    u = qm.load().qm_debug_launch(family.encode(), CUS, nvec, table, ctypes.byref(blocks))
    assert u in (1, 2, 4) and 1 <= blocks.value < 1 << 23
    return u, blocks.value


def test_unknown_family():
    assert qm.load().qm_debug_launch(b"QM_SHAPE_X", CUS, 1, 0, ctypes.byref(ctypes.c_ulonglong())) == -1


@pytest.mark.parametrize("family", FAMILIES)
def test_overrides_hold_for_every_size(family, monkeypatch):
    """QM_UNROLL, or "0,u" for one family: that many vectors per lane, from the
    smallest launch to the largest; a number of workgroups caps them all."""
    sizes = [0, 1, 1 << 16, 1 << 22, 1 << 25, 1 << 27, 1 << 29]
    for u in (1, 2, 4):
        monkeypatch.setenv("QM_UNROLL", str(u))
        assert [launch(family, n)[0] for n in sizes] == [u] * len(sizes)
        monkeypatch.delenv("QM_UNROLL")
        monkeypatch.setenv(family, "0,%d" % u)
        assert [launch(family, n)[0] for n in sizes] == [u] * len(sizes)
        monkeypatch.setenv(family, "3,%d" % u)
        assert max(launch(family, n)[1] for n in sizes) == 3 * CUS
        monkeypatch.delenv(family)


@pytest.mark.parametrize("family", FAMILIES)
def test_large_launches(family):
    """From 2 GB of one array on (2^27 vectors): one tile of four vectors to a
    workgroup for the families that gain by it; two tiles of their own else."""
    u, blocks = launch(family, 1 << 27)
    if family[9:] in ("STREAM", "LIGHT64", "NQ64", "T32", "T64", "H32"):
        assert (u, blocks) == (4, 1 << 17)
    elif family[9:] in ("STREAM32", "LIGHT32", "NQ32"):
        assert (u, blocks) == (4, 1 << 16)
    elif family == "QM_SHAPE_H64":
        assert (u, blocks) == (2, 1 << 17)


@pytest.mark.parametrize("family", ["QM_SHAPE_LIGHT32", "QM_SHAPE_LIGHT64", "QM_SHAPE_NQ64"])
def test_light_maps_take_two_vectors(family):
    """Arrays of 32 to 256 MB: with four vectors in flight these lost up to a
    fifth to the grids before on some cards."""
    for lg in (21, 22, 23):
        assert launch(family, 1 << lg) == (2, min(64 * CUS, (1 << lg) // 512))


@pytest.mark.parametrize("family,per_unit", [("T32", 2), ("T64", 2), ("H32", 16), ("H64", 16)])
def test_large_tables_are_staged_by_few_workgroups(family, per_unit):
    """More than 24 KB to stage: large launches keep a fixed grid."""
    family = "QM_SHAPE_" + family
    for nvec in (1 << 24, 1 << 26, 1 << 28):
        assert launch(family, nvec, 24 * 1024) == launch(family, nvec)
        assert launch(family, nvec)[1] > 64 * CUS - 1
        assert launch(family, nvec, 28 * 1024) == (4, per_unit * CUS)
    assert launch(family, 1 << 21, 50 * 1024) == launch(family, 1 << 21)
