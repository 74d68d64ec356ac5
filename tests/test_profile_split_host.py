"""The counter summaries know every kernel of an FP64 CG iteration by the names it has now, the direction-split hop of
small lattices among them, and are stamped with every source that a hop is built from."""
import os

import pytest

from paper_1710_09621_amd import profile_summary as PS

SPLIT = "void eofa::(anonymous namespace)::k_hop_split<%s>(eofa::HopArgsMR<%s>)"
XP = "void eofa::k_cg_xp<%s>(eofa::cpx<double>*, eofa::cpx<double>*, eofa::cpx<double> const*, double*, unsigned long, eofa::XpFin)"


@pytest.mark.parametrize("name,cls", [
    (SPLIT % ("16, false, 1, false, double, false", "double"), "hop"),
    (SPLIT % ("16, false, 2, true, double, false", "double"), "schur_w"),
    (SPLIT % ("16, true, 1, false, double, false", "double"), "hop_dag"),
    (SPLIT % ("16, true, 3, true, double, false", "double"), "schur_q"),
    (SPLIT % ("16, false, 1, false, float, false", "float"), None),
    (SPLIT % ("16, false, 2, true, float, true", "float"), None),
    (SPLIT % ("16, false, 4, false, double, false", "double"), None),
    (XP % "double, true, false", "xp"), (XP % "double, false, false", "xp"), (XP % "double, false, true", "xp"),
    (XP % "float, false, true", None)])
def test_cg_kernel_classes(name, cls):
    assert PS._cg_class(name) == cls


def test_stamp_covers_every_hop_source():
    """Every source of the library that defines or includes a part of the hop kernels."""
    csrc = os.path.join(PS.ROOT, "paper_1710_09621_amd", "csrc")
    hop = [f for f in os.listdir(csrc) if "k_hop" in open(os.path.join(csrc, f)).read() and f.endswith((".hip", ".h"))]
    assert {os.path.join("paper_1710_09621_amd", "csrc", f) for f in hop} <= set(PS.KERNEL_SOURCES)
