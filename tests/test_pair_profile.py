"""tn_plan_profile refuses a pairwise plan, which has no slices and no control
block on the device."""
import pytest

from paper_2111_01066_amd import tnrcs


def _refused(dry_run):
    pp = tnrcs.PairPlan([0, 1, 2], [2, 3], [0, 1, 3], dry_run=dry_run)
    n = tnrcs.ctypes.c_int32()
    rc = tnrcs._lib.tn_plan_profile(pp._h, 0, tnrcs.c_void_p(4096), None, None, 0, tnrcs.byref(n))
    pp.close()
    return rc


def test_dry_run():
    assert _refused(True) == -1


@pytest.mark.gpu
def test_device_plan():
    print("profile of a pairwise plan", flush=True)
    assert _refused(False) == -1
