"""What the library launches, recorded on the CPU (launch_util.py): every call
stays within the runtime's launch limits up to its largest sizes."""
import os

import pytest

from launch_util import LIB, build_recorder, record

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libbgpo.so not built")


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return build_recorder(str(tmp_path_factory.mktemp("rec") / "librec.so"))


def test_moments_update_takes_any_length(recorder):
    """The header bounds n nowhere; the runtime refuses 2^32 work-items in one
    dimension.  (Three arrays of 2^34 floats are 206 GB.)"""
    ns = (1, 1024, 1025, (24 << 20) + 1, (1 << 34) - 1024, 1 << 34, (1 << 34) + 5, 1 << 40)
    res = record(recorder, [("bgpo_moments_update", ["ptr", "ptr", "ptr", n, ("i32", 3), None]) for n in ns])
    for n, r in zip(ns, res):
        assert r["status"] == 0, n
        (name, grid, block), = r["launches"]
        assert "k_moments_update" in name and grid[0] * 1024 >= min(n, 1 << 32), (n, grid)
