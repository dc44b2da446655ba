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


CALLS = ("bgpo_elbo_fwd", "bgpo_elbo_bwd_accumulate", "bgpo_elbo_fwd_rmsnorm",
         "bgpo_elbo_bwd_accumulate_rmsnorm")


def _call(fn, p, timing=None, ell_old=None):
    norm = ["ptr"] if fn.endswith("rmsnorm") else []
    head, tail = [("prob", bytes(p.c())), "ptr", *norm, "ptr", "ptr", "ptr"], ["ws", None, timing]
    if "fwd" in fn:
        return fn, [*head, "ptr", "ptr", None, *tail]
    return fn, [*head, "ptr", ell_old, 0.125, "ptr", *norm, "ptr", "ptr", "ptr", "ptr", "ptr", None, None, *tail]


def test_launches_at_the_corners_of_the_supported_shapes(recorder):
    """Smallest and largest B*L, d and V, all at once too: every launch is
    accepted, and the W copies and the gather have a workgroup for every 64 x 64
    tile (one head of 2^36 weights fits a GPU twice: its forward is a call that
    can be made)."""
    from paper_2510_11683_amd import bgpo as b
    todo = []
    for B, L, n_t in ((1, 1, 1), (1, 1 << 20, 1), (600, 1, 1), (4096, 256, 1), (1, 1 << 19, 8)):
        for d in (64, 65536):
            for V in (64, 1 << 20):
                for f32 in (0, 1):
                    for kw in ({}, dict(vocab_chunk=256, ws_budget=1 << 44)):
                        p = b.Problem(B, L, d, V, n_t, in_dtype=f32, **kw)
                        todo += [(p, fn) for fn in CALLS]
    for (p, fn), r in zip(todo, record(recorder, [_call(fn, p) for p, fn in todo])):
        assert r["status"] == 0, (p, fn)
        G = b.bgpo_workspace_plan(p)["samples_per_unit"]
        rows = min(G, p.n_t) * ((p.B * p.L + 255) // 256 * 256)
        need = {"transpose_w": p.d // 64 * (p.V // 64), "masks_and_w": p.d // 64 * (p.V // 64),
                "k_gather": rows // 64 * (p.d // 64)}
        for k, n in need.items():      # (a range's last unit may be smaller)
            wgs = [grid[0] * grid[1] for name, grid, _ in r["launches"] if k in name]
            assert not wgs or max(wgs) >= n, (p, fn, k, wgs)
