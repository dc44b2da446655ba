"""What the library launches, recorded on the CPU (launch_util.py): every call
stays within the runtime's launch limits up to its largest sizes, and the
timing record counts what was launched."""
import os
import re

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


# kernel -> class of the timing record (bgpo_timing); k_gemm4w by its epilogue
# and the layout of its A operand (the dW GEMM's is the transposed one)
CLASS_OF = {"k_transpose_w": 0, "k_masks_and_w": 0, "k_mask_compact": 1, "k_timesteps": 1, "k_mask_bits": 1,
            "k_mask_scan": 1, "k_mask_scatter": 1, "k_row_rms": 2, "k_gather": 2, "k_combine_rows": 4,
            "k_seq_terms": 4, "k_mean_ratio": 4, "k_row_termsILb0E": 4, "k_row_termsILb1E": 5,
            "k_gemm4w_dx_dw": 6, "k_dx_reduce": 7, "k_dgamma": 7}


def _class_of(name):
    m = re.search(r"k_gemm4wILi(\d)ELi(\d)E", name)
    if m:
        epi, layout = int(m[1]), int(m[2])
        return 3 if epi < 2 else 9 if epi == 4 else 8 if layout == 1 else 6
    return next(c for k, c in CLASS_OF.items() if k in name)


@pytest.mark.parametrize("fn", CALLS)
@pytest.mark.parametrize("kw", [
    dict(B=2, L=64, d=128, V=1024, n_t=10),                          # masks beside W, dW beside dX
    dict(B=2, L=64, d=128, V=1024, n_t=10, vocab_chunk=256),         # recompute
    dict(B=2, L=64, d=128, V=1024, n_t=10, sample_stride=64 * 128),  # overlapping samples: a reduction each
    dict(B=2, L=64, d=128, V=1024, n_t=10, sample_stride=2 * 64 * 128),
    dict(B=2, L=64, d=128, V=1024, n_t=10, bound=3),
    dict(B=2, L=64, d=128, V=1024, n_t=10, bound=3, retain_samples=1),
    dict(B=8, L=512, d=256, V=4096, n_t=9),                          # masks of a launch of their own
    dict(B=1, L=65537, d=64, V=128, n_t=3),                          # multi-block masks
    dict(B=2, L=500, d=1024, V=65600, n_t=10, ws_budget=400 << 20),  # dW batches that end themselves
    dict(B=8, L=512, d=4096, V=126464, n_t=64),
], ids=lambda kw: " ".join(f"{k}={v}" for k, v in kw.items()))
def test_timing_record_counts_the_launches_made(recorder, fn, kw):
    """Per class, the record's count is the number of its kernels launched, and
    every launch lies inside an interval of its class (the recorder's events
    measure launches)."""
    from paper_2510_11683_amd import bgpo as b
    r, = record(recorder, [_call(fn, b.Problem(**kw), "timing", "ptr" if kw.get("bound") else None)])
    assert r["status"] == 0
    want = [0] * len(b.KERNEL_CLASSES)
    for name, _, _ in r["launches"]:
        want[_class_of(name)] += 1
    assert dict(zip(b.KERNEL_CLASSES, r["counts"])) == dict(zip(b.KERNEL_CLASSES, want))
    assert r["ms"] == want


@pytest.mark.parametrize("V,copied", [
    (32768, True), (65536, True), (88064, True),                         # rows a multiple of 2 KB apart
    (32512, True), (33024, True), (65024, True), (66048, True), (99072, True),   # of 127 or 129 x 512 bytes
    (32000, False), (60928, False), (65600, False), (70656 - 64, False), (126464, False), (151936, False),
])
def test_short_calls_copy_w_at_slow_row_pitches_only(recorder, V, copied):
    """Which W the dX GEMM of a call over 512 positions reads: its slab-major copy
    (layout 2) or the caller's rows (0); over 16384 positions always the copy."""
    from paper_2510_11683_amd import bgpo as b
    probs = [b.Problem(B, L, 1024, V, 1) for B, L in ((2, 256), (16, 1024))]
    res = record(recorder, [_call("bgpo_elbo_bwd_accumulate", p) for p in probs])
    layouts = [{m[1] for n, _, _ in r["launches"] for m in [re.search(r"k_gemm4wILi2ELi(\d)E", n)] if m}
               for r in res]
    assert layouts == [{"2" if copied else "0"}, {"2"}]
