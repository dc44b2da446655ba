"""Units of several samples through the kernels that handle a whole unit per
launch: every sample's masks, l, and the gradients against the float64 oracle
at response counts and lengths off the kernels' vector widths.

Bars as in test_gpu_parity.py: counts and timesteps bit-exact, l within 1e-3
relative, dX and dW within 2e-2 relative max-norm (bf16 dZ).
"""
import numpy as np
import pytest
import torch

import workloads
from oracle import elbo
from gpu_util import Runner, lib, rel_maxnorm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib()


@pytest.mark.parametrize("B,L,n_t,lengths", [
    (1, 1, 3, None),            # one position: empty samples among the unit's
    (3, 7, 17, (1, 7)),         # three units of 8, 8, 1; L not a multiple of the Philox block
    (1500, 3, 9, (1, 3)),       # timesteps of two samples at a time in the mask kernel
    (5, 997, 10, (100, 997)),   # more positions than threads
    (512, 4, 4, (1, 4)),        # the most responses and positions drawn beside W's copies
    (513, 3, 4, (1, 3)),        # one response more: a launch of their own
    (2, 4096, 1, (60, 4096)),   # one sample, 32 positions per thread
])
def test_units_of_samples_match_oracle(B, L, n_t, lengths):
    w = workloads.Workload("unit", B=B, L=L, d=128, V=576, n_t=n_t, lengths=lengths, group=B,
                           adv="normal", data_seed=2100 + B, philox_seed=0xB6B30000 + L,
                           seq_id_base=77)
    x = workloads.generate(w)
    ref = elbo.elbo_collapsed(elbo.Problem(B, L, 128, 576, n_t, seed=w.philox_seed, seq_id_base=77),
                              x["hidden"], x["W"], x["targets"], x["resp_mask"], x["adv"])
    r = Runner(w, x)
    r.bwd()
    o = r.out()
    np.testing.assert_array_equal(o["nm"], ref.n_masked)
    np.testing.assert_array_equal(o["t"].astype(np.float64), ref.t)
    assert np.abs(o["ell"] - ref.ell).max() <= 1e-3 * np.abs(ref.ell).max()
    assert rel_maxnorm(o["dX"], ref.dX) <= 2e-2
    assert rel_maxnorm(o["dW"], ref.dW) <= 2e-2
    assert o["flags"] == 0
    r.fwd()
    assert np.array_equal(r.out()["ell"], o["ell"])


@pytest.mark.parametrize("offset", [1, 2, 4])
def test_masks_of_a_misaligned_response_mask(offset):
    """bgpo_sample_masks reads the response mask from any byte address."""
    b = lib()
    B, L = 3, 203
    resp = np.random.default_rng(offset).integers(0, 2, (B, L)).astype(np.uint8)
    buf = torch.zeros(B * L + 8, dtype=torch.uint8, device="cuda")
    view = buf[offset:offset + B * L].view(B, L)
    view.copy_(torch.from_numpy(resp))
    idx = torch.full((B * L,), -1, dtype=torch.int32, device="cuda")
    nm = torch.zeros(B, dtype=torch.int32, device="cuda")
    b.bgpo_sample_masks(b.Problem(B, L, 64, 64, 5, seed=99), view, 2, idx, nm)
    p = elbo.Problem(B, L, 64, 64, 5, seed=99)
    want = elbo.sample_masks(p, resp, 2)[3]
    np.testing.assert_array_equal(idx[:want.size].cpu().numpy(), want)
    assert int(nm.sum()) == want.size


@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("stride_rows", [7, 21, 30])
def test_overlapping_sample_strides(stride_rows, norm):
    """Sample strides below B*L*d (21 rows), where consecutive samples' head
    inputs and dX share rows, and above: one call over a range gives the sum
    of one call per sample at that sample's offset (reassociation of fp32
    sums only: 1e-5)."""
    b = lib()
    B, L, d, V, n_t = 3, 7, 1088, 192, 10
    stride = stride_rows * d
    rng = np.random.default_rng(5)
    rows = (n_t - 1) * stride_rows + B * L
    x = torch.from_numpy(rng.standard_normal((rows, d), dtype=np.float32)).to(torch.bfloat16).cuda()
    W = torch.from_numpy(0.05 * rng.standard_normal((d, V), dtype=np.float32)).to(torch.bfloat16).cuda()
    gamma = torch.from_numpy((1 + 0.1 * rng.standard_normal(d)).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.integers(0, V, (B, L)).astype(np.int32)).cuda()
    resp = torch.ones(B, L, dtype=torch.uint8, device="cuda")
    adv = torch.from_numpy(rng.standard_normal(B).astype(np.float32)).cuda()

    def run(ranges):
        dX = torch.zeros(rows, d, device="cuda")
        dW, dg = torch.zeros(d, V, device="cuda"), torch.zeros(d, device="cuda")
        ell = torch.zeros(B, n_t, dtype=torch.float64, device="cuda")
        g, loss = torch.zeros_like(ell), torch.zeros(1, dtype=torch.float64, device="cuda")
        nm = torch.zeros(B, n_t, dtype=torch.int32, device="cuda")
        for j0, n in ranges:
            p = b.Problem(B, L, d, V, n_t, j_begin=j0, j_count=n, seed=41, sample_stride=stride)
            ws = b.alloc_workspace(p)
            xj, dj = x[j0 * stride_rows:].data_ptr(), dX[j0 * stride_rows:].data_ptr()
            tail = [W, y, resp, adv]
            out = [ell, g, loss, nm]
            a = [t.data_ptr() for t in tail] + [None, 0.125, dj] + ([dg.data_ptr()] if norm else []) + \
                [dW.data_ptr()] + [t.data_ptr() for t in out] + [None, None, ws.data_ptr(), ws.numel(), None, None]
            f = b._lib.bgpo_elbo_bwd_accumulate_rmsnorm if norm else b._lib.bgpo_elbo_bwd_accumulate
            head = [xj] + ([gamma.data_ptr()] if norm else [])
            torch.cuda.synchronize()
            assert f(p.c(), *head, *a) == 0
            torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (dX, dW, dg, ell)]

    for one, many in zip(run([(0, n_t)]), run([(j, 1) for j in range(n_t)])):
        assert rel_maxnorm(one, many) <= 1e-5


@pytest.mark.parametrize("d,V", [
    (64, 64),        # one tile of either size, most of it past the edges
    (128, 128),      # one whole 128-wide tile
    (192, 320),      # ragged in both
    (1024, 8256),    # several 128-wide tiles per workgroup in dW, one in the forward
    (2048, 32064),   # 256-wide tiles in the forward and dW
])
@pytest.mark.parametrize("L", [2, 127, 300])
def test_tile_sizes_match_oracle(d, V, L):
    """The GEMMs on 128-wide and 256-wide tiles, chosen by the sizes, with the
    unit's rows below, around and above a tile; off-policy."""
    w = workloads.Workload("tiles", B=2, L=L, d=d, V=V, n_t=2, lengths=(max(1, L - 5), L), adv="normal",
                           targets="uniform", data_seed=2200 + d, philox_seed=0xB6B40000 + L)
    x = workloads.generate(w)
    p = elbo.Problem(2, L, d, V, 2, seed=w.philox_seed)
    args = (x["hidden"], x["W"], x["targets"], x["resp_mask"], x["adv"])
    old = elbo.elbo_collapsed(p, *args, backward=False).ell + np.random.default_rng(L).normal(0, 0.5, (2, 2))
    ref = elbo.elbo_collapsed(p, *args, ell_old=old)
    r = Runner(w, x)
    r.bwd(ell_old=old)
    o = r.out()
    np.testing.assert_array_equal(o["nm"], ref.n_masked)
    np.testing.assert_allclose(o["ell"], ref.ell, rtol=1e-3, atol=0)
    assert rel_maxnorm(o["dX"], ref.dX) <= 2e-2
    assert rel_maxnorm(o["dW"], ref.dW) <= 2e-2
    r.fwd()
    assert np.array_equal(r.out()["ell"], o["ell"])


@pytest.mark.parametrize("d", [128, 256, 576])
def test_empty_splits_of_the_last_vocabulary_chunk(d):
    """Recompute backward whose last vocabulary chunk (64 ids, one slab) leaves
    splits of the dX GEMM empty: their partials keep the earlier chunks' sums.
    Against the oracle, and l bit-identical to the stored backward."""
    w = workloads.Workload("empty", B=4, L=150, d=d, V=2048 + 64, n_t=3, adv="normal", group=4,
                           data_seed=2300 + d, philox_seed=0xB6B50000 + d)
    x = workloads.generate(w)
    ref = elbo.elbo_collapsed(elbo.Problem(4, 150, d, w.V, 3, seed=w.philox_seed), x["hidden"], x["W"],
                              x["targets"], x["resp_mask"], x["adv"])
    r, q = Runner(w, x, vocab_chunk=1024), Runner(w, x)
    r.bwd()
    q.bwd()
    o = r.out()
    assert np.array_equal(o["ell"], q.out()["ell"])
    assert rel_maxnorm(o["dX"], ref.dX) <= 2e-2
    assert rel_maxnorm(o["dW"], ref.dW) <= 2e-2


@pytest.mark.parametrize("n", [1, 3, 1024, 4097, (24 << 20) - 1, (24 << 20) + 5])
@pytest.mark.parametrize("offset", [0, 1])
def test_moments_around_the_streaming_line(n, offset):
    """Both forms of the moment kernels (streaming from 24 * 2^20 elements), a
    ragged tail, and a summary of arrays off 16 bytes: the update against
    float64 (a few fp32 roundings per element: 1e-6), the summary against
    float64 sums of the same fp32 values (sums of positive terms: 1e-12)."""
    b = lib()
    gen = torch.Generator(device="cuda").manual_seed(n)
    g, mean, m2, ref = (torch.randn(n + offset, generator=gen, device="cuda")[offset:] for _ in range(4))
    m2 = m2.square_()
    if offset == 0:
        delta = g.double() - mean.double()
        want = mean.double() + delta / 3
        want2 = m2.double() + delta * (g.double() - want)
        b.bgpo_moments_update(g, mean, m2, 2)
        assert float((mean.double() - want).norm() / want.norm()) <= 1e-6
        assert float((m2.double() - want2).norm() / want2.norm()) <= 1e-6
        m2.abs_()
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    for r in (ref, None):
        ws = b.moments_workspace()
        st = b._lib.bgpo_moments_summary(mean.data_ptr(), m2.data_ptr(), r.data_ptr() if r is not None else None,
                                         n, 3, out.data_ptr(), ws.data_ptr(), ws.numel(), None)
        torch.cuda.synchronize()
        assert st == 0
        exp = [(m2.double() / 2).sqrt().mean(), 0.0, 0.0]
        if r is not None:
            exp[1:] = (mean.double() - r.double()).abs().mean(), r.double().abs().mean()
        np.testing.assert_allclose(out.cpu().numpy(), [float(e) for e in exp], rtol=1e-12)


@pytest.mark.parametrize("B,L,V", [
    (32, 128, 576),     # the largest call that reads W in place
    (32, 129, 576),     # the smallest that makes the slab-major copy
    (4, 33, 1024),      # rows a multiple of 2 KB apart: the copy at any size
    (1, 33, 33024),     # of 129 times 512 bytes: the same
])
def test_w_in_place_or_copied(B, L, V):
    """The dX GEMM on the caller's row-major bf16 W and on its slab-major copy,
    around the line between them; the call's two samples split in two calls
    (in place) give the same dX up to the order of the fp32 sums over the
    vocabulary splits (1e-5)."""
    w = workloads.Workload("copy", B=B, L=L, d=192, V=V, n_t=2, adv="normal", group=4, data_seed=2400 + L,
                           philox_seed=0xB6B60000 + L)
    x = workloads.generate(w)
    ref = elbo.elbo_collapsed(elbo.Problem(B, L, 192, V, 2, seed=w.philox_seed), x["hidden"], x["W"],
                              x["targets"], x["resp_mask"], x["adv"])
    r, q = Runner(w, x), Runner(w, x)
    r.bwd()
    for j in range(2):
        q.bwd(j_begin=j, j_count=1)
    o = r.out()
    assert rel_maxnorm(o["dX"], ref.dX) <= 2e-2
    assert rel_maxnorm(o["dW"], ref.dW) <= 2e-2
    assert rel_maxnorm(q.out()["dX"], o["dX"]) <= 1e-5


@pytest.mark.parametrize("budget_mib", [400, 450])
def test_dw_batches_end_where_rows_no_longer_fit(budget_mib):
    """Units of one sample on buffers for one and for two fully masked units:
    how many of the partly masked ones share a dW GEMM follows from their rows
    (responses of 500 with random timesteps: some pairs fit in one unit's rows,
    some do not).  The whole range in one call against one call per sample on
    the same layout, which flushes after each: dX bit for bit, dW up to the
    order of fp32 sums (1e-5)."""
    b = lib()
    w = workloads.Workload("flush", B=2, L=500, d=1024, V=65600, n_t=10, adv="normal", group=2,
                           targets="uniform", data_seed=2500, philox_seed=0xB6B70001)
    plan = b.bgpo_workspace_plan(b.Problem(2, 500, 1024, 65600, 10, ws_budget=budget_mib << 20))
    assert (plan["mode"], plan["samples_per_unit"], plan["dw_batch"]) == ("stored", 1, budget_mib // 225)
    x = workloads.generate(w)
    outs = []
    for ranges in ([(0, 10)], [(j, 1) for j in range(10)]):
        r = Runner(w, x, ws_budget=budget_mib << 20)
        for j0, n in ranges:
            r.bwd(j_begin=j0, j_count=n)
        outs.append(r.out())
    one, many = outs
    rows = one["nm"].sum(0)
    fits = [(int(a) + 63) // 64 * 64 + (int(c) + 255) // 256 * 256 <= 1024 for a, c in zip(rows, rows[1:])]
    assert any(fits) and not all(fits)
    for k in ("ell", "g", "nm", "dX"):
        assert np.array_equal(one[k], many[k]), k
    assert rel_maxnorm(one["dW"], many["dW"]) <= 1e-5


@pytest.mark.parametrize("B,L,d,V,n_t,budget_mib,plan", [
    (2, 500, 1024, 65600, 22, 640, (3, 1)),      # units of three samples, the last of one
    (2, 500, 1024, 65600, 22, 1040, (3, 2)),
    (1, 65600, 2048, 33024, 6, 12500, (2, 1)),   # of two, masks in several passes over the GPU
], ids=["units of 3", "units of 3, two at least", "multi-block masks"])
def test_dw_batches_of_units_of_several_samples(B, L, d, V, n_t, budget_mib, plan):
    """As above with several samples per unit: some units join the batch of the
    one before them and some do not, as their rows decide.  The whole range in
    one call against one call per unit: dX bit for bit, dW up to the order of
    fp32 sums (1e-5)."""
    b = lib()
    budget = budget_mib << 20
    w = workloads.Workload("flush", B=B, L=L, d=d, V=V, n_t=n_t, adv="normal", group=B, targets="uniform",
                           data_seed=2600, philox_seed=0xB6B80001)
    p = b.bgpo_workspace_plan(b.Problem(B, L, d, V, n_t, ws_budget=budget))
    G = p["samples_per_unit"]
    assert (p["mode"], G, p["dw_batch"]) == ("stored", *plan)
    x = workloads.generate(w)
    outs = []
    for ranges in ([(0, n_t)], [(j, min(G, n_t - j)) for j in range(0, n_t, G)]):
        r = Runner(w, x, ws_budget=budget)
        for j0, n in ranges:
            r.bwd(j_begin=j0, j_count=n)
        outs.append(r.out())
        del r
    one, many = outs
    per_sample = one["nm"].sum(0)
    rows = [int(per_sample[j:j + G].sum()) for j in range(0, n_t, G)]
    cap = plan[1] * G * ((B * L + 255) // 256 * 256)
    end, joined = 0, []
    for n in rows:                       # the column after the batch's last unit
        joined.append(end > 0 and end + (n + 255) // 256 * 256 <= cap)
        end = (end if joined[-1] else 0) + (n + 63) // 64 * 64
    assert any(joined) and not all(joined[1:])
    for k in ("ell", "g", "nm", "dX"):
        assert np.array_equal(one[k], many[k]), k
    assert rel_maxnorm(one["dW"], many["dW"]) <= 1e-5
    assert np.abs(one["dW"]).max() > 0 and one["flags"] == 0


def test_binding_passes_the_current_stream(monkeypatch):
    """The handle that the binding passes is the current stream's, on the default
    stream and inside a stream context, with and without torch's unlisted
    accessor; a stream that is named goes as it is."""
    b = lib()
    side = torch.cuda.Stream()
    for raw in (b._raw_stream, None):
        monkeypatch.setattr(b, "_raw_stream", raw)
        assert b._stream(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert b._stream(None) == side.cuda_stream != 0
        assert b._stream(side) == side.cuda_stream
