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
