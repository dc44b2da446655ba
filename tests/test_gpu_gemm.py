"""The GEMM core in every form that the library launches, on both tile sizes and
two GEMMs in one launch, against exact products of the bf16 operands.

Bar: an fp32 sum of K products differs from the exact one by a few sqrt(K)
roundings of its largest partial sums (2e-5 sqrt(K) of the largest result, as
for the hooks of test_gpu_parity.py).
"""
import pytest
import torch

from gpu_util import lib

pytestmark = pytest.mark.gpu

ROW, MSLAB, KSLAB = 0, 1, 2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib()


def _slab(X):
    """[R, K] -> [K/64, R, 64]."""
    return X.reshape(X.shape[0], -1, 64).permute(1, 0, 2).contiguous()


def _lay(A, layout):
    if layout == ROW:
        return A.contiguous()
    return _slab(A) if layout == KSLAB else A.reshape(-1, 64, A.shape[1]).permute(0, 2, 1).contiguous()


class _Operands:
    """A [M, K], B [N, K] in bf16, C [n_split, N, M] from nonzero values, and what
    C holds after one stored or accumulated product."""

    def __init__(self, M, N, K, n_split, layout, accumulate, seed):
        g = torch.Generator().manual_seed(seed)
        A = torch.randn(M, K, generator=g).to(torch.bfloat16)
        B = torch.randn(N, K, generator=g).to(torch.bfloat16)
        C = torch.randn(n_split, N, M, generator=g)
        ks = ((K + n_split - 1) // n_split + 63) // 64 * 64
        prod = torch.stack([B[:, s * ks:(s + 1) * ks].double() @ A[:, s * ks:(s + 1) * ks].double().T
                            for s in range(n_split)])
        self.want = prod + C.double() if accumulate else prod
        self.bar = 2e-5 * K ** 0.5 * prod.abs().max().item() + 1e-4
        self.empty = [s for s in range(n_split) if s * ks >= K]
        self.A, self.B, self.C = _lay(A, layout).cuda(), _slab(B).cuda(), C.cuda()

    def check(self):
        got = self.C.cpu().double()
        err = (got - self.want).abs().max().item()
        assert err <= self.bar, err
        for s in self.empty:      # zeros, or the values that were there
            assert torch.equal(got[s], self.want[s])


FORMS = [(ROW, False), (KSLAB, False), (ROW, True), (KSLAB, True), (MSLAB, True)]


@pytest.mark.parametrize("tile", [128, 256])
@pytest.mark.parametrize("layout,accumulate", FORMS, ids=["row", "kslab", "row+", "kslab+", "mslab+"])
@pytest.mark.parametrize("M,N,K,n_split", [
    (64, 1, 64, 1),          # one row, fewer slabs than ring stages
    (128, 128, 128, 1),      # one whole 128-wide tile, two slabs
    (192, 130, 192, 1),      # ragged in both, three slabs
    (320, 257, 256, 1),      # as many slabs as stages
    (512, 256, 320, 3),      # whole tiles, split, the last slice shorter
    (256, 384, 64, 4),       # empty slices
    (4288, 576, 128, 1),     # more tiles than one band
])
def test_forms_match_exact_products(tile, layout, accumulate, M, N, K, n_split):
    o = _Operands(M, N, K, n_split, layout, accumulate, M + 3 * N + 5 * K)
    lib().bgpo_test_gemm(o.A, layout, o.B, o.C, accumulate, tile)
    torch.cuda.synchronize()
    o.check()


@pytest.mark.parametrize("layout", [ROW, KSLAB])
@pytest.mark.parametrize("n_first", [8, 64, 248])
@pytest.mark.parametrize("first,second", [
    ((64, 1, 64, 1), (64, 64, 64)),               # a tile each: most workgroups find none
    ((576, 300, 4288, 8), (4288, 576, 320)),      # several tiles per workgroup of the smaller side
    ((200, 129, 64, 4), (1024, 128, 192)),        # empty slices beside whole tiles
])
def test_two_gemms_in_one_launch(layout, n_first, first, second):
    """Each half alone walks its own tiles, whatever the split of the grid."""
    p = _Operands(*first, layout, False, 7)
    q = _Operands(*second, 1, MSLAB, True, 8)
    lib().bgpo_test_gemm_pair(p.A, layout, p.B, p.C, q.A, q.B, q.C, n_first)
    torch.cuda.synchronize()
    p.check()
    q.check()
