"""Float32 kernels alone against float64 references, at the edges of their tiles."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2512_20920_amd as R
    from helpers import relerr


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 1), (1, 0)])
# one element, tails in every dimension around 32 and the 32-wide chunks of k, rows that are not 16-byte aligned
# (odd leading dimensions), no k at all, and enough tiles for the larger tile shape
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 65), (64, 96, 64), (61, 130, 2048), (7, 200, 31), (40, 40, 0),
                                   (1030, 1040, 70), (1024, 1056, 33),
                                   # whole groups of four throughout (straight into LDS without the odd padding): less than a
                                   # piece, one past it, fewer pieces than waves, several per wave, ragged tiles
                                   (4, 8, 4), (36, 44, 68), (64, 32, 36), (132, 260, 516), (400, 512, 1024)])
def test_f32_gemm(M, N, K, a_trans, b_trans):
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, B = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (K, N)))
    a, b = (A.T if a_trans else A), (B if b_trans else B.T)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    for pad in (0 if K else 4, 3):
        ap, bp = (np.pad(x, ((0, 1), (0, pad))) for x in (a, b))
        c = torch.full((M, N + pad), float("nan"), dtype=torch.float32, device="cuda")
        R.revffn_op_gemm(0, 0, _dev(ap), _dev(bp), c, M, N, K, ap.shape[1], bp.shape[1], N + pad, a_trans, b_trans)
        torch.cuda.synchronize()
        got = c.cpu().numpy()
        assert np.isnan(got[:, N:]).all()
        if K:
            assert relerr(got[:, :N].astype(np.float64), ref) < 2e-6
        else:
            assert (got[:, :N] == 0).all()
