"""RESCALE's broadcast first pass on either side of the launch size up to which
it runs in workgroups of four waves (two of them per CU: 256 polynomials at
N = 2^13, 128 at 2^14 with 256 CUs), exactly equal to the oracle."""
import numpy as np
import pytest

from oracle import ckks
from paper_2212_14191_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("log_n,level,batch", [(13, 3, 64), (13, 3, 65), (14, 2, 64), (14, 2, 65), (14, 5, 1)])
def test_rescale_matches_oracle(log_n, level, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_14191_amd import tfhe
    pr = ckks.Params(1 << log_n, L=5, K=1, dnum=5)
    ct = np.stack([inputs.uniform_residues(60 + c, pr.mods(range(level)), (batch, pr.n)) for c in range(2)])
    ctx = tfhe.CkksContext(log_n, 5, 1, 5, moduli=pr.moduli)
    got = ctx.rescale(torch.from_numpy(ct.view(np.int32)).cuda(), level)
    assert np.array_equal(got.cpu().numpy().view(np.uint32), ckks.rescale(pr, ct, level))
