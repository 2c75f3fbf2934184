"""The two-pass kernels with 8-wave items at the launch sizes where the number
of workgroups per CU changes (24 and 48 items per CU, ranges 16 n polynomials
apart) and around one item per CU: both directions equal the explicit three
workgroups per CU bit for bit, and a sampled polynomial equals the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_14191_amd import tfhe
    tfhe.load()
    return tfhe


# (256 CUs; 8 items per polynomial at N = 2^16, 4 at 2^15)
@pytest.mark.parametrize("log_n,limbs,batch", [(16, 3, 1), (16, 3, 11), (16, 7, 13), (16, 6, 128), (16, 1, 769),
                                               (16, 3, 512), (16, 5, 410), (15, 6, 256), (15, 29, 53)])
def test_grid_of_wide_passes(tf, log_n, limbs, batch):
    qs = oracle.ntt_primes(limbs - 1, 31, 1 << 17) + oracle.ntt_primes(1, 30, 1 << 17)
    plan = tf.NttPlan(log_n, qs, algo="mfma")
    plan.set_param("fs_passes", 2)
    gen = torch.Generator(device="cuda").manual_seed(batch)
    x = torch.stack([torch.randint(0, q, (batch, 1 << log_n), dtype=torch.int64, device="cuda", generator=gen)
                     .to(torch.int32) for q in qs])
    l, b = limbs - 1, batch - 1
    one = x[l:l + 1, b:b + 1].cpu().numpy().view(np.uint32)
    y = plan.fwd(x, algo="mfma")
    assert np.array_equal(y[l:l + 1, b:b + 1].cpu().numpy().view(np.uint32),
                          oracle.ntt_fwd(one, qs[l:], plan.psi[l:]))
    z = plan.inv(y, algo="mfma")
    assert torch.equal(z, x)
    plan.set_param("fs_wg_per_cu", 3)
    assert torch.equal(y, plan.fwd(x, algo="mfma"))
    assert torch.equal(z, plan.inv(y, algo="mfma"))
