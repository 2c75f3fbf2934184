"""The default choice between the one-pass and the two-pass four-step kernels
at the launch sizes where it changes: both directions equal two passes bit
for bit, and sampled polynomials equal the oracle."""
import numpy as np
import pytest

import oracle
from paper_2212_14191_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_14191_amd import tfhe
    tfhe.load()
    return tfhe


def to_dev(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int32)).cuda()


def to_host(t):
    return t.cpu().numpy().view(np.uint32)


# 256 CUs: below and above half of them, just all of them, one round and a bit
@pytest.mark.parametrize("batch", [1, 42, 43, 85, 86, 128])
@pytest.mark.parametrize("log_n", [12, 13, 14, 15])
def test_default_passes_at_the_edges_of_the_rule(tf, log_n, batch):
    qs = oracle.ntt_primes(2, 31, 1 << 17) + oracle.ntt_primes(1, 30, 1 << 17)
    plan = tf.NttPlan(log_n, qs, algo="mfma")
    host = inputs.uniform_residues(500 + log_n + batch, qs, (batch, 1 << log_n))
    x = to_dev(host)
    f0, i0 = plan.fwd(x, algo="mfma"), plan.inv(x, algo="mfma")
    plan.set_param("fs_passes", 2)
    assert torch.equal(f0, plan.fwd(x, algo="mfma"))
    assert torch.equal(i0, plan.inv(x, algo="mfma"))
    l, b = batch % 3, batch - 1
    one = (slice(l, l + 1), slice(b, b + 1))
    assert np.array_equal(to_host(f0)[one], oracle.ntt_fwd(host[one], qs[l:l + 1], plan.psi[l:l + 1]))
    assert np.array_equal(to_host(i0)[one], oracle.ntt_inv(host[one], qs[l:l + 1], plan.psi[l:l + 1]))
