"""GPU parity of the basis conversions fused with the transforms' first pass
(and of RESCALE's broadcast first pass) at the shapes where they can go wrong:
every N1 of the four-step range, up to four and up to eight inputs, partial
digits, one special prime, targets that do not divide into equal chunks, and
batches whose chunks do not fill groups of eight workgroups.  Exact: every
quantity is an integer."""
import numpy as np
import pytest

import oracle
from oracle import ckks
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


def random_ct(pr, level, batch, seed):
    return np.stack([inputs.uniform_residues(seed + c, pr.mods(range(level)), (batch, pr.n)) for c in range(2)])


@pytest.mark.parametrize("log_n,L,K,dnum,level,batch", [
    (12, 8, 4, 2, 7, 9),     # N1 = 16: four inputs, a digit of three
    (12, 8, 1, 1, 8, 2),     # eight inputs up, one down
    (13, 24, 8, 3, 18, 3),   # N1 = 32: a digit of two limbs
    (14, 12, 2, 6, 11, 5),   # N1 = 64: two inputs, a digit of one
    (15, 16, 8, 2, 13, 1),   # N1 = 128: quad-tiled inputs
    (16, 16, 5, 2, 9, 3),    # N1 = 256: five special primes, a digit of one limb
])
def test_key_switch_conversions_match_oracle(tf, log_n, L, K, dnum, level, batch):
    pr = ckks.Params(1 << log_n, L=L, K=K, dnum=dnum)
    key = np.stack([np.stack([inputs.uniform_residues(7 + 2 * j + c, pr.moduli, (pr.n,)) for c in range(2)])
                    for j in range(dnum)])
    a, b = random_ct(pr, level, batch, 20), random_ct(pr, level, batch, 30)
    ctx = tf.CkksContext(log_n, L, K, dnum, moduli=pr.moduli)
    got = to_host(ctx.hmult(to_dev(a), to_dev(b), to_dev(key), level))
    assert np.array_equal(got, ckks.hmult(pr, a, b, key, level))
    # natural-order inputs at every N (the one-pass inverse transforms), and
    # the separate conversion kernels
    for name, value in (("fs_passes", 1 if log_n < 16 else 2), ("ks_inner", 2)):
        ctx.plan.set_param(name, value)
        assert np.array_equal(to_host(ctx.hmult(to_dev(a), to_dev(b), to_dev(key), level)), got), name


@pytest.mark.parametrize("log_n,passes", [(12, 0), (13, 0), (14, 0), (15, 0), (15, 1), (16, 0)])
@pytest.mark.parametrize("level,batch", [(2, 1), (11, 7)])
def test_rescale_broadcast_matches_oracle(tf, log_n, passes, level, batch):
    pr = ckks.Params(1 << log_n, L=11, K=1, dnum=11)
    ct = random_ct(pr, level, batch, 40)
    ct[:, level - 1, 0, :3] = [[0, pr.q[level - 1] - 1, 1]]  # the top limb's extremes
    ctx = tf.CkksContext(log_n, 11, 1, 11, moduli=pr.moduli)
    ctx.plan.set_param("fs_passes", passes)
    assert np.array_equal(to_host(ctx.rescale(to_dev(ct), level)), ckks.rescale(pr, ct, level))
