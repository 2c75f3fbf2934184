"""The FrobeniusMap by whole polynomials (and, below its smallest launch, element
by element) equals the index map, for plain arrays, a ciphertext's two
components with one Galois element per batch element, and mixed levels.  The
multi-rotation and mixed-level launches are covered through their results
against single rotations.  Exact."""
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


@pytest.mark.parametrize("batch", [1, 16, 32, 33])
@pytest.mark.parametrize("log_n", [10, 12, 13, 14, 15, 16])
def test_map_matches_the_index_map(tf, log_n, batch):
    n = 1 << log_n
    plan = tf.NttPlan(log_n, oracle.ntt_primes(2, 30, 1 << 17))
    gen = torch.Generator(device="cuda").manual_seed(log_n)
    x = torch.randint(0, 1 << 29, (2, batch, n), dtype=torch.int32, device="cuda", generator=gen)
    j = torch.arange(n, dtype=torch.int64, device="cuda")
    for g in (1, 5, pow(5, 37, 2 * n), 2 * n - 1):
        src = ((2 * j + 1) * g % (2 * n) - 1) // 2
        assert torch.equal(plan.frobenius(x, g), x[:, :, src]), g


@pytest.mark.parametrize("log_n,level,batch", [(12, 4, 9), (13, 5, 7), (14, 4, 8), (15, 4, 5), (16, 4, 5)])
def test_multi_rotation_equals_single_rotations(tf, log_n, level, batch):
    """One launch for all elements (by polynomial), of one level and of two,
    against one rotation per element (few polynomials: element by element)."""
    ctx = tf.CkksContext(log_n, 6, 3, 2)
    n = 1 << log_n
    gen = torch.Generator(device="cuda").manual_seed(7)

    def residues(moduli, shape):
        return torch.stack([torch.randint(0, q, shape, dtype=torch.int64, device="cuda", generator=gen)
                            for q in moduli]).to(torch.int32)

    q = ctx.moduli[:level]
    a = torch.stack([residues(q, (batch, n)) for _ in range(2)])
    gs = [pow(5, 3 + 2 * b, 2 * n) for b in range(batch)]
    keys = [torch.stack([torch.stack([residues(ctx.moduli, (n,)) for _ in range(2)]) for _ in range(2)])
            for _ in range(batch)]
    out = ctx.rotate_multi(a, keys, gs, level)
    levels = [level - b % 2 for b in range(batch)]
    mixed = ctx.rotate_levels([a[:, :lv, b].contiguous() for b, lv in enumerate(levels)], keys, gs)
    for b, lv in enumerate(levels):
        one = ctx.rotate(a[:, :, b:b + 1].contiguous(), keys[b], gs[b], level)
        assert torch.equal(out[:, :, b:b + 1], one), b
        one = ctx.rotate(a[:, :lv, b:b + 1].contiguous(), keys[b], gs[b], lv)
        assert torch.equal(mixed[b], one[:, :, 0]), b
