"""The key-switching inner product fused with the transforms' second pass, with
resident and with streamed keys: equal to the separate inner-product kernel bit
for bit where the choice between them changes (few and many batch elements,
one to four digits, ranges that end inside a key block, mixed levels)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_14191_amd import tfhe
    tfhe.load()
    return tfhe


def residues(moduli, shape, gen):
    return torch.stack([torch.randint(0, q, shape, dtype=torch.int64, device="cuda", generator=gen)
                        for q in moduli]).to(torch.int32)


def pairs(moduli, shape, gen):
    return torch.stack([residues(moduli, shape, gen) for _ in range(2)])


@pytest.mark.parametrize("log_n,L,K,dnum,level,batch", [
    (12, 6, 2, 3, 6, 40),    # no block pairs: streamed
    (13, 6, 2, 3, 6, 63),    # fewer items than the resident path takes
    (13, 6, 2, 3, 6, 67),    # resident
    (13, 6, 2, 3, 3, 211),   # two digits, one of them partial
    (14, 8, 2, 4, 8, 29),    # four digits: streamed
    (14, 6, 6, 1, 6, 23),    # one digit
    (15, 6, 2, 3, 6, 3),     # too few elements per key: streamed
    (16, 4, 2, 2, 4, 11),
])
def test_fused_inner_product_equals_separate(tf, log_n, L, K, dnum, level, batch):
    ctx = tf.CkksContext(log_n, L, K, dnum)
    gen = torch.Generator(device="cuda").manual_seed(log_n + batch)
    q = ctx.moduli[:level]
    a, b = pairs(q, (batch, 1 << log_n), gen), pairs(q, (batch, 1 << log_n), gen)
    key = torch.stack([pairs(ctx.moduli, (1 << log_n,), gen) for _ in range(dnum)])
    out = ctx.hmult(a, b, key, level)
    ctx.plan.set_param("ks_inner", 2)
    assert torch.equal(out, ctx.hmult(a, b, key, level))


def test_resident_keys_over_mixed_levels(tf):
    """Groups of the same key blocks with one, two and three digits."""
    log_n, L = 15, 6
    ctx = tf.CkksContext(log_n, L, 2, 3)
    gen = torch.Generator(device="cuda").manual_seed(3)
    levels = [1] * 9 + [6] * 9 + [3] * 8
    a = [pairs(ctx.moduli[:lv], (1 << log_n,), gen) for lv in levels]
    b = [pairs(ctx.moduli[:lv], (1 << log_n,), gen) for lv in levels]
    key = torch.stack([pairs(ctx.moduli, (1 << log_n,), gen) for _ in range(3)])
    outs = ctx.hmult_levels(a, b, key)
    ctx.plan.set_param("ks_inner", 2)
    for o, r in zip(outs, ctx.hmult_levels(a, b, key)):
        assert torch.equal(o, r)
