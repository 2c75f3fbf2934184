"""A tuned context leaves the number of passes to the library's rule, whichever
number the table holds for the shape it was measured at."""
import pytest

from paper_2212_14191_amd import autotune


class Plan:
    log_n = 15

    def __init__(self):
        self.params = {}

    def set_param(self, name, value):
        self.params[name] = value


class Ctx:
    log_n = 15

    def __init__(self):
        self.plan = Plan()


@pytest.mark.parametrize("passes", [0, 1, 2])
def test_context_takes_the_rule(passes):
    t = autotune.TuneTable()
    t.put(autotune.ntt_key(15, 24, 64), {"algo": "mfma", "fs_passes": passes, "fs_wide": 2, "fs_ring": 2})
    ctx = Ctx()
    got = autotune.apply_ckks(ctx, t)
    assert got["ntt"]["fs_passes"] == 0 and ctx.plan.params["fs_passes"] == 0
    assert ctx.plan.params["fs_wide"] == 2 and ctx.plan.params["fs_ring"] == 2
