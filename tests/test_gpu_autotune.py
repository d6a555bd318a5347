"""GPU test of the autotuner: a context made from its result runs the kernel that
was timed, and every kernel that could run a problem is tried."""
import numpy as np
import pytest

from paper_2210_10513_amd import binding as b
from paper_2210_10513_amd.binding import Sampler

from test_gpu_full import _problem

pytestmark = pytest.mark.gpu

CHAINS = 3072  # (of the trials too: those of one context, from 3072 to 4096)


# (int64 fields up to 1024 bits, random sets of them and of floats of 513 to 1024
# bits run the step kernel on the tile: 64x4, 128x2, 256x1 and the next larger)
@pytest.mark.parametrize("mode,kind,N,n,trials", [
    ("rf", "i16", 700, 0, 1), ("rf", "f32", 300, 0, 1), ("rf", "i64", 600, 0, 3), ("basic", "i32", 1500, 40, 1),
    ("unbiased_rand", "f32", 700, 40, 3), ("unbiased_rand", "f32", 3000, 40, 1), ("unbiased_rand", "i64", 700, 40, 3),
    ("unbiased_sys", "i16", 1000, 100, 1), ("unbiased_sys", "f32", 900, 60, 3)])
def test_a_context_made_from_the_result_runs_the_timed_kernel(mode, kind, N, n, trials):
    Q, beta, layout = _problem(kind, N)
    o = b.pns_opts_default()
    o.dtype = {"i16": b.PNS_I16, "f32": b.PNS_F32}.get(kind, b.PNS_I32)
    o.layout = b.PNS_UPPER if layout == "upper" else b.PNS_SYMMETRIC
    o.num_chains = CHAINS
    t = b.pns_autotune(Q, N, beta, n, b.MODES[mode], o, 64)
    assert t.trials >= trials
    s = Sampler(Q, beta, t.subset_size, mode, num_chains=CHAINS, layout=layout, block=t.block, groups=t.groups)
    rates = []
    s.run(64)
    for _ in range(3):
        b.pns_profile(s.ctx)
        s.run(64)
        (c,) = b.pns_profile_read(s.ctx)
        rates.append(c["records"] / (c["kernel_ms"] * 1e-3))
    s.close()
    if t.block == 0:
        assert t.groups == 0 and c["flavour"] in (6, 7)
    else:
        assert (c["block"], c["groups"]) == (t.block, t.groups) and c["flavour"] < 6
    # (the same launches: the other kernel would take 1.5 to 3 times as long)
    assert 0.7 * t.records_per_s < max(rates)


def test_created_with_the_autotuner():
    Q, beta, layout = _problem("i16", 700)
    s = Sampler(Q, beta, 0, "basic", num_chains=64, layout=layout, autotune=True).run(20)
    assert 16 <= b.pns_problem_info_get(s.ctx, 0).subset_size <= 350
    assert (s.stats()["steps"] == 20).all()
    s.close()
