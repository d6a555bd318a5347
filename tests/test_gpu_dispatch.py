"""GPU test of the kernel chosen for open tiles: on both sides of the lines where
the step kernel measured faster than the kernel of all bits and drawn subsets
(flavours 6, 7) or the window kernel (5)."""
import numpy as np
import pytest

from paper_2210_10513_amd import binding, inputs
from paper_2210_10513_amd.binding import Sampler

from test_gpu_full import _pair, _problem, _state

pytestmark = pytest.mark.gpu


def _Q(kind, N):
    if kind == "f32":
        A = np.random.default_rng(N).standard_normal((N, N), dtype=np.float32) / np.float32(np.sqrt(N))
        return np.triu(A) + np.triu(A, 1).T
    return inputs.symmetric_int(N, -100, 100, np.int16, seed=N, density=0.5)


def _classes(s):
    binding.pns_profile(s.ctx)
    s.run(3)
    return binding.pns_profile_read(s.ctx)


@pytest.mark.parametrize("mode,kind,N,n,chains,log,flavours", [
    ("unbiased_rand", "f32", 200, 2, 4096, False, (2,)),      # one group: smallest sets of a full chip
    ("unbiased_rand", "f32", 200, 2, 1000, False, (7,)),
    ("unbiased_rand", "f32", 400, 64, 300, False, (2,)),      # two waves either way
    ("unbiased_rand", "f32", 400, 64, 600, False, (7,)),
    ("unbiased_rand", "f32", 1500, 4, 64, False, (2,)),       # few members to the tile's bits
    ("unbiased_rand", "f32", 1500, 16, 64, False, (7,)),
    ("unbiased_rand", "f32", 1500, 200, 600, False, (2,)),    # as many rounds of the chip
    ("unbiased_rand", "f32", 1500, 200, 1000, False, (7,)),
    ("unbiased_rand", "f32", 1500, 200, 1536, False, (2,)),
    ("unbiased_rand", "f32", 3500, 16, 64, False, (2,)),
    ("unbiased_rand", "f32", 3500, 200, 64, False, (7,)),
    ("unbiased_rand", "i16", 900, 64, 300, False, (2,)),
    ("unbiased_rand", "i16", 900, 64, 200, False, (7,)),
    ("unbiased_rand", "i16", 1500, 64, 300, True, (2,)),      # outputs of every step
    ("unbiased_rand", "i16", 1500, 64, 300, False, (7,)),
    ("basic", "f32", 1030, 2, 600, False, (2,)),
    ("basic", "f32", 1030, 8, 600, False, (7,)),
    ("rf", "i16", 900, 0, 600, False, (0,)),
    ("rf", "i16", 900, 0, 1024, False, (6,)),
    ("unbiased_sys", "i16", 150, 16, 4096, False, (1, 3, 4)),  # more chains than the chip holds of the window kernel's
    ("unbiased_sys", "i16", 150, 16, 2048, False, (5,)),
])
def test_kernel_of_an_open_tile(mode, kind, N, n, chains, log, flavours):
    s = Sampler(_Q(kind, N), 0.01, n, mode, num_chains=chains, log_capacity=4 if log else 0)
    (c,) = _classes(s)
    assert c["flavour"] in flavours
    s.close()


# (the classes whose exact-time runs take the step kernel, and one beside each)
@pytest.mark.parametrize("kind,N,n,chains", [("i64", 200, 24, 3), ("i64", 700, 64, 3), ("i64", 1000, 8, 300),
                                             ("f32", 700, 4, 300), ("f32", 900, 4, 600), ("f32", 1500, 8, 600),
                                             ("f32", 1500, 40, 600), ("f32", 6200, 4, 2), ("i16", 900, 4, 600)])
def test_exact_time_runs_of_drawn_subsets(kind, N, n, chains):
    """Between sampling runs, where the two kernels take turns: the step kernel's
    records and states."""
    Q, beta, layout = _problem(kind, N)
    _pair(Q, beta, n, "basic", layout, chains, lambda s: _state(s.run(20).run_original(300).run(5)))


def test_exact_time_runs_of_int64_fields():
    Q, beta, layout = _problem("i64", 1100)
    _pair(Q, beta, 0, "rf", layout, 600, lambda s: _state(s.run(10).run_original(40).run(5)))


@pytest.mark.parametrize("kind,N", [("i16", 13400), ("i64", 13400), ("i16", 16384)])
def test_widest_drawn_subsets(kind, N):
    """The table of occurrences past 64 KB of LDS (tables and members with it)."""
    Q, beta, layout = _problem(kind, N)
    _pair(Q, beta, 700, "basic", layout, 2, lambda s: _state(s.run(20), log=True), log_capacity=20)
    if kind == "i16":
        _pair(Q, beta, 90, "unbiased_rand", layout, 2, lambda s: _state(s.run(20), log=True), log_capacity=20, L0=30)
