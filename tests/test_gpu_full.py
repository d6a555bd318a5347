"""GPU tests of the kernels that run problems whose tile the caller left open
(all bits, drawn subsets, and systematic windows of integers): records, states,
outputs and counters equal the step kernel's (an explicit tile) bit for bit at
the edges of the tile rule, for every field type, mode, launch form and kind of
run."""
import numpy as np
import pytest

from paper_2210_10513_amd import inputs
from paper_2210_10513_amd.binding import BatchSampler, Sampler

pytestmark = pytest.mark.gpu

TILES = {256: (64, 1), 512: (128, 1), 1024: (256, 1), 2048: (256, 2), 4096: (256, 4), 8192: (512, 4), 16384: (1024, 4)}


def _problem(kind, N, seed=0):
    """(Q, beta, layout); i64: int32 entries whose field bound needs 64 bits."""
    rng = np.random.default_rng(N + seed)
    if kind == "f32":
        A = (rng.standard_normal((N, N)) / np.sqrt(N)).astype(np.float32)
        return np.triu(A) + np.triu(A, 1).T, 1.0, "symmetric"
    if kind == "i64":
        hi = 2**29
        Q = np.triu(rng.integers(-hi, hi + 1, (N, N), dtype=np.int32))
        return Q, 4.0 / (hi * np.sqrt(N)), "upper"
    Q = inputs.symmetric_int(N, -100, 100, np.int16 if kind == "i16" else np.int32, seed=N + seed, density=0.5)
    return Q, 0.01 * np.sqrt(2048.0 / N), "symmetric"


def _step_tile(N):
    return TILES[min(t for t in TILES if t >= N)]


def _same(a, b):
    assert set(a) == set(b)
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=a[k].dtype.kind == "f"), k


def _state(s, log=False):
    out = {f"cur_{k}": v for k, v in s.read_current().items()}
    out.update({f"stat_{k}": v for k, v in s.stats().items()})
    for k, v in zip(("s", "m", "e"), s.read()):
        out[f"rec_{k}"] = v
    if log:
        out.update({f"log_{k}": v for k, v in s.read_log().items()})
    return out


def _pair(Q, beta, n, mode, layout, chains, fn, **kw):
    out = []
    for tile in ((0, 0), _step_tile(Q.shape[0])):
        s = Sampler(Q, beta, n, mode, num_chains=chains, layout=layout, seed=11, block=tile[0], groups=tile[1], **kw)
        out.append(fn(s))
        s.close()
    _same(out[0], out[1])
    return out[0]


# (N, chains): both sides of each line of the tile rule and ragged sizes between
SIZES = [(1, 3), (5, 3), (256, 3), (257, 3), (511, 600), (513, 3), (513, 600), (768, 600), (769, 600), (1000, 3),
         (1025, 3), (1030, 600), (2049, 3), (3000, 2), (3073, 2), (3073, 600), (4097, 2), (6145, 2)]


@pytest.mark.parametrize("kind", ["i16", "i32", "i64", "f32"])
@pytest.mark.parametrize("N,chains", SIZES)
def test_records_equal_the_step_kernels(kind, N, chains):
    Q, beta, layout = _problem(kind, N)
    for mode, n in (("rf", 0), ("basic", max(1, N // 3)), ("basic", 1), ("unbiased_rand", max(1, N // 9))):
        _pair(Q, beta, n, mode, layout, chains, lambda s: _state(s.run(45), log=True), log_capacity=45, L0=30)


@pytest.mark.parametrize("kind", ["i16", "f32", "i64"])
@pytest.mark.parametrize("N", [8193, 12001])
def test_records_of_the_widest_tile(kind, N):
    Q, beta, layout = _problem(kind, N)
    for mode, n in (("rf", 0), ("basic", 999)):
        _pair(Q, beta, n, mode, layout, 2, lambda s: _state(s.run(25), log=True), log_capacity=25)


@pytest.mark.parametrize("kind", ["i16", "i64", "f32"])
@pytest.mark.parametrize("N,n", [(200, 24), (700, 64), (1500, 100)])
def test_kinds_of_run_equal(kind, N, n):
    """Exact-time, optimization and resumed runs, snapshots, launch forms."""
    Q, beta, layout = _problem(kind, N)

    def runs(s):
        out = {}
        if s.mode in (0, 1):  # (runs of original samples: Rejection-Free and Basic PNS)
            s.run_original(900)
        else:
            s.run(30)
        out.update({f"a_{k}": v for k, v in _state(s).items()})
        s.optimize(40, 0.7)
        out["best_s"], out["best_e"] = s.read_best()
        s.adopt_best().run(33)
        out.update({f"b_{k}": v for k, v in _state(s).items()})
        buf = s.save()
        s.run(21)
        out.update({f"c_{k}": v for k, v in _state(s).items()})
        s.load(buf).run(21)
        for k, v in _state(s).items():
            if not k.startswith("stat_"):
                assert np.array_equal(out[f"c_{k}"], v, equal_nan=v.dtype.kind == "f"), k
        return out

    for mode, m in (("rf", 0), ("basic", n), ("unbiased_rand", n)):
        plain = _pair(Q, beta, m, mode, layout, 3, runs, launch="plain", chunk=7)
        graph = _pair(Q, beta, m, mode, layout, 3, runs, launch="graph", chunk=7)
        _same(plain, graph)

        def snaps(s):
            s.run(60)
            x, w, e, cnt = s.read_snapshots()
            return {"x": x, "w": w, "e": e, "cnt": np.asarray(cnt), "rb": s.rb_weights()["snap"]}

        _pair(Q, beta, m, mode, layout, 3, snaps, snapshot_every=4, snapshot_capacity=15)


@pytest.mark.parametrize("kind,scale", [("i16", 40.0), ("i32", 4000.0), ("f32", 3000.0), ("i64", 1e4)])
def test_rescaled_and_overflowing_weights_equal(kind, scale):
    """Large beta: weights past the tables, sums that vanish and are rescaled,
    saturated multiplicities."""
    for N, n in ((13, 2), (300, 5), (900, 40)):
        Q, beta, layout = _problem(kind, N, seed=3)
        for mode, m in (("rf", 0), ("basic", n), ("unbiased_rand", n)):
            _pair(Q, beta * scale, m, mode, layout, 4, lambda s: _state(s.run(80), log=True), log_capacity=80, L0=20)


@pytest.mark.parametrize("N,n", [(30, 7), (900, 60), (3000, 200)])
def test_more_draws_than_the_table_of_occurrences_numbers(N, n):
    """One launch of more than 4095 draws: the keys' draw numbers run out and
    the table is cleared."""
    Q, beta, layout = _problem("i16", N)
    _pair(Q, beta, n, "basic", layout, 2, lambda s: _state(s.run(9000)))


def test_histogram_equal():
    for kind in ("i16", "f32"):
        Q, beta, layout = _problem(kind, 12)
        for mode, m in (("rf", 0), ("basic", 5), ("unbiased_rand", 5)):
            def hist(s):
                s.run(500)
                w, v = s.read_hist()
                return {"w": w, "v": v, "rb": s.rb_weights()["hist"]}
            got = _pair(Q, beta, m, mode, layout, 1, hist, hist=True)
            assert got["v"].sum() > 0


# (both sides of the chain counts where the window kernel takes over, its one-
# and two-wave tiles, workgroups that are shared by two and four chains)
@pytest.mark.parametrize("kind", ["i16", "i32"])
@pytest.mark.parametrize("N,n,chains", [(200, 30, 3), (512, 100, 300), (700, 100, 1024), (700, 100, 1026),
                                        (1500, 128, 770), (2050, 200, 515), (4000, 256, 513), (5000, 300, 769),
                                        (7000, 256, 769), (9000, 256, 2)])
def test_windows_equal_the_step_kernels(kind, N, n, chains):
    Q, beta, layout = _problem(kind, N)
    got = _pair(Q, beta, n, "unbiased_sys", layout, chains, lambda s: _state(s.run(40)), L0=30)
    assert (got["stat_anomalies"] == 0).all()


@pytest.mark.parametrize("N,tile", [(3000, (64, 16)), (5000, (64, 24)), (7000, (128, 16)), (9000, (128, 24)),
                                    (16000, (256, 16))])
def test_int32_rows_of_the_wide_window_tiles(N, tile):
    """The row of a flip in one piece (16 groups) or two (24), both signs."""
    Q, beta, layout = _problem("i32", N)
    out = []
    for block, groups in (tile, _step_tile(N)):
        s = Sampler(Q, beta, 250, "unbiased_sys", num_chains=2, layout=layout, seed=4, init="random", block=block,
                    groups=groups, log_capacity=120)
        out.append(_state(s.run(120), log=True))
        s.close()
    _same(out[0], out[1])


@pytest.mark.parametrize("mode,kind", [("rf", "i16"), ("basic", "f32"), ("unbiased_sys", "i32"), ("unbiased_rand", "i16")])
def test_batch_on_merged_tiles_equals_single_problems(mode, kind):
    """Problems of a batch that run on a larger problem's tile."""
    sizes, chains = (30, 200, 300, 600, 900, 1500, 2500, 5000), 3
    probs = []
    for i, N in enumerate(sizes):
        Q, beta, layout = _problem(kind, N)
        probs.append(dict(Q=Q, beta=beta, layout=layout, num_chains=chains, subset_size=0 if mode == "rf" else max(2, N // 10)))
    b = BatchSampler(probs, mode, seed=11, log_capacity=30)
    b.run(30)
    log, cur = b.read_log(), b.read_current()
    for i, (N, pr) in enumerate(zip(sizes, probs)):
        t = _step_tile(N)
        s = Sampler(pr["Q"], pr["beta"], pr["subset_size"], mode, num_chains=chains, layout=pr["layout"], seed=11,
                    chain_id_base=chains * i, block=t[0], groups=t[1], log_capacity=30).run(30)
        _same({k: v[i] for k, v in log.items()}, s.read_log())
        c = s.read_current()
        for k in ("x", "E", "h"):
            assert np.array_equal(cur[k][i], c[k]), (N, k)
        s.close()
    b.close()


@pytest.mark.parametrize("kind", ["i16", "f32"])
@pytest.mark.parametrize("N,chains", [(600, 257), (769, 257), (1000, 513), (1024, 1025)])
def test_exact_time_runs_equal(kind, N, chains):
    """Exact-time runs between sampling runs, where the two kernels take turns."""
    Q, beta, layout = _problem(kind, N)
    _pair(Q, beta, 0, "rf", layout, chains, lambda s: _state(s.run(20).run_original(70).run(5)))
