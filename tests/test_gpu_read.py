"""GPU tests of the rows and arrays that the read calls return: states and
fields against the energies and products they belong to, on both sides of the
sizes where the rows are gathered on the device or sorted out on the host, in
one piece or several, aligned or not, to host and to device buffers."""
import numpy as np
import pytest
import torch

from paper_2210_10513_amd import binding, inputs
from paper_2210_10513_amd.binding import BatchSampler, Sampler

pytestmark = pytest.mark.gpu


def _energies(Q, x):
    x = x.astype(np.float64)
    return ((x @ Q.astype(np.float64)) * x).sum(1)


# 64 KB of states is the last size sorted out on the host, 32 MB the largest piece
@pytest.mark.parametrize("N,chains", [(5, 3), (64, 1024), (64, 1025), (1, 70000), (317, 300), (1008, 70), (1000, 40000),
                                      (16, 3000000)])
def test_rows_belong_to_their_energies(N, chains):
    Q = inputs.symmetric_int(N, -50, 50, np.int16, seed=N, density=0.7)
    s = Sampler(Q, 0.02, max(1, N // 2), "basic", num_chains=chains, seed=3, init="random").run(3)
    x, m, e = s.read()
    c = s.read_current()
    pick = np.unique(np.r_[0:min(chains, 50), chains // 2, max(0, chains - 50):chains])
    assert np.array_equal(_energies(Q, x[pick]), e[pick])
    assert np.array_equal(_energies(Q, c["x"][pick]), c["E"][pick])
    off = Q.astype(np.int64) - np.diag(np.diag(Q.astype(np.int64)))
    assert np.array_equal(c["x"][pick].astype(np.int64) @ off, c["h"][pick])
    assert (x != c["x"]).sum(1).max() <= 1 and (m >= 1).all()
    # the same in device buffers, one of them not aligned to 16 bytes
    xd = torch.zeros(chains * N + 1, dtype=torch.uint8, device="cuda")[1:]
    md = torch.zeros(chains, dtype=torch.int64, device="cuda")
    ed = torch.zeros(chains, dtype=torch.float64, device="cuda")
    binding.pns_read(s.ctx, xd, md, ed)
    hd = torch.zeros((chains, N), dtype=torch.int32, device="cuda")
    binding.pns_read_current(s.ctx, fields=hd)
    assert np.array_equal(xd.cpu().numpy().reshape(chains, N), x)
    assert np.array_equal(md.cpu().numpy(), m) and np.array_equal(ed.cpu().numpy(), e)
    assert np.array_equal(hd.cpu().numpy(), c["h"])
    s.close()


def test_batch_rows_and_snapshots():
    sizes, chains = (17, 300, 64, 1023, 256), 60
    Qs = [inputs.symmetric_int(N, -50, 50, np.int16, seed=N, density=0.7) for N in sizes]
    s = BatchSampler([dict(Q=Q, beta=0.02, num_chains=chains, subset_size=8) for Q in Qs], "basic", seed=2,
                     snapshot_every=2, snapshot_capacity=3).run(6)
    x, m, e = s.read()
    for Q, xp, ep in zip(Qs, x, e):
        assert np.array_equal(_energies(Q, xp), ep)
    total = sum(sizes) * chains
    xs = np.zeros(total * 3, np.uint8)
    es = np.zeros((len(sizes) * chains, 3))
    binding.pns_read_snapshots(s.ctx, xs, None, es)
    xd = torch.zeros(total * 3, dtype=torch.uint8, device="cuda")
    binding.pns_read_snapshots(s.ctx, xd, None, None)
    assert np.array_equal(xd.cpu().numpy(), xs)
    at, row = 0, 0
    for Q, N in zip(Qs, sizes):
        for c in range(chains):
            snap = xs[at:at + 3 * N].reshape(3, N)
            assert np.array_equal(_energies(Q, snap), es[row])
            at, row = at + 3 * N, row + 1
    s.close()


# more rows than one launch of a workgroup per row holds (2^32 threads), of a
# size that a piece for host memory holds too (N = 1) or not
@pytest.mark.parametrize("N", [1, 3])
def test_reads_of_more_rows_than_one_launch_holds(N):
    chains, keep = 4200, 4000
    assert chains * keep > 2**24
    Q = inputs.symmetric_int(N, -50, 50, np.int16, seed=N)
    s = Sampler(Q, 0.02, 0, "rf", num_chains=chains, seed=5, init="random", snapshot_every=1, snapshot_capacity=keep)
    s.run(keep)
    xd = torch.full((chains, keep, N), 9, dtype=torch.uint8, device="cuda")
    ed = torch.zeros((chains, keep), dtype=torch.float64, device="cuda")
    binding.pns_read_snapshots(s.ctx, xd, None, ed)
    Qd = torch.from_numpy(Q.astype(np.float64)).cuda()
    for part in range(0, chains, 600):
        x = xd[part:part + 600].double()
        assert bool(((x @ Qd * x).sum(-1) == ed[part:part + 600]).all())
    xh = np.zeros((chains, keep, N), np.uint8)
    binding.pns_read_snapshots(s.ctx, xh, None, None)
    assert np.array_equal(xd.cpu().numpy(), xh)
    s.close()
