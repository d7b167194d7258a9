"""GPU parity of the kernels that a rule on sizes selects, at the edges of their ranges, against
the CPU oracle on the same seeded inputs (tolerances as in tests/parity.py)."""
import numpy as np
import pytest
import torch

import pnn_inputs as I
from oracle import oracle as O
from paper_2304_09590_amd import pnn as B
from tests.parity import EPOCH_TOL, assert_close, log

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def make_net(w, th0):
    return B.PNN(B.config_from_workload(w), th0)


def train_both(w, N, epochs, **env):
    """Every CN of `epochs` epochs on the GPU against the oracle's, elementwise."""
    X, y = I.train_set(w, N)
    th0 = I.init_params(w)
    log(f"{w.sizes} {w.acts} K={w.replicas} B={w.batch} N={N} precision={w.precision}")
    net = make_net(w, th0)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)
    xd, yd = dev(X), dev(y)
    for _ in range(epochs):
        net.train_epoch(xd, yd)
        o.train_epoch(ref, X, y, threads=8)
    for k in range(w.replicas):
        assert_close(w.sizes, net.get_params(k), ref[k], EPOCH_TOL, f"replica {k}")
    return net


# ------------------------------------------------------------------------------------
# per-sample SGD with 129 to 384 hidden neurons: chunks of 32 steps in one persistent launch,
# 4 or 6 neurons per lane; 16- and 32-row tiles; slices that end at, before and after a chunk

@pytest.mark.parametrize("over,N", [
    (dict(sizes=(784, 136, 10), replicas=1), 1),
    (dict(sizes=(784, 136, 10), replicas=2), 2 * 32),
    (dict(sizes=(784, 256, 10), replicas=3), 3 * 33 + 2),
    (dict(sizes=(784, 264, 16), acts=(I.RELU, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.01, replicas=2), 2 * 65 + 1),
    (dict(sizes=(784, 384, 1), replicas=2), 2 * 31),
    (dict(sizes=(784, 256, 10), replicas=20), 20 * 40 + 3),   # 32-row tiles
    (dict(sizes=(784, 144, 10), replicas=70), 70 * 34 + 1),   # two launches of 35 CNs
])
def test_wide_per_sample(over, N):
    train_both(I.WORKLOADS[1].scaled(**over), N, 2).close()


def test_wide_per_sample_late_tiles(monkeypatch):
    """Half of the tile workgroups start late: the sequential workgroup waits for every tile."""
    monkeypatch.setenv("PNN_TEST_TILE_DELAY", "2000")
    train_both(I.WORKLOADS[1].scaled(sizes=(784, 256, 10), replicas=2), 2 * 100 + 1, 2).close()


def test_wide_per_sample_gives_up_waiting(monkeypatch):
    """A wait that runs into its bound ends the launch; the next call reports it."""
    w = I.WORKLOADS[1].scaled(sizes=(784, 256, 10), replicas=2)
    X, y = I.train_set(w, 80)
    monkeypatch.setenv("PNN_SPIN_LIMIT", "2000")
    monkeypatch.setenv("PNN_TEST_STALL_WAITS", "1")
    net = make_net(w, I.init_params(w))
    net.train_epoch(dev(X), dev(y))
    with pytest.raises(B.PnnError) as ei:
        net.merge()
    assert ei.value.status == B.PNN_EHIP and "timed out" in str(ei.value)
    net.close()


@pytest.mark.parametrize("idx,over,N", [
    (1, dict(sizes=(784, 256, 10), replicas=3), 3 * 70 + 1),
])
def test_epoch_recorded_into_a_graph(idx, over, N):
    """An epoch and a merge recorded into a graph on a handle that has trained before, replayed
    with eager work between the replays; each replay against the oracle."""
    w = I.WORKLOADS[idx].scaled(**over)
    X, y = I.train_set(w, N)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    xd, yd = dev(X), dev(y)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)
    net.train_epoch(xd, yd)  # (workspaces grow here)
    o.train_epoch(ref, X, y, threads=4)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.train_epoch(xd, yd)
        net.merge()
    for e in range(3):
        log(f"replay {e}")
        g.replay()
        torch.cuda.synchronize()
        o.train_epoch(ref, X, y, threads=4)
        assert_close(w.sizes, net.get_params(-1), o.merge(ref), EPOCH_TOL, f"merged, replay {e}")
        net.train_epoch(xd, yd)
        o.train_epoch(ref, X, y, threads=4)
        for k in range(w.replicas):
            assert_close(w.sizes, net.get_params(k), ref[k], EPOCH_TOL, f"replica {k}, after replay {e}")
    net.close()
