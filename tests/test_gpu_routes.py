"""GPU parity of the kernels that a rule on sizes selects, at the edges of their ranges, against
the CPU oracle on the same seeded inputs (tolerances as in tests/parity.py)."""
import numpy as np
import pytest
import torch

import pnn_inputs as I
from oracle import oracle as O
from paper_2304_09590_amd import pnn as B
from tests.parity import BF16_TOL, EPOCH_TOL, assert_close, log

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def make_net(w, th0):
    return B.PNN(B.config_from_workload(w), th0)


def train_both(w, N, epochs):
    """Every CN of `epochs` epochs on the GPU against the oracle's: elementwise in fp32, normwise per
    layer in bf16-mixed precision (where one-ulp differences of the start reach the elementwise
    bar)."""
    X, y = I.train_set(w, N) if w.sizes[0] == 784 else I.random_batch(w.sizes[0], w.sizes[-1], N, 5)
    if w.sizes[-1] < 10:
        y = y % w.sizes[-1]
    th0 = I.init_params(w)
    bf16 = w.precision == I.BF16_MIXED
    log(f"{w.sizes} {w.acts} K={w.replicas} B={w.batch} N={N} precision={w.precision}")
    net = make_net(w, th0)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)
    xd, yd = dev(X), dev(y)
    for _ in range(epochs):
        net.train_epoch(xd, yd)
        o.train_epoch(ref, X, y, threads=8)
    for k in range(w.replicas):
        assert_close(w.sizes, net.get_params(k), ref[k], BF16_TOL if bf16 else EPOCH_TOL, f"replica {k}", layerwise=bf16)
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
    (2, dict(replicas=3), 3 * 70 + 1),
    (2, dict(replicas=3, batch=50), 3 * 110 + 1),
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


# ------------------------------------------------------------------------------------
# the persistent mini-batch kernel: 2 or 4 row tiles of 16 per batch, 16- or 32-neuron tiles, fp32 and
# bf16-mixed; batches at the edges of a row tile and of the range, ragged last batches, input widths
# of 1, 49 and 52 blocks of 16 (waves without a block, with six and with seven), one to 16 tiles

@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("over,N", [
    (dict(sizes=(784, 256, 10), batch=33, replicas=3), 3 * 100 + 2),
    (dict(sizes=(784, 256, 10), batch=64, replicas=2), 2 * 130 + 1),      # last batches of 2 and 3 rows
    (dict(sizes=(784, 256, 10), batch=50, replicas=2), 2 * 150),
    (dict(sizes=(784, 8, 1), acts=(I.SIGMOID, I.SIGMOID), batch=64, replicas=2), 2 * 96 + 1),
    (dict(sizes=(832, 136, 16), acts=(I.TANH, I.SOFTMAX), loss=I.LOSS_XENT, batch=49, replicas=2), 2 * 120 + 1),
    (dict(sizes=(16, 48, 3), batch=48, replicas=3), 3 * 60 + 2),
    (dict(sizes=(784, 512, 10), batch=40, replicas=3), 3 * 90 + 1),       # 16 tiles of 32 neurons
    (dict(sizes=(784, 256, 10), batch=64, replicas=18), 18 * 70 + 5),     # 32-neuron tiles, one launch
    (dict(sizes=(784, 256, 10), batch=36, replicas=40), 40 * 40 + 3),     # two launches of 20 CNs
    (dict(sizes=(784, 64, 10), batch=32, replicas=3), 3 * 70 + 1),
    (dict(sizes=(784, 56, 10), batch=1, replicas=2), 2 * 20 + 1),         # (fp32: per-sample kernel)
    (dict(sizes=(784, 256, 10), batch=17, replicas=33), 33 * 40 + 3),     # 2 launches in all widths
])
def test_persistent_mini_batch(over, N, precision):
    w = I.WORKLOADS[2].scaled(precision=precision, **over)
    net = train_both(w, N, 2)
    if precision == I.BF16_MIXED:
        # the operand copy of the weights was refreshed: an evaluation of a CN (which reads it)
        # agrees with the oracle's forward of the CN's parameters
        X, y = I.train_set(w, 200) if w.sizes[0] == 784 else I.random_batch(w.sizes[0], w.sizes[-1], 200, 6)
        out = torch.empty((200, w.sizes[-1]), dtype=torch.float32, device="cuda")
        net.infer(dev(X), torch.empty(200, dtype=torch.int32, device="cuda"), which=0, out=out)
        ref = O.Oracle.from_workload(w).forward(net.get_params(0).astype(np.float64), X)
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= BF16_TOL
    net.close()


def test_persistent_mini_batch_gives_up_waiting(monkeypatch):
    """(batches above 32 rows and bf16-mixed: a wait that runs into its bound ends the launch; the
    next call reports it)"""
    for over in (dict(batch=50), dict(precision=I.BF16_MIXED)):
        w = I.WORKLOADS[2].scaled(replicas=2, **over)
        X, y = I.train_set(w, 120)
        monkeypatch.setenv("PNN_SPIN_LIMIT", "2000")
        monkeypatch.setenv("PNN_TEST_STALL_WAITS", "1")
        net = make_net(w, I.init_params(w))
        net.train_epoch(dev(X), dev(y))
        with pytest.raises(B.PnnError) as ei:
            net.get_params(0)
        assert ei.value.status == B.PNN_EHIP and "timed out" in str(ei.value)
        net.close()
