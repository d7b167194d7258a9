"""GPU parity of the kernels that a rule on sizes selects, at the edges of their ranges, against
the CPU oracle on the same seeded inputs (tolerances as in tests/parity.py)."""
import numpy as np
import pytest
import torch

import pnn_inputs as I
from oracle import oracle as O
from paper_2304_09590_amd import pnn as B
from tests.cases import LAST_LAYER_CASES, MB_PERSISTENT_CASES, SPLIT_FORWARD_CASES, TAIL_CASES
from tests.parity import BF16_TOL, EPOCH_TOL, assert_close, assert_trained, log, oracle_replicas

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def make_net(w, th0):
    return B.PNN(B.config_from_workload(w), th0)


def train_both(w, N, epochs):
    """Every CN of `epochs` epochs on the GPU against the oracle's: elementwise in fp32, normwise per
    layer in bf16-mixed precision (where one-ulp differences of the start reach the elementwise
    bar), and what the epochs added to the start normwise per layer in both.  The network, and the
    launches of each kernel that ran."""
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
    net.profile(True)
    for _ in range(epochs):
        net.train_epoch(xd, yd)
        o.train_epoch(ref, X, y, threads=8)
    ran = {name: launches for name, (_, launches) in net.profile_read().items()}
    net.profile(False)
    for k in range(w.replicas):
        got = net.get_params(k)
        assert_close(w.sizes, got, ref[k], BF16_TOL if bf16 else EPOCH_TOL, f"replica {k}", layerwise=bf16)
        assert_trained(w, got, ref[k], th0, f"replica {k}")
    return net, ran


# ------------------------------------------------------------------------------------
# per-sample SGD with 129 to 384 hidden neurons: chunks of 32 steps in one persistent launch,
# 4 or 6 neurons per lane; 16- and 32-row tiles; slices that end at, before and after a chunk

@pytest.mark.parametrize("over,N,kernel", [
    (dict(sizes=(784, 136, 10), replicas=1), 1, "psgd_chunk"),
    (dict(sizes=(784, 136, 10), replicas=2), 2 * 32, "psgd_persistent"),
    (dict(sizes=(784, 256, 10), replicas=3), 3 * 33 + 2, "psgd_persistent"),
    (dict(sizes=(784, 264, 16), acts=(I.RELU, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.01, replicas=2), 2 * 65 + 1,
     "psgd_persistent"),
    (dict(sizes=(784, 384, 1), replicas=2), 2 * 31, "psgd_persistent"),
    (dict(sizes=(784, 256, 10), replicas=20), 20 * 40 + 3, "psgd_persistent"),    # 32-row tiles
    (dict(sizes=(784, 144, 10), replicas=70), 70 * 34 + 1, "psgd_persistent"),    # two launches of 35 CNs
    (dict(sizes=(784, 264, 10), replicas=16), 16 * 40 + 3, "psgd_persistent"),    # 32-row tiles, six neurons per lane
    (dict(sizes=(784, 136, 10), replicas=256), 256 * 130 + 1, "psgd_persistent"), # the most CNs of the persistent launches
    (dict(sizes=(784, 136, 10), replicas=257), 257 * 3 + 1, "psgd_chunk"),
    (dict(sizes=(840, 128, 10), replicas=2), 2 * 300 + 1, "psgd_chunk"),          # chunks of 128 steps (wide inputs)
    (dict(sizes=(784, 256, 10), replicas=257), 257 * 70 + 1, "psgd_chunk"),       # of 64
    (dict(sizes=(784, 392, 10), replicas=2), 2 * 70 + 1, "psgd_chunk"),           # of 32
])
def test_wide_per_sample(over, N, kernel):
    net, ran = train_both(I.WORKLOADS[1].scaled(**over), N, 2)
    assert kernel in ran and {"psgd_chunk": "psgd_persistent", "psgd_persistent": "psgd_chunk"}[kernel] not in ran, ran
    net.close()


def kernels_of_an_epoch(net, X, y):
    net.profile(True)
    net.train_epoch(dev(X), dev(y))
    names = set(net.profile_read())
    net.profile(False)
    return names


@pytest.mark.parametrize("over,rows,persistent", [
    (dict(sizes=(784, 256, 10), replicas=2), 100, True),
    (dict(sizes=(784, 256, 10), replicas=2), 2, False),      # one launch's start-up is more than two steps
    (dict(sizes=(784, 256, 10), replicas=128), 40, False),   # five launches against all CNs at once
    (dict(sizes=(784, 256, 10), replicas=128), 100, True),
    (dict(sizes=(784, 384, 10), replicas=128), 60, False),
    (dict(sizes=(784, 384, 10), acts=(I.TANH, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.01, replicas=4), 60, True),
    (dict(sizes=(784, 384, 10), acts=(I.TANH, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.01, replicas=128), 300, False),
])
def test_wide_per_sample_short_slices(over, rows, persistent):
    """Where several persistent launches would follow each other for short slices, or for a slower
    step than all CNs take together, an epoch takes the launches per chunk; both agree with the oracle."""
    w = I.WORKLOADS[1].scaled(**over)
    K = w.replicas
    X, y = I.train_set(w, K * rows)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    names = kernels_of_an_epoch(net, X, y)
    assert ("psgd_persistent" in names, "psgd_chunk" in names) == (persistent, not persistent), names
    o = O.Oracle.from_workload(w)
    ids = sorted({0, K // 2, K - 1})
    ref = oracle_replicas(o, np.tile(th0.astype(np.float64), (len(ids), 1)), ids, X, y)
    for i, k in enumerate(ids):
        assert_close(w.sizes, net.get_params(k), ref[i], EPOCH_TOL, f"replica {k}")
    net.close()


def test_wide_per_sample_of_many_chunks():
    """More Gram products than a launch can take (65,535), in the launches per chunk."""
    w = I.WORKLOADS[1].scaled(sizes=(8, 384, 10), acts=(I.TANH, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.005, replicas=128)
    K = w.replicas
    X, y = I.random_batch(8, 10, K * (32 * 512 + 5), 5)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    assert "psgd_chunk" in kernels_of_an_epoch(net, X, y)
    ids = [0, 126, 127]
    ref = oracle_replicas(O.Oracle.from_workload(w), np.tile(th0.astype(np.float64), (len(ids), 1)), ids, X, y)
    for i, k in enumerate(ids):
        assert_close(w.sizes, net.get_params(k), ref[i], EPOCH_TOL, f"replica {k}")
        assert_trained(w, net.get_params(k), ref[i], th0, f"replica {k}")
    net.close()


def first_step_w2(H, act2, b1, b2):
    """W2 after an epoch from W2 = 0 with eta = 1 and the cross-entropy error, in which only the first
    row counts: -(x2 - e) a1^T of the activations of the biases themselves.  The first row is zero; the
    others are one at input 0, whose weights of -1000 leave their hidden activations zero."""
    w = I.WORKLOADS[1].scaled(sizes=(784, H, len(b2)), acts=(I.SIGMOID, act2), loss=I.LOSS_XENT, lr=1.0, replicas=1)
    W1 = np.zeros((H, 784))
    W1[:, 0] = -1000
    net = make_net(w, np.concatenate([W1.ravel(), b1, np.zeros(H * len(b2)), b2]).astype(np.float32))
    X = np.zeros((200, 784), np.float32)
    X[1:, 0] = 1
    net.train_epoch(dev(X), dev(np.zeros(200, np.int32)))
    W2 = net.get_params(0)[785 * H:-len(b2)].astype(np.float64).reshape(len(b2), H)
    net.close()
    return W2


@pytest.mark.parametrize("H", [136, 256, 264, 384])
def test_wide_per_sample_activations_are_exact(H):
    """The activations are as exact as the launches per chunk make them (e^x within one ulp, 1 + e and
    the quotient within half an ulp each: 2.4e-7 in all; the hardware's exp2 and reciprocal alone
    are off by 9e-7 at z = -15)."""
    def sig(z):
        return 1 / (1 + np.exp(-z.astype(np.float64)))
    b1 = np.linspace(-15, 4, H).astype(np.float32)
    # hidden: the output of b2 = 0 is 0.5 exactly, and so is its error (the label is output 0)
    W2 = first_step_w2(H, I.SIGMOID, b1, np.zeros(2, np.float32))
    assert np.max(np.abs(W2[1] / -0.5 / sig(b1) - 1)) <= 2.4e-7
    # output: a1 = 0.5 exactly
    b2 = -3 * np.arange(10).astype(np.float32)
    W2 = first_step_w2(H, I.SIGMOID, np.zeros(H, np.float32), b2)
    assert np.max(np.abs(W2[1:, 0] / -0.5 / sig(b2)[1:] - 1)) <= 2.4e-7
    # softmax: e^x within one ulp, a sum of ten within one ulp and four roundings, 1 / sum and the
    # product within half an ulp each
    W2 = first_step_w2(H, I.SOFTMAX, np.zeros(H, np.float32), b2)
    e = np.exp(b2.astype(np.float64))
    assert np.max(np.abs(W2[1:, 0] / -0.5 / (e / e.sum())[1:] - 1)) <= 6e-7


def test_wide_per_sample_activations_at_the_ends_of_the_range():
    """Sigmoids of -inf, -100 and 100 are 0, 0 and 1 (the hardware's e^x and reciprocal stand there,
    within the smallest normal number), and that of NaN is NaN."""
    b1 = np.zeros(256, np.float32)
    b1[:3] = -np.inf, -100, 100
    W2 = first_step_w2(256, I.SIGMOID, b1, np.zeros(2, np.float32))
    assert np.allclose(W2[1, :4], [0, 0, -0.5, -0.25], rtol=0, atol=1.2e-38)
    b1[3] = np.nan
    assert np.isnan(first_step_w2(256, I.SIGMOID, b1, np.zeros(2, np.float32))).all()


@pytest.mark.parametrize("over", [dict(sizes=(784, 256, 10), replicas=4),
                                  dict(sizes=(784, 136, 10), replicas=20),   # 32-row tiles
                                  dict(sizes=(784, 384, 10), acts=(I.TANH, I.SOFTMAX), loss=I.LOSS_XENT, lr=0.005, replicas=2)])
def test_wide_per_sample_is_as_exact_as_launches_per_chunk(over):
    """The persistent kernel's parameters after 500 steps are no further from the oracle's (64 bits)
    than those of the launches per chunk, which a recorded epoch takes."""
    w = I.WORKLOADS[1].scaled(**over)
    K = w.replicas
    X, y = I.train_set(w, K * 500)
    th0 = I.init_params(w)
    xd, yd = dev(X), dev(y)
    net = make_net(w, th0)
    assert "psgd_persistent" in kernels_of_an_epoch(net, X, y)
    ids = [0, K - 1]
    got = [net.get_params(k) for k in ids]
    net.set_params(-2, th0)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        net.train_epoch(xd, yd)
    g.replay()
    torch.cuda.synchronize()
    launches = [net.get_params(k) for k in ids]
    net.close()
    ref = oracle_replicas(O.Oracle.from_workload(w), np.tile(th0.astype(np.float64), (2, 1)), ids, X, y)

    def off(p):
        return float(np.linalg.norm(np.stack(p) - ref) / np.linalg.norm(ref))
    log(f"persistent {off(got):.2e}, launches per chunk {off(launches):.2e}")
    assert off(got) <= off(launches)


def test_wide_per_sample_late_tiles(monkeypatch):
    """Half of the tile workgroups start late: the sequential workgroup waits for every tile."""
    monkeypatch.setenv("PNN_TEST_TILE_DELAY", "2000")
    net, ran = train_both(I.WORKLOADS[1].scaled(sizes=(784, 256, 10), replicas=2), 2 * 100 + 1, 2)
    assert "psgd_persistent" in ran
    net.close()


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


@pytest.mark.parametrize("idx,over,rows", [
    (1, dict(sizes=(784, 384, 10), replicas=2), (100, 120, 120, 600)),  # (an eager epoch's blocks: 40 floats a row, not 32)
    (1, dict(sizes=(784, 512, 10), replicas=2), (100, 100, 130, 600)),
])
def test_recorded_epoch_outlives_larger_ones(idx, over, rows):
    """A recorded epoch replayed after epochs of more rows, whose workspace has taken the place of the
    recorded one's: every replay against the oracle."""
    w = I.WORKLOADS[idx].scaled(**over)
    K = w.replicas
    first, recorded, *later = (K * r for r in rows)
    X, y = I.train_set(w, K * rows[-1])
    xd, yd = dev(X), dev(y)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)

    def eager(n):
        net.train_epoch(xd[:n], yd[:n])
        o.train_epoch(ref, X[:n], y[:n], threads=K)

    eager(first)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.train_epoch(xd[:recorded], yd[:recorded])
    for n in later:
        eager(n)
        junk = torch.full((64 << 20,), float("nan"), device="cuda")  # (takes memory that was freed)
        log(f"replay of {recorded} rows after {n}")
        g.replay()
        torch.cuda.synchronize()
        o.train_epoch(ref, X[:recorded], y[:recorded], threads=K)
        for k in range(K):
            assert_close(w.sizes, net.get_params(k), ref[k], EPOCH_TOL, f"replica {k}, after {n} rows")
        del junk
    net.close()


def test_recorded_calls_keep_their_workspace():
    """Recorded inference and recorded epochs in a given order, replayed after calls with more rows."""
    w = I.WORKLOADS[2].scaled(replicas=2)
    X, y = I.train_set(w, 2 * 300)
    xd, yd = dev(X), dev(y)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)
    small, large = 2 * 70, 2 * 300
    order = np.random.default_rng(1).permutation(small).astype(np.int32)
    od, ol = dev(order), dev(np.arange(large, dtype=np.int32))
    pred = torch.empty(large, dtype=torch.int32, device="cuda")
    out = torch.empty((small, 10), dtype=torch.float32, device="cuda")
    net.train_epoch_order(xd[:small], yd[:small], od)
    o.train_epoch(ref, X[order], y[order], threads=2)
    net.infer(xd[:small], pred[:small], which=1, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.train_epoch_order(xd[:small], yd[:small], od)
        net.infer(xd[:small], pred[:small], which=1, out=out)
    net.train_epoch_order(xd, yd, ol)
    o.train_epoch(ref, X, y, threads=2)
    net.infer(xd, pred, which=0)
    for e in range(2):
        junk = torch.full((64 << 20,), float("nan"), device="cuda")
        log(f"replay {e}")
        g.replay()
        torch.cuda.synchronize()
        o.train_epoch(ref, X[order], y[order], threads=2)
        for k in range(2):
            assert_close(w.sizes, net.get_params(k), ref[k], EPOCH_TOL, f"replica {k}, replay {e}")
        assert np.max(np.abs(out.cpu().numpy() - o.forward(ref[1], X[:small]))) <= EPOCH_TOL
        del junk
    net.close()


@pytest.mark.parametrize("call", ["epoch", "order", "infer"])
def test_growth_is_refused_while_recording(call):
    """A recorded call with more rows than the workspace holds is refused with a message that says
    what to do; the handle stays usable and its workspace whole."""
    w = I.WORKLOADS[1].scaled(sizes=(784, 384, 10), replicas=2)
    X, y = I.train_set(w, 400)
    xd, yd = dev(X), dev(y)
    od = dev(np.arange(400, dtype=np.int32))
    pred = torch.empty(400, dtype=torch.int32, device="cuda")
    th0 = I.init_params(w)
    net = make_net(w, th0)
    o = O.Oracle.from_workload(w)
    ref = o.replicate(th0)
    net.train_epoch_order(xd[:40], yd[:40], od[:40])
    o.train_epoch(ref, X[:40], y[:40], threads=2)
    net.infer(xd[:40], pred[:40])
    torch.cuda.synchronize()
    calls = {"epoch": lambda: net.train_epoch(xd, yd), "order": lambda: net.train_epoch_order(xd, yd, od),
             "infer": lambda: net.infer(xd, pred)}
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        with pytest.raises(B.PnnError) as ei:
            calls[call]()
        net.merge()
    assert ei.value.status == B.PNN_EHIP and "records a graph" in str(ei.value)
    g.replay()   # (the recording went on)
    torch.cuda.synchronize()
    assert_close(w.sizes, net.get_params(-1), o.merge(ref), EPOCH_TOL, "merged")
    calls[call]()
    if call != "infer":
        o.train_epoch(ref, X, y, threads=2)
    for k in range(2):
        assert_close(w.sizes, net.get_params(k), ref[k], EPOCH_TOL, f"replica {k}")
    net.close()


# ------------------------------------------------------------------------------------
# the persistent mini-batch kernel

@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("over,N", MB_PERSISTENT_CASES)
def test_persistent_mini_batch(over, N, precision):
    w = I.WORKLOADS[2].scaled(precision=precision, **over)
    net, ran = train_both(w, N, 2)
    assert ("psgd_persistent" if w.batch == 1 and precision == I.FP32 else "mb_persistent") in ran, ran
    assert not {"fwd_gemm", "fwd_gemm_x3", "tail", "out_layer"} & set(ran), ran
    if precision == I.BF16_MIXED:
        # the operand copy of the weights was refreshed: an evaluation of a CN (which reads it)
        # agrees with the oracle's forward of the CN's parameters
        X, y = I.train_set(w, 200) if w.sizes[0] == 784 else I.random_batch(w.sizes[0], w.sizes[-1], 200, 6)
        out = torch.empty((200, w.sizes[-1]), dtype=torch.float32, device="cuda")
        net.infer(dev(X), torch.empty(200, dtype=torch.int32, device="cuda"), which=0, out=out)
        ref = O.Oracle.from_workload(w).forward(net.get_params(0).astype(np.float64), X)
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= BF16_TOL
    net.close()


@pytest.mark.parametrize("precision,over,persistent", [
    (I.BF16_MIXED, dict(sizes=(16, 512, 10), batch=32, replicas=200), False),
    (I.BF16_MIXED, dict(sizes=(64, 384, 10), batch=24, replicas=200), False),
    (I.BF16_MIXED, dict(sizes=(256, 384, 10), batch=1, replicas=200), False),
    (I.BF16_MIXED, dict(sizes=(784, 256, 10), batch=16, replicas=100), True),
    (I.BF16_MIXED, dict(sizes=(16, 16, 10), batch=16, replicas=600), True),   # three launches of 16 neurons
    (I.BF16_MIXED, dict(sizes=(64, 64, 10), batch=64, replicas=332), False),
    (I.FP32, dict(sizes=(16, 256, 10), batch=64, replicas=64), False),
    (I.FP32, dict(sizes=(784, 384, 10), batch=48, replicas=32), True),
    (I.FP32, dict(sizes=(16, 512, 10), batch=32, replicas=100), True),        # (up to 32 rows: always)
])
def test_persistent_mini_batch_or_launches(over, precision, persistent):
    """Several persistent launches for a step, or a launch per layer that takes all CNs at once; both
    agree with the oracle."""
    w = I.WORKLOADS[2].scaled(precision=precision, **over)
    K = w.replicas
    X, y = I.random_batch(w.sizes[0], w.sizes[-1], K * w.batch + 3, 5)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    names = kernels_of_an_epoch(net, X, y)
    assert ("mb_persistent" in names) == persistent and ("upd_gemm" in names or "upd_gemm_x3" in names) != persistent, names
    o = O.Oracle.from_workload(w)
    ids = sorted({0, 2, K // 2, K - 1})
    ref = oracle_replicas(o, np.tile(th0.astype(np.float64), (len(ids), 1)), ids, X, y)
    bf16 = precision == I.BF16_MIXED
    for i, k in enumerate(ids):
        got = net.get_params(k)
        assert_close(w.sizes, got, ref[i], BF16_TOL if bf16 else EPOCH_TOL, f"replica {k}", layerwise=bf16)
        assert_trained(w, got, ref[i], th0, f"replica {k}")
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


# ------------------------------------------------------------------------------------
# forward products with the contraction split over the waves of a workgroup (tiles of 16 and of
# 32), the update in 64 x 64 tiles where there are few strips, and the inference output layer:
# rows and widths at the edges of their tiles, contractions of 1 to 52 blocks

@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("over,N", SPLIT_FORWARD_CASES)
def test_split_forward_and_few_strips(over, N, precision, monkeypatch):
    monkeypatch.setenv("PNN_MB_PLAN", "launch")
    net, ran = train_both(I.WORKLOADS[2].scaled(precision=precision, **over), N, 1)
    # (the update on the split-bf16 products with more than 128 strips, and with more than 128 samples)
    x3 = precision == I.FP32 and (over["replicas"] == 72 or over["batch"] == 129)
    assert "fwd_gemm" in ran and "fwd_gemm_x3" not in ran and ("upd_gemm_x3" in ran) == x3, ran
    net.close()


@pytest.mark.parametrize("over", [
    dict(sizes=(784, 1024, 10), batch=128, replicas=64),  # 128 x 256 tiles: one round of workgroups
    dict(sizes=(64, 384, 10), batch=300, replicas=64),    # 128 x 256: two rounds, a short contraction
    dict(sizes=(784, 384, 10), batch=300, replicas=64),   # 128 x 128: two rounds of the larger would take longer
    dict(sizes=(784, 1024, 10), batch=128, replicas=17),  # 128 x 128 in one round; the update in strips
])
def test_split_bf16_forward_of_many_cns(over, monkeypatch):
    """The split-bf16 forward with the last layer in launches of its own, in tiles of 128 x 256 and of
    128 x 128, the last batch ragged."""
    monkeypatch.setenv("PNN_MB_PLAN", "launch")
    w = I.WORKLOADS[4].scaled(**over)
    K = w.replicas
    X, y = I.random_batch(w.sizes[0], w.sizes[-1], K * (w.batch + 5) + 1, 5)
    th0 = I.init_params(w)
    net = make_net(w, th0)
    names = kernels_of_an_epoch(net, X, y)
    assert {"fwd_gemm_x3", "out_layer", "last_layer"} <= names, names
    ids = [0, K // 2, K - 1]
    ref = oracle_replicas(O.Oracle.from_workload(w), np.tile(th0.astype(np.float64), (len(ids), 1)), ids, X, y)
    for i, k in enumerate(ids):
        got = net.get_params(k)
        assert_close(w.sizes, got, ref[i], EPOCH_TOL, f"replica {k}")
        assert_trained(w, got, ref[i], th0, f"replica {k}")
    net.close()


@pytest.mark.parametrize("batch", [50, 96])
def test_update_strips_of_short_batches(batch, monkeypatch):
    """The weight update in strips of 128 rows with at most 96 samples (three k-chunks or fewer)."""
    monkeypatch.setenv("PNN_MB_PLAN", "launch")
    net, ran = train_both(I.WORKLOADS[2].scaled(batch=batch, replicas=72), 72 * (batch + 3) + 1, 1)
    assert "upd_gemm_x3" in ran, ran
    net.close()


@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("sizes,acts,loss,rows", [
    ((784, 128, 10), (I.SIGMOID, I.SIGMOID), I.LOSS_MSE, 1),
    ((784, 40, 10), (I.RELU, I.SOFTMAX), I.LOSS_XENT, 17),
    ((784, 264, 16), (I.TANH, I.SOFTMAX), I.LOSS_XENT, 300),
    ((784, 1024, 10), (I.SIGMOID, I.SIGMOID), I.LOSS_XENT, 1809),
    ((784, 512, 256, 3), (I.RELU, I.LEAKY_RELU, I.SIGMOID), I.LOSS_MSE, 8192 + 33),  # two chunks
    ((784, 1), (I.SIGMOID,), I.LOSS_XENT, 50),
    ((784, 10), (I.SOFTMAX,), I.LOSS_XENT, 33),
    ((24, 8, 2), (I.TANH, I.SIGMOID), I.LOSS_MSE, 15),
])
def test_inference_routes(sizes, acts, loss, rows, precision):
    """Outputs, predictions, count and cost of one CN against the oracle's forward of the same
    parameters (fp32 1e-5, the one-step bar; bf16 2e-2)."""
    w = I.WORKLOADS[2].scaled(sizes=sizes, acts=acts, loss=loss, precision=precision, replicas=2, batch=8)
    X, _ = I.random_batch(sizes[0], sizes[-1], rows, 3)
    y = np.random.default_rng(4).integers(0, sizes[-1], rows).astype(np.int32)
    th = I.random_params(sizes, 9, 0.1)
    log(f"{sizes} rows {rows} precision {precision}")
    net = make_net(w, I.init_params(w))
    net.set_params(1, th)
    pred = torch.full((rows,), -1, dtype=torch.int32, device="cuda")
    out = torch.empty((rows, sizes[-1]), dtype=torch.float32, device="cuda")
    correct = net.infer(dev(X), pred, which=1, out=out, y=dev(y), count=True)
    got, p = out.cpu().numpy(), pred.cpu().numpy()
    o = O.Oracle.from_workload(w)
    ref = o.forward(th.astype(np.float64), X)
    tol = 1e-5 if precision == I.FP32 else 2e-2
    assert np.max(np.abs(got - ref)) <= tol
    assert np.array_equal(p, np.argmax(got, axis=1))   # (of its own outputs: lowest index on ties)
    assert correct == int(np.sum(p == y))
    c, cost = net.evaluate(dev(X), dev(y), which=1)
    c2, cost2 = net.evaluate_noalloc(dev(X), dev(y), which=1)
    g64 = got.astype(np.float64)
    hot = np.eye(sizes[-1])[y]
    if loss == I.LOSS_MSE:
        want = 0.5 * np.sum((g64 - hot) ** 2, axis=1)
    elif acts[-1] == I.SOFTMAX:
        want = -np.log(np.sum(g64 * hot, axis=1))
    else:
        want = -np.sum(hot * np.log(g64) + (1 - hot) * np.log(1 - g64), axis=1)
    assert (c, c2) == (correct, correct) and abs(cost - want.mean()) <= 1e-12 * max(1, rows) and cost2 == cost
    net.close()


def test_inference_of_not_a_number():
    """A NaN output is never the greatest one, unless it is the first: the prediction of a row
    without any number is 0, and other rows are not touched."""
    w = I.WORKLOADS[2].scaled(sizes=(784, 16, 10), replicas=1, batch=8)
    X, _ = I.random_batch(784, 10, 40, 3)
    net = make_net(w, I.init_params(w))
    pred = torch.empty(40, dtype=torch.int32, device="cuda")
    out = torch.empty((40, 10), dtype=torch.float32, device="cuda")
    net.infer(dev(X), pred, out=out)
    clean, ref = out.cpu().numpy(), pred.cpu().numpy()
    X[7] = np.nan
    net.infer(dev(X), pred, out=out)
    got, p = out.cpu().numpy(), pred.cpu().numpy()
    rest = np.arange(40) != 7
    assert np.all(np.isnan(got[7])) and p[7] == 0
    assert np.array_equal(got[rest], clean[rest]) and np.array_equal(p[rest], ref[rest])
    net.close()


# ------------------------------------------------------------------------------------
# the last layer in two kernels (errors by row, then hidden errors and update by columns), and in one
# workgroup per CN

@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("over,N", LAST_LAYER_CASES)
def test_last_layer_in_two_kernels(over, N, precision, monkeypatch):
    monkeypatch.setenv("PNN_MB_PLAN", "launch")
    w = I.WORKLOADS[2].scaled(precision=precision, **over)
    net, ran = train_both(w, N, 2)
    assert {"out_layer", "last_layer"} <= set(ran) and "tail" not in ran, ran
    if precision == I.BF16_MIXED and len(w.sizes) == 4:   # (up to 64 rows both wide layers in one launch)
        assert ran["upd_gemm"] == ran["last_layer"] * (1 if w.batch <= 64 else 2), ran
    net.close()


@pytest.mark.parametrize("precision", [I.FP32, I.BF16_MIXED])
@pytest.mark.parametrize("over,N", TAIL_CASES)
def test_last_layer_in_one_workgroup_per_cn(over, N, precision, monkeypatch):
    monkeypatch.setenv("PNN_MB_PLAN", "launch")
    net, ran = train_both(I.WORKLOADS[2].scaled(precision=precision, **over), N, 2)
    assert "tail" in ran and "last_layer" not in ran, ran
    net.close()
