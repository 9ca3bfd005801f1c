"""Calls under HIP graph capture: each captured once, replayed several times
with eager work and synchronizations between the replays, and every replay
compared bit for bit with the eager call's outputs (the oracle's, by the
parity tests)."""
import ctypes

import numpy as np
import pytest

import oracle as orc
from paper_1206_1187_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1206_1187_amd as nn  # noqa: E402
from paper_1206_1187_amd import _native  # noqa: E402

SENTINEL = -77


@pytest.fixture(scope="module", autouse=True)
def _device():
    assert torch.cuda.is_available()
    nn.init(0)
    yield
    torch.cuda.synchronize()


def _replayed(call, out):
    """`call` captured on a stream of its own; the contents of `out` after each
    of four replays into cleared memory, with other launches between them."""
    call()  # one-time set-up stays out of the graph
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    other = torch.empty(5000, dtype=torch.float64, device="cuda")
    got = []
    for k in range(4):
        out.fill_(SENTINEL)
        torch.cuda.synchronize()
        graph.replay()
        if k % 2:
            nn.generate_into(orc.seed(wl.INDEX_MIN + k), other)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy().copy())
    return got


@pytest.mark.parametrize("count", [1, 1000, 3_000_017, (1 << 24) + 5])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("what", ["f64", "u64", "e40"])
def test_captured_generation(what, count, skew):
    buf = torch.empty(count + 3, dtype=torch.int64, device="cuda")
    out = buf[skew:skew + count].view(torch.float64 if what == "f64" else torch.uint64)
    if what == "e40":
        z0 = orc.e40_seed(orc.E40_INDEX_MIN + 9)
        call = lambda: nn.e40_generate_into(z0, out)  # noqa: E731
    else:
        z0 = orc.seed(wl.INDEX_MIN + 9)
        call = lambda: nn.generate_into(z0, out)  # noqa: E731
    buf.fill_(SENTINEL)
    call()
    want = buf.cpu().numpy().copy()
    for got in _replayed(call, buf):
        assert np.array_equal(got, want)


@pytest.mark.parametrize("new,count", [(True, 0)] + [(new, count) for new in (False, True)
                                                     for count in (1000, 1 << 15, 300_001)])
def test_captured_consumer(new, count):
    """Adding to a result, and setting it (one workgroup up to 2^15 outputs, a
    clearing launch before several above)."""
    z0 = orc.seed(wl.INDEX_MIN + 11)
    ref, _ = orc.gen(z0, count, "u64", threads=0)
    want = int(sum(int(x) for x in ref)) % 2 ** 64
    res = torch.zeros(1, dtype=torch.int64, device="cuda")
    fn = _native.lib().nn_consume_set if new else _native.lib().nn_consume

    def call():
        st = ctypes.c_uint64(z0)
        _native.check(fn(ctypes.byref(st), count, nn._native.NN_OUT_U64, res.data_ptr(),
                         torch.cuda.current_stream().cuda_stream, None))

    for got in _replayed(call, res):
        assert int(got[0]) % 2 ** 64 == (want if new else (want + SENTINEL) % 2 ** 64)


@pytest.mark.parametrize("n", [3, 128, 129, 1100])
def test_captured_static_batch(n):
    """The batched call that allocates nothing: under capture at every number of
    windows it copies its descriptors, which the graph reads again at each
    replay, also where an eager call puts them in the kernel arguments."""
    rng = np.random.default_rng(n)
    lengths = np.floor(np.exp(rng.uniform(0.0, np.log(9000.0), n))).astype(np.uint64)
    states = np.array([orc.seed(wl.INDEX_MIN + 31 * i) for i in range(n)], dtype=np.uint64)
    offsets = 1 + np.concatenate([[0], np.cumsum(lengths)[:-1]]).astype(np.uint64)
    total = int(lengths.sum()) + 4
    buf = torch.full((total,), SENTINEL, dtype=torch.int64, device="cuda")
    descs = nn._batch_descs(states, lengths, offsets, buf)

    def call():
        _native.check(_native.lib().nn_generate_batch_static(
            descs.ctypes.data, n, buf.data_ptr(), nn._native.NN_OUT_U64,
            torch.cuda.current_stream().cuda_stream, None))

    call()
    torch.cuda.synchronize()
    want = buf.cpu().numpy().copy()
    for s, k, o in zip(states.tolist(), lengths.tolist(), offsets.tolist()):
        assert np.array_equal(want[o:o + k].view(np.uint64), orc.gen(s, k, "u64")[0])
    for got in _replayed(call, buf):
        assert np.array_equal(got, want)
