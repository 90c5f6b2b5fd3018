"""The few-row GEMM kernels behind oc_rest_of_layer, stage by stage against
float64 products of the same bfloat16 inputs, at the edges of their row
tiles, K splits and of the rule that hands products to the GEMM library; on
several streams, under capture, and where one stream handle's calls overlap."""
import threading

import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()
    import torch
    torch.cuda.synchronize()
    yield
    torch.cuda.synchronize()


class Layer:
    """Random weights, input and sentinel-padded output buffers of one layer."""

    def __init__(self, nq, nkv, d, F, T, seed, pad=3):
        import torch
        import paper_2605_22850_amd as oc
        g = torch.Generator(device="cuda").manual_seed(seed)
        H, NQ = nq * d, (nq + 2 * nkv) * d

        def normal(*shape, scale=1.0):
            return torch.randn(*shape, dtype=torch.bfloat16, device="cuda", generator=g) * scale

        self.T, self.F, self.pad = T, F, pad
        self.layout = oc.Layout(1, nq, nkv, d, 16, 16, 1)
        self.x = normal(T, H)
        self.w = [normal(1, K, N, scale=K ** -0.5) for K, N in ((H, H), (H, 2 * F), (F, H), (H, NQ))]
        self.weights = oc.LayerWeights(F, *self.w)
        self.bufs = [torch.full((T + pad, n), 7.0, dtype=torch.bfloat16, device="cuda") for n in (H, 2 * F, F, H, NQ)]

    def run(self, stream=None):
        import paper_2605_22850_amd as oc
        oc.oc_rest_of_layer(self.x, self.T, self.layout, self.weights, 0, *self.bufs, stream=stream)

    def check(self, what):
        o, gu, act, h, qkv = (b[:self.T] for b in self.bufs)
        for y, x, w, name in ((o, self.x, self.w[0], "o"), (gu, o, self.w[1], "gate_up"), (h, act, self.w[2], "h"),
                              (qkv, h, self.w[3], "qkv")):
            a, b = x.double(), w[0].double()
            ref = a @ b
            # half a bf16 ulp of the result (2^-8 of it: 8 significant bits),
            # plus K fp32 additions of products that sum to at most |x| . |w|
            # in magnitude
            bound = 2.0 ** -8 * ref.abs() + a.shape[1] * 2.0 ** -23 * (a.abs() @ b.abs()) + 1e-30
            worst = ((y.double() - ref).abs() / bound).max().item()
            assert worst <= 1.0, f"{what} {name}: {worst:.2f} of the bound"
        gate, up = gu[:, :self.F].double(), gu[:, self.F:].double()
        ref = gate / (1 + (-gate).exp()) * up
        # half a bf16 ulp (2^-8 of the value: 8 significant bits) plus a few
        # fp32 ulps of exp, divide and multiply
        worst = ((act.double() - ref).abs() / ((2.0 ** -8 + 2.0 ** -18) * ref.abs() + 1e-30)).max().item()
        assert worst <= 1.0, f"{what} act: {worst:.2f} of the bound"
        for b in self.bufs:
            untouched = (b[self.T:] == 7.0).all().item()
            assert untouched, f"{what}: rows past the last written"


# row tiles of 32, 64, 128 and 256, one past each, and past the rule's limits
ROWS = [1, 31, 32, 33, 64, 65, 127, 128, 129, 256, 257, 300, 385, 512, 513]


@pytest.mark.parametrize("T", ROWS)
def test_row_tiles(T):
    # F = 192: K of 3 steps; 2F = 384: three column tiles
    print(f"[gemm rows] T {T}", flush=True)
    c = Layer(8, 2, 64, 192, T, seed=T)
    c.run()
    c.check(f"T {T}")


# one K step; ffn sizes that leave the last split short; products the library
# keeps (N or K not whole tiles); the 8B layer on both sides of the unsplit
# limit; gate|up of as many column tiles as CUs, and of more (the library's)
SHAPES = [(4, 4, 64, 64, 5), (8, 8, 64, 1728, 40), (8, 2, 128, 832, 100), (4, 1, 64, 72, 9), (6, 2, 24, 40, 33),
          (32, 8, 128, 14336, 64), (32, 8, 128, 14336, 65), (4, 1, 64, 16384, 9), (4, 1, 64, 16512, 9)]


@pytest.mark.parametrize("nq,nkv,d,F,T", SHAPES)
def test_shapes(nq, nkv, d, F, T):
    print(f"[gemm rows] nq {nq} nkv {nkv} d {d} F {F} T {T}", flush=True)
    c = Layer(nq, nkv, d, F, T, seed=F + T)
    c.run()
    c.check(f"F {F} T {T}")


@pytest.mark.parametrize("T", [1, 40, 130, 400])
def test_a_call_repeats_itself_bit_for_bit(T):
    import torch
    print(f"[gemm rows] twice, T {T}", flush=True)
    c = Layer(32, 8, 128, 2048, T, seed=60)
    c.run()
    torch.cuda.synchronize()
    want = [b.clone() for b in c.bufs]
    for _ in range(4):
        for b in c.bufs:
            b[:T].fill_(3.0)
        c.run()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(c.bufs, want))


def test_streams_do_not_share_partials():
    import torch
    print("[gemm rows] four streams", flush=True)
    cases = [Layer(32, 8, 128, 2048, 40 + 90 * i, seed=50 + i) for i in range(4)]
    streams = [torch.cuda.Stream() for _ in cases]
    torch.cuda.synchronize()
    for _ in range(5):
        for c, s in zip(cases, streams):
            c.run(s)
    torch.cuda.synchronize()
    for i, c in enumerate(cases):
        c.check(f"stream {i}")


def test_under_capture():
    import torch
    print("[gemm rows] captured", flush=True)
    c = Layer(8, 2, 64, 1792, 130, seed=9)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        c.run(s)            # the stream's workspace is made before the capture
    torch.cuda.synchronize()
    want = [b.clone() for b in c.bufs]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run(s)
    for k in range(4):
        for b in c.bufs:
            b[:c.T].fill_(float(k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(c.bufs, want)), f"replay {k}"
        c.check(f"replay {k}")


@pytest.mark.parametrize("T,offset", [(40, 0), (64, 256), (1, 0), (200, 64)])
def test_act_may_take_the_memory_of_o(T, offset):
    """A caller that keeps no o lets act write over it (F <= H here, from
    `offset` elements on): the chain behind it is that of separate buffers."""
    import torch
    print(f"[gemm rows] act over o, T {T} offset {offset}", flush=True)
    a, b = (Layer(8, 2, 64, 256, T, seed=90) for _ in range(2))
    F = 256
    b.bufs[2] = b.bufs[0].view(-1)[offset:offset + (T + b.pad) * F].view(T + b.pad, F)
    a.run()
    b.run()
    torch.cuda.synchronize()
    a.check(f"apart, T {T}")
    for i, name in ((1, "gate_up"), (2, "act"), (3, "h"), (4, "qkv")):
        x, y = a.bufs[i][:T].double(), b.bufs[i][:T].double()
        # two correct results of bf16 stages: a few ulps, each stage on the last one's
        assert ((x - y).norm() / x.norm()).item() < 1e-2, name


def test_graphs_of_one_stream_replayed_together():
    """Two graphs captured on one stream, replayed on two others beside eager
    calls on it: no call's kernels may use another's partial sums."""
    import torch
    print("[gemm rows] two graphs of one stream and eager calls, overlapping", flush=True)
    a, b, c = (Layer(32, 8, 128, 2048, t, seed=70 + t) for t in (40, 130, 60))
    s, s1, s2 = (torch.cuda.Stream() for _ in range(3))
    with torch.cuda.stream(s):
        c.run(s)
    torch.cuda.synchronize()
    graphs = []
    for x in (a, b):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            x.run(s)
        graphs.append(g)
    torch.cuda.synchronize()
    for k in range(4):
        for _ in range(5):
            with torch.cuda.stream(s1):
                graphs[0].replay()
            with torch.cuda.stream(s2):
                graphs[1].replay()
            c.run(s)
        torch.cuda.synchronize()
        for x, what in ((a, "first graph"), (b, "second graph"), (c, "eager")):
            x.check(f"round {k}, {what}")


def test_threads_on_the_per_thread_stream():
    """hipStreamPerThread is one handle for a stream per host thread."""
    import torch
    print("[gemm rows] two threads on the per-thread stream", flush=True)
    cases = [Layer(32, 8, 128, 2048, t, seed=80 + t) for t in (40, 130)]
    torch.cuda.synchronize()
    start, errors = threading.Barrier(2), []

    def work(c):
        try:
            start.wait(30)
            for _ in range(10):
                c.run(stream=2)               # hipStreamPerThread
            torch.cuda.synchronize()
        except Exception as e:                # reported by the main thread
            errors.append(e)
    threads = [threading.Thread(target=work, args=(c,)) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i, c in enumerate(cases):
        c.check(f"thread {i}")


def test_captured_on_a_stream_warmed_with_other_rows():
    """The first call on a stream makes all that later calls on it need: 1024
    rows (the GEMM library's), then 130 (this library's kernels) captured."""
    import torch
    print("[gemm rows] warmed with 1024 rows, captured with 130", flush=True)
    big, c = Layer(8, 2, 64, 1792, 1024, seed=10), Layer(8, 2, 64, 1792, 130, seed=11)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        big.run(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        c.run(s)
    for k in range(3):
        for b in c.bufs:
            b[:c.T].fill_(float(k))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        c.check(f"replay {k}")
