"""The library's per-stream scratch buffer on the GPU: two host threads calling on
one stream and on the stream handle that is each thread's own, and a captured graph whose stream's buffer grows afterwards.  Every
result is compared bit for bit with the same call made alone."""
import threading

import pytest
import torch

import paper_2312_06881_amd as dy

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [  # (n_in, n_out, n_dyad, tokens): split reduction, plain-block form, 4-wave tiles with splits
    (3072, 768, 4, 16),
    (2048, 3072, 4, 4097),
    (3072, 768, 4, 200),
]


def layer(case, seed):
    n_in, n_out, D, M = case
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device=DEV) * std).bfloat16()

    return normal(M, n_in), normal(D, n_out // D, n_in // D, std=0.02), normal(D, n_out // D, n_in // D, std=0.02)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_two_threads_on_one_stream(case):
    print("CASE threads", *case, flush=True)
    inputs = [layer(case, s) for s in (1, 2)]
    alone = [dy.forward(*i, variant="IT") for i in inputs]
    torch.cuda.synchronize()
    wrong = [torch.zeros((), dtype=torch.int64, device=DEV) for _ in inputs]

    def work(n):
        for _ in range(60):
            wrong[n] += (dy.forward(*inputs[n], variant="IT") != alone[n]).sum()

    threads = [threading.Thread(target=work, args=(n,)) for n in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert [int(w) for w in wrong] == [0, 0]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_each_threads_own_stream(case):
    n_in, n_out, D, M = case
    print("CASE own streams", *case, flush=True)
    inputs = [layer(case, s) for s in (4, 5)]
    alone = [dy.forward(*i, variant="IT") for i in inputs]
    out = [torch.zeros((20, M, n_out), dtype=torch.bfloat16, device=DEV) for _ in inputs]
    torch.cuda.synchronize()
    codes = [[], []]

    def work(n):
        x, w1, w2 = inputs[n]
        for y in out[n]:
            codes[n].append(dy.dyad_forward(dy.IT, n_in, n_out, D, M, dy.BF16, x.data_ptr(), w1.data_ptr(),
                                            w2.data_ptr(), None, dy.ACT_NONE, y.data_ptr(), None,
                                            2))   # hipStreamPerThread
        torch.cuda.synchronize()

    threads = [threading.Thread(target=work, args=(n,)) for n in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert codes == [[0] * 20] * 2
    for y, a in zip(out, alone):
        assert torch.equal(y, a.expand_as(y))


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_graph_keeps_its_buffer(case):
    n_in, n_out, D, M = case
    print("CASE graph", *case, flush=True)
    x, w1, w2 = layer(case, 3)
    s, other = torch.cuda.Stream(DEV), torch.cuda.Stream(DEV)
    y = torch.empty((M, n_out), dtype=torch.bfloat16, device=DEV)

    def call(stream, x, y, tokens):
        rc = dy.dyad_forward(dy.IT, n_in, n_out, D, tokens, dy.BF16, x.data_ptr(), w1.data_ptr(), w2.data_ptr(), None,
                             dy.ACT_NONE, y.data_ptr(), None, stream.cuda_stream)
        assert rc == 0

    torch.cuda.synchronize()
    call(s, x, y, M)                     # the stream has its buffer
    s.synchronize()
    eager = y.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        call(s, x, y, M)
    # the buffer grows on its stream, and another stream takes one of the old size
    more = 4 * M
    x4, y4 = x.repeat(4, 1), torch.empty((more, n_out), dtype=torch.bfloat16, device=DEV)
    torch.cuda.synchronize()
    call(s, x4, y4, more)
    y_other = torch.empty_like(y)
    call(other, x, y_other, M)
    torch.cuda.synchronize()
    expect = y4.clone()
    for _ in range(4):
        y.zero_()
        y4.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):   # eager work of the other stream beside the replay
            call(other, x4, y4, more)
        with torch.cuda.stream(s):
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager)
        assert torch.equal(y4, expect)
