"""Layer tables and graph captures: a captured call's graph holds its own table.

A table whose copy was only recorded is never taken for one on the device; a
graph replays right after any number of other tables have been used, and
leaves alone the table that calls outside it will use next; an append whose
descriptors are those of the append before finds that one's table.  Every
call's result is that of a fresh context on the same buffers, bit for bit.
"""
import pytest
import torch

from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu

H_Q, H_KV, D, CACHE, CHUNK = 4, 2, 64, 70, 45
N = CACHE + CHUNK


class Case:
    def __init__(self, layers, seed=5):
        g = torch.Generator(device="cuda").manual_seed(seed)
        rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
        self.layers = layers
        self.q, self.k, self.v = rnd(layers, H_Q, CHUNK, D), rnd(layers, H_KV, N, D), rnd(layers, H_KV, N, D)
        self.ck, self.cv = rnd(layers, H_KV, CHUNK, D), rnd(layers, H_KV, CHUNK, D)
        self.mod = (torch.arange(N, device="cuda") % 3 == 0).to(torch.uint8).repeat(layers, 1)
        self.cmod = (torch.arange(CHUNK, device="cuda") % 2).to(torch.uint8)
        self.ctx = om.Context(layers, H_Q, H_KV, D, N, CHUNK)
        self.a, self.s = (torch.zeros(layers, H_KV, N, device="cuda") for _ in range(2))
        self.chunks = [om.make_chunk(self.ck[l], self.cv[l], self.cmod) for l in range(layers)]

    def table(self, rows=N):
        return [om.make_layer(self.q[l], self.k[l], self.v[l], self.mod[l], rows - CHUNK, 0.1, n=rows)
                for l in range(self.layers)]

    def calls(self, stream, rows=N):
        self.ctx.omnimem_score(self.table(rows), self.a, None, stream)
        self.ctx.omnimem_redundancy(self.table(rows), self.s, stream)

    def append(self, stream):
        self.ctx.omnimem_append(self.table(), self.chunks, stream)

    def check(self, rows=N):
        torch.cuda.synchronize()
        fresh = om.Context(self.layers, H_Q, H_KV, D, N, CHUNK)
        a, s = torch.zeros_like(self.a), torch.zeros_like(self.s)
        fresh.omnimem_score(self.table(rows), a)
        fresh.omnimem_redundancy(self.table(rows), s)
        torch.cuda.synchronize()
        fresh.close()
        assert torch.equal(self.a[:, :, :rows], a[:, :, :rows]) and torch.equal(self.s[:, :, :rows], s[:, :, :rows])
        self.a.fill_(-7)
        self.s.fill_(-7)
        torch.cuda.synchronize()


def _capture(stream, work):
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        work()
    torch.cuda.synchronize()
    return graph


@pytest.mark.parametrize("layers", [1, 8, 9, 28])  # a table in one, two and four kernels' arguments
@pytest.mark.parametrize("append_first", [False, True])
def test_calls_before_the_first_replay(append_first, layers):
    c, one = Case(layers), torch.cuda.Stream()

    def work():
        if append_first:
            c.append(one)
        c.calls(one)

    graph = _capture(one, work)
    c.calls(one)      # equal descriptors: the recorded copy has not run
    c.check()
    graph.replay()
    torch.cuda.synchronize()
    if append_first:
        assert torch.equal(c.k[:, :, CACHE:], c.ck) and torch.equal(c.mod[:, CACHE:], c.cmod.expand(layers, -1))
    c.check()
    c.ctx.close()


@pytest.mark.parametrize("layers", [1, 28])
@pytest.mark.parametrize("warm", [False, True])  # the table in use before the capture, too
def test_replays_between_other_tables(warm, layers):
    c, one = Case(layers), torch.cuda.Stream()
    one.wait_stream(torch.cuda.current_stream())
    if warm:
        c.append(one)
        c.calls(one)
    graph = _capture(one, lambda: (c.append(one), c.calls(one)))
    other = _capture(one, lambda: c.calls(one, N - 3))
    for rep in range(3):
        for i in range(20):                     # more tables than a ring of 16 holds
            c.calls(one, N - 1 - i % 20)
        c.check(N - 20)
        c.k[:, :, CACHE:] = 0                   # the replay appends again
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c.k[:, :, CACHE:], c.ck) and torch.equal(c.v[:, :, CACHE:], c.cv)
        c.check()
        c.calls(one, N - 20)                    # the last table used outside the graph
        c.check(N - 20)
        other.replay()
        c.check(N - 3)
    c.ctx.close()


@pytest.mark.parametrize("layers", [1, 28])
def test_equal_appends_share_a_table(layers):
    c, one = Case(layers), torch.cuda.Stream()
    torch.cuda.synchronize()
    c.ctx.omnimem_profile(True)
    for value in (1.0, 2.0, 3.0):
        with torch.cuda.stream(one):
            c.ck.fill_(value)
        c.append(one)
        c.calls(one)
    torch.cuda.synchronize()
    assert (c.k[:, :, CACHE:] == 3).all()
    assert c.ctx.omnimem_profile_report()["layer_table"][0] == 1
    c.check()
    c.ctx.omnimem_profile(True)
    c.chunks = [om.make_chunk(c.cv[l], c.ck[l], c.cmod) for l in range(layers)]  # other chunk rows: another table
    c.append(one)
    c.append(one)
    torch.cuda.synchronize()
    assert torch.equal(c.k[:, :, CACHE:], c.cv)
    assert c.ctx.omnimem_profile_report()["layer_table"][0] == 1
    c.ctx.close()
