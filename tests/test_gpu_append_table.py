"""The layer table that an append leaves on the device serves the calls that follow it on the same stream; a call on
another stream or inside a graph capture, and one whose descriptors differ, gets a table of its own.  Every route
gives what a fresh context gives on the same buffers, bit for bit."""
import pytest
import torch

from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", ["same-stream", "other-stream", "captured", "captured-append", "other-rows"])
@pytest.mark.parametrize("layers", [1, 28])  # one workgroup and several copy the table
def test_calls_after_an_append(route, layers):
    h_q, h_kv, d, cache, chunk = 4, 2, 64, 70, 45
    n = cache + chunk
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v = rnd(layers, h_q, chunk, d), rnd(layers, h_kv, n, d), rnd(layers, h_kv, n, d)
    ck, cv = rnd(layers, h_kv, chunk, d), rnd(layers, h_kv, chunk, d)
    mod = torch.zeros(layers, n, dtype=torch.uint8, device="cuda")
    cmod = (torch.arange(chunk, device="cuda") % 3 == 0).to(torch.uint8)

    def table(rows):
        return [om.make_layer(q[l], k[l], v[l], mod[l], rows - chunk, 0.1, n=rows) for l in range(layers)]

    chunks = [om.make_chunk(ck[l], cv[l], cmod) for l in range(layers)]
    ctx = om.Context(layers, h_q, h_kv, d, n, chunk)
    a, s = (torch.zeros(layers, h_kv, n, device="cuda") for _ in range(2))
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    rows = n - 7 if route == "other-rows" else n
    desc = table(rows)

    def calls(stream):
        ctx.omnimem_score(desc, a, None, stream)
        ctx.omnimem_redundancy(desc, s, stream)

    if route == "captured-append":
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=one):
            ctx.omnimem_append(table(n), chunks, one)
        calls(one)                 # its table may not be the append's: that copy has not run
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        calls(one)
    else:
        ctx.omnimem_append(table(n), chunks, one)
        if route == "captured":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=one):
                calls(one)
            for _ in range(2):
                a.fill_(-7)
                s.fill_(-7)
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
        elif route == "other-stream":
            two.wait_stream(one)
            calls(two)
        else:
            calls(one)
    torch.cuda.synchronize()
    assert torch.equal(k[:, :, cache:], ck) and torch.equal(v[:, :, cache:], cv)
    assert all(torch.equal(mod[l, cache:], cmod) for l in range(layers))
    fresh = om.Context(layers, h_q, h_kv, d, n, chunk)
    a2, s2 = (torch.zeros(layers, h_kv, n, device="cuda") for _ in range(2))
    fresh.omnimem_score(desc, a2)
    fresh.omnimem_redundancy(desc, s2)
    torch.cuda.synchronize()
    assert torch.equal(a[:, :, :rows], a2[:, :, :rows]) and torch.equal(s[:, :, :rows], s2[:, :, :rows])
    for c in (ctx, fresh):
        c.close()
