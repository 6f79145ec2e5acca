"""Score passes that cut long rows into many segments: few rows (a short chunk, one layer, few heads) over all of the
chip, at the edges of the plan -- one tile per chunk, rows longer than the most segments they may have, a call far below its
context's capacity, a layer whose normaliser is given between two that compute theirs.  Against 64 bits."""
import math

import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h_q,h_kv,d,cache,chunk,given,cap_tokens,cap_chunk", [
    (1, 1, 64, 0, 1, (), 1, 1),                  # one tile
    (2, 1, 128, 63, 65, (), 128, 65),            # a row of two tiles, a second query tile of one row
    (1, 1, 64, 4500, 40, (), 4540, 40),          # 71 tiles: more than a row's segments
    (5, 1, 128, 1000, 300, (), 1300, 300),       # two blocks, the second of 44 queries
    (4, 2, 64, 700, 129, (1,), 5000, 2000),      # below capacity, a given normaliser between two layers
    (2, 2, 64, 10, 2100, (), 2110, 2100),        # long query rows: many column-sum segments
])
def test_few_rows_many_segments(dtype, h_q, h_kv, d, cache, chunk, given, cap_tokens, cap_chunk):
    layers, n = (3 if given else 1), cache + chunk
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(11)
    q = torch.randn(layers, h_q, chunk, d, generator=g).to(td)
    k = torch.randn(layers, h_kv, n, d, generator=g).to(td)
    scale = float(np.float32(1.7 / math.sqrt(d)))
    refs = []
    for l in range(layers):
        kk = k[l].double().repeat_interleave(h_q // h_kv, 0)
        s = (q[l].double() @ kk.transpose(1, 2)) * scale
        s.masked_fill_(torch.arange(n)[None, :] > cache + torch.arange(chunk)[:, None], -math.inf)
        refs.append(torch.logsumexp(s, 2))
    dev = [dict(q=q[l].cuda(), k=k[l].cuda(), z=refs[l].float().cuda() if l in given else None) for l in range(layers)]
    mod = torch.zeros(n, dtype=torch.uint8, device="cuda")
    descs = [om.make_layer(x["q"], x["k"], x["k"], mod, cache, scale, x["z"]) for x in dev]
    ctx = om.Context(layers, h_q, h_kv, d, cap_tokens, cap_chunk, dtype=om.BF16 if dtype == "bf16" else om.F32)
    a = torch.full((layers, h_kv, cap_tokens), -1.0, device="cuda")
    lse = torch.full((layers, h_q, cap_chunk), -1.0, device="cuda")
    for _ in range(2):
        ctx.omnimem_score(descs, a, lse)
    torch.cuda.synchronize()
    for l in range(layers):
        ref = orc.attention_importance(q[l].double().numpy(), k[l].double().numpy(), cache, scale)
        # probabilities of fp32 exponents (relative 2^-24 times |exponent| < 40) and fp32 sums
        assert np.allclose(a[l, :, :n].cpu().numpy(), ref, rtol=1e-5, atol=1e-5 * ref.mean())
        # a log-sum-exp below 40: a few roundings of 2^-24 of it
        assert np.allclose(lse[l, :, :chunk].cpu().numpy(), refs[l].numpy(), rtol=0, atol=2e-5)
        assert (a[l, :, n:] == -1).all()
    ctx.close()
