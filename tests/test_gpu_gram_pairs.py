"""All-pairs redundancy of bf16 rows where its share of the work is cut.

The kernel cuts the cost of all segments (layer, KV head, modality) evenly
over its workgroups: segments around multiples of a tile (64 rows) and of a
register block (256 rows), rows of one to six tiles, shares that end inside
a row of work or pass over empty modalities, more layers than a wavefront has lanes,
more work than one tile per workgroup.  Against the float64 oracle; a dot
product of d terms accumulated in float32 and two scalings are within
(d + 4) 2^-24 of a cosine.
"""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu

CASES = {
    "edges": ([1, 2, 63, 64, 65, 128, 255, 256, 257, 321, 385, 513], 2),
    "many-layers": ([(37 * i) % 150 + 1 for i in range(130)], 1),
    "one-layer": ([2311], 1),
    "uneven": ([1500, 3, 900, 64, 1], 5),
}


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("visual", [0.0, 0.7, 1.0])
@pytest.mark.parametrize("name", sorted(CASES))
def test_all_pairs_match_the_oracle(name, visual, d):
    sizes, heads = CASES[name]
    rng = np.random.default_rng([len(name), d, int(10 * visual)])
    top = max(sizes)
    descs, refs, keep = [], [], []
    for n in sizes:
        x = rng.standard_normal((heads, n, d), dtype=np.float32)
        x[:, n // 2] = 0.5 * x[:, 0]  # a near-duplicate
        v = torch.from_numpy(x).to("cuda", torch.bfloat16)
        mod = (rng.random(n) >= visual).astype(np.uint8)
        m = torch.from_numpy(mod).cuda()
        keep.append((v, m))
        descs.append(om.make_layer(None, v, v, m, 0))
        refs.append(orc.redundancy(v.float().cpu().numpy().astype(np.float64), mod, "max"))
    ctx = om.Context(len(sizes), 2 * heads, heads, d, top, top, sim=om.SIM_MAX)
    s = torch.full((len(sizes), heads, top), 7.0, device="cuda")
    for _ in range(2):  # the second pass finds the first one's maxima in the workspace
        ctx.omnimem_redundancy(descs, s)
        got = s.cpu().numpy()
        for l, (n, ref) in enumerate(zip(sizes, refs)):
            assert np.abs(got[l, :, :n] - ref).max() <= (d + 4) * 2.0**-24, (l, n)
            assert (got[l, :, n:] == 7.0).all()
    ctx.close()
