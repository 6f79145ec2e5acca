"""Adjacent redundancy (Eq. 7 as printed) at the edges of its row groups.

The kernel takes groups of six or eight consecutive positions of the
modality lists: working sets around multiples of a group, modalities that
start, end or alternate inside one, lone rows, strided rows and rows whose
pieces do not fill a wavefront, against the float64 oracle.  The kernel sums
in float64, so its result is the oracle's rounded to float32 (half an ulp of
values up to 1 is 6e-8).
"""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu

MASKS = {
    "visual": lambda n, rng: np.zeros(n),
    "audio": lambda n, rng: np.ones(n),
    "alternating": lambda n, rng: np.arange(n) % 2,
    "one-audio": lambda n, rng: (np.arange(n) == n // 2),
    "random": lambda n, rng: rng.random(n) < 0.4,
}


def _rows(rng, *shape):
    x = rng.standard_normal(shape, dtype=np.float32)
    x[..., 0, :] = 0.0  # a zero row: cosine 0
    return x


@pytest.mark.parametrize("mask", sorted(MASKS))
@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (64, "bf16"), (128, "f32"), (64, "f32")])
@pytest.mark.parametrize("n", [1, 2, 6, 7, 8, 9, 97, 129, 1025])
def test_adjacent_rows_match_the_oracle(n, d, dtype, mask):
    rng = np.random.default_rng([n, d, len(mask)])
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    mod = MASKS[mask](n, rng).astype(np.uint8)
    # rows strided inside a wider buffer
    wide = torch.from_numpy(_rows(rng, 2, n, d + 16)).to("cuda", td)
    v = wide[:, :, :d]
    m = torch.from_numpy(mod).cuda()
    ctx = om.Context(1, 4, 2, d, n + 5, n, dtype=om.BF16 if dtype == "bf16" else om.F32, sim=om.SIM_ADJ)
    s = torch.full((1, 2, n + 5), 7.0, device="cuda")
    ctx.omnimem_redundancy([om.make_layer(None, v, v, m, 0)], s)
    got = s.cpu().numpy()
    ref = orc.redundancy(v.float().cpu().numpy().astype(np.float64), mod, "adj")
    assert np.abs(got[0, :, :n] - ref).max() <= 1e-7
    assert (got[0, :, n:] == 7.0).all()  # entries past N untouched
    ctx.close()


@pytest.mark.parametrize("n,dh,dtype", [(1, 64, "bf16"), (9, 200, "f32"), (33, 520, "bf16"), (70, 4, "f32"), (65, 1024, "bf16")])
def test_adjacent_hidden_rows_match_the_oracle(n, dh, dtype):
    rng = np.random.default_rng([n, dh])
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    mod = MASKS["random"](n, rng).astype(np.uint8)
    h = torch.from_numpy(_rows(rng, n, dh)).to("cuda", td)
    k = torch.zeros(2, n, 64, device="cuda", dtype=td)
    m = torch.from_numpy(mod).cuda()
    ctx = om.Context(1, 4, 2, 64, n, n, dtype=om.BF16 if dtype == "bf16" else om.F32, sim=om.SIM_ADJ,
                     sim_source=om.SRC_HIDDEN, hidden_dim=dh)
    s = torch.zeros((1, 2, n), device="cuda")
    ctx.omnimem_redundancy([om.make_layer(None, k, k, m, 0, hidden=h)], s)
    got = s.cpu().numpy()[0]
    ref = orc.redundancy(h.float().cpu().numpy().astype(np.float64)[None], mod, "adj")[0]
    assert np.abs(got - ref[None]).max() <= 1e-7
    ctx.close()
