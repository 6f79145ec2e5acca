"""Adjacent redundancy on hidden states where the rows per wavefront change: calls below and from 4096 rows (layers
times the longest working set), rows of one and of several steps of a wavefront's lanes, short layers beside the longest,
against the float64 oracle.  The kernel sums in float64: half an ulp of values up to 1 is 6e-8."""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh,dtype", [(64, "bf16"), (512, "bf16"), (520, "bf16"), (256, "f32"), (260, "f32"), (1032, "f32")])
@pytest.mark.parametrize("sizes", [[1365, 1, 9], [1366, 4, 33], [4095], [4096]])
def test_rows_per_wavefront(sizes, dh, dtype):
    rng = np.random.default_rng([dh, sizes[0]])
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    top, keep, descs = max(sizes), [], []
    for n in sizes:
        x = torch.from_numpy(rng.standard_normal((n, dh), dtype=np.float32)).to("cuda", td)
        mod = (rng.random(n) < 0.4).astype(np.uint8)
        k = torch.zeros(2, n, 64, device="cuda", dtype=td)
        keep.append((x, mod, k, torch.from_numpy(mod).cuda()))
        descs.append(om.make_layer(None, k, k, keep[-1][3], 0, hidden=x))
    ctx = om.Context(len(sizes), 4, 2, 64, top + 700, top, dtype=om.BF16 if dtype == "bf16" else om.F32, sim=om.SIM_ADJ,
                     sim_source=om.SRC_HIDDEN, hidden_dim=dh)
    s = torch.full((len(sizes), 2, top + 700), 7.0, device="cuda")
    ctx.omnimem_redundancy(descs, s)
    got = s.cpu().numpy()
    ctx.close()
    for l, (n, (x, mod, *_)) in enumerate(zip(sizes, keep)):
        ref = orc.redundancy(x.float().cpu().numpy().astype(np.float64)[None], mod, "adj")
        assert np.abs(got[l, :, :n] - ref).max() <= 1e-7
        assert (got[l, :, n:] == 7.0).all()
