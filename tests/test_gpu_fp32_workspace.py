"""An fp32 context for which there is no memory for rows as bf16 parts (here: capacities whose parts pass any GPU's
memory) is created all the same, and its scores and redundancy come from the rows as they are: the oracle's within the
tolerances of fp32 sums of d products."""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,source", [(128, om.SRC_VALUES), (64, om.SRC_KEYS)])
def test_context_without_room_for_parts(d, source):
    cap = (1 << 30) * 64 // d  # 6 d bytes a row: 412 GB
    rng = np.random.default_rng(d)
    ctx = om.Context(1, 1, 1, d, cap, 300, dtype=om.F32, sim_source=source)
    a, s = (torch.zeros(1, 1, cap, device="cuda") for _ in range(2))
    for n_cache, c in [(0, 1), (70, 65), (900, 300)]:
        n = n_cache + c
        q, k = rng.standard_normal((1, c, d), dtype=np.float32), rng.standard_normal((1, n, d), dtype=np.float32)
        v = rng.standard_normal((1, n, d), dtype=np.float32)
        mod = (rng.random(n) < 0.3).astype(np.uint8)
        dq, dk, dv, dm = (torch.from_numpy(x).cuda() for x in (q, k, v, mod))
        lay = [om.make_layer(dq, dk, dv, dm, n_cache)]
        ctx.omnimem_score(lay, a)
        ctx.omnimem_redundancy(lay, s)
        a_ref = orc.attention_importance(q.astype(np.float64), k.astype(np.float64), n_cache, 1.0 / np.sqrt(d))
        s_ref = orc.redundancy((v if source == om.SRC_VALUES else k).astype(np.float64), mod, "max")
        assert np.abs(a[0, :, :n].double().cpu().numpy() - a_ref).max() <= 3e-6 * a_ref.max()
        assert np.abs(s[0, :, :n].double().cpu().numpy() - s_ref).max() <= 6e-7
    ctx.close()
