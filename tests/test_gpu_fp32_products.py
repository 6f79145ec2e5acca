"""fp32 inputs: products on the matrix cores from three bf16 parts per value.

Working sets around the tile and block edges of the score and Gram passes
(32-row register blocks, 64-row tiles, 256-row workgroups), and rows of
scales from 2^-39 to 2^30, against the float64 oracle (what the parts lose or
cannot hold: test_gpu_fp32_bias.py, test_gpu_fp32_range.py).  An fp32 sum of d products carries about sqrt(d) / 2
roundings of 2^-24 of its size, and the part products left out less than one,
under 6e-7 at d = 128 relative to the norms; the importance adds the
exponential's and the sum's own roundings.
"""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


def _run(q, k, mod, n_cache, **options):
    h_q, c, d = q.shape
    h_kv, n, _ = k.shape
    ctx = om.Context(1, h_q, h_kv, d, n + 3, max(c, 1), dtype=om.F32, **options)
    dq, dk = torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()
    m = torch.from_numpy(mod).cuda()
    lay = [om.make_layer(dq, dk, dk, m, n_cache)]
    a = torch.full((1, h_kv, n + 3), 7.0, device="cuda")
    s = torch.full((1, h_kv, n + 3), 7.0, device="cuda")
    ctx.omnimem_score(lay, a)
    ctx.omnimem_redundancy(lay, s)
    torch.cuda.synchronize()
    ctx.close()
    a, s = a.cpu().numpy()[0], s.cpu().numpy()[0]
    assert (a[:, n:] == 7.0).all() and (s[:, n:] == 7.0).all()
    return a[:, :n].astype(np.float64), s[:, :n].astype(np.float64)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_cache,c", [(0, 1), (0, 64), (1, 31), (31, 33), (63, 65), (255, 1), (200, 57), (300, 257),
                                       (1000, 129)])
def test_scores_and_redundancy_at_tile_edges(n_cache, c, d, causal):
    rng = np.random.default_rng([n_cache, c, d])
    n = n_cache + c
    q = rng.standard_normal((4, c, d), dtype=np.float32)
    k = rng.standard_normal((2, n, d), dtype=np.float32)
    mod = (rng.random(n) < 0.3).astype(np.uint8)
    a, s = _run(q, k, mod, n_cache, causal=causal)
    a_ref = orc.attention_importance(q.astype(np.float64), k.astype(np.float64), n_cache, 1.0 / np.sqrt(d),
                                     causal=bool(causal))
    s_ref = orc.redundancy(k.astype(np.float64), mod, "max")
    assert np.abs(a - a_ref).max() <= 3e-6 * np.abs(a_ref).max()
    assert np.linalg.norm(a - a_ref) <= 1e-6 * np.linalg.norm(a_ref)
    assert np.abs(s - s_ref).max() <= 6e-7


@pytest.mark.parametrize("d", [64, 128])
def test_parts_are_exact_at_every_scale(d):
    rng = np.random.default_rng(d)
    n = 333
    k = rng.standard_normal((2, n, d), dtype=np.float32)
    k *= np.exp2(rng.integers(-30, 30, size=(2, n, 1))).astype(np.float32)   # rows of very different norms
    k[:, :, : d // 2] *= np.float32(2.0**-9)                                   # and elements within a row
    k[0, 5] = 0.0
    mod = (np.arange(n) % 3 == 0).astype(np.uint8)
    q = np.zeros((4, 1, d), dtype=np.float32)
    _, s = _run(q, k, mod, n - 1)
    assert np.abs(s - orc.redundancy(k.astype(np.float64), mod, "max")).max() <= 6e-7
