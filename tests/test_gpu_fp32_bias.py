"""fp32 products from three bf16 parts lose nothing systematic.

One key per query, so that the log-sum-exp is the scaled dot product itself:
rows whose significands leave the largest rests (just above a power of two,
all lower bits set), rows with near-copies of themselves (all products of one
sign), one channel that carries the sum, and ordinary ones, against 64 bits.
A dot product of d fp32 terms is within (sqrt(d) / 2 + 2) 2^-24 of the norms
here (sqrt(d) / 2 for its additions, one for the products left out, one for the
factors log2 e and ln 2), and its mean error over 2048 of them far below one
2^-24: a loss of one sign in every product would show there.
"""
import math

import numpy as np
import pytest
import torch

from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu

L, H, HKV = 32, 64, 8


def _rows(kind, d, rng):
    q = rng.standard_normal((L, H, d), dtype=np.float32)
    k = rng.standard_normal((L, HKV, d), dtype=np.float32)
    if kind == "awkward":
        q = np.full_like(q, np.float32(1 + 65535 * 2.0**-23))
        k = np.full_like(k, np.float32(1 + 65535 * 2.0**-23))
    elif kind == "near":
        k = k.astype(np.float32)
        q = np.repeat(k, H // HKV, 1) + np.float32(0.05) * q
    elif kind == "late-channel":
        q[..., -1] *= 1000
    return q.astype(np.float32), k


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kind", ["awkward", "near", "late-channel", "ordinary"])
def test_dot_products_against_64_bits(kind, d):
    rng = np.random.default_rng([d, len(kind)])
    q, k = _rows(kind, d, rng)
    dq, dk = torch.from_numpy(q).cuda().reshape(L, H, 1, d), torch.from_numpy(k).cuda().reshape(L, HKV, 1, d)
    mod = torch.zeros(1, dtype=torch.uint8, device="cuda")
    ctx = om.Context(L, H, HKV, d, 1, 1, dtype=om.F32)
    a = torch.zeros(L, HKV, 1, device="cuda")
    lse = torch.zeros(L, H, 1, device="cuda")
    ctx.omnimem_score([om.make_layer(dq[l], dk[l], dk[l], mod, 0, 1.0) for l in range(L)], a, lse)
    got = lse[..., 0].double().cpu().numpy()
    ctx.close()
    # the factors as the library has them: log2 e and ln 2 in fp32
    factor = float(np.float32(1 / math.log(2))) * float(np.float32(math.log(2)))
    kk = np.repeat(k, H // HKV, 1).astype(np.float64)
    ref = (q.astype(np.float64) * kk).sum(2) * factor
    err = (got - ref) / (np.linalg.norm(q.astype(np.float64), axis=2) * np.linalg.norm(kk, axis=2)) * 2.0**24
    assert np.abs(err).max() <= math.sqrt(d) / 2 + 2
    assert abs(err.mean()) <= 0.3
