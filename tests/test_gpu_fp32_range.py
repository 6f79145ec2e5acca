"""fp32 values that three bf16 parts do not serve: infinities, NaN, and magnitudes outside [2^-50, 2^60).

A row block or a head with one is multiplied as fp32.  Scores: a key that
is -inf in one channel has no weight, a NaN key spoils what attends to it and nothing else.  Redundancy: rows of
extreme norms have ordinary cosines, and a row with an infinity or NaN does not touch the others'.  Tolerances as for
ordinary fp32 rows (a dot product of d terms, sqrt(d) / 2 roundings of 2^-24).
"""
import numpy as np
import pytest
import torch

from oracle import omnimem_oracle as orc
from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


def _scores(q, k, n_cache, causal):
    h_q, c, d = q.shape
    h_kv, n, _ = k.shape
    ctx = om.Context(1, h_q, h_kv, d, n + 3, c + 2, dtype=om.F32, causal=causal)
    dq, dk = torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()
    a = torch.full((1, h_kv, n + 3), 7.0, device="cuda")
    lse = torch.zeros(1, h_q, c + 2, device="cuda")
    ctx.omnimem_score([om.make_layer(dq, dk, dk, torch.zeros(n, dtype=torch.uint8, device="cuda"), n_cache)], a, lse)
    a, lse = a[0].double().cpu().numpy(), lse[0].double().cpu().numpy()
    ctx.close()
    assert (a[:, n:] == 7.0).all()
    return a[:, :n], lse[:, :c]


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_cache,c,at", [(0, 1, 0), (50, 40, 3), (50, 40, 60), (300, 257, 299), (1000, 300, 640)])
def test_infinite_and_nan_keys(n_cache, c, at, d, causal):
    rng = np.random.default_rng([n_cache, at, d])
    n = n_cache + c
    q = rng.standard_normal((4, c, d), dtype=np.float32)
    k = rng.standard_normal((2, n, d), dtype=np.float32)
    q[:2, :, 3] = 1.5                      # exact in 8 bits: the lower parts are zero
    q[:2, ::2, 3] = np.float32(1.2345678)  # and not
    k0 = k.copy()
    ref = orc.attention_importance(q.astype(np.float64), k0.astype(np.float64), n_cache, 1.0 / np.sqrt(d),
                                   causal=bool(causal))
    tol = 3e-6 * np.abs(ref).max()
    if n > 1:
        k[0, at, 3] = -np.inf
        a, lse = _scores(q, k, n_cache, causal)
        expect = np.zeros(n)
        for h in range(2):
            s = (q[h].astype(np.float64) @ k0[0].astype(np.float64).T) / np.sqrt(d)
            s[:, at] = -np.inf
            if causal:
                s[np.arange(n)[None, :] > n_cache + np.arange(c)[:, None]] = -np.inf
            z = np.log(np.exp(s).sum(1))
            assert np.abs(lse[h] - z).max() <= 1e-5
            expect += np.exp(s - z[:, None]).sum(0)
        assert a[0, at] == 0.0
        assert np.abs(a[0] - expect).max() <= tol
        assert np.abs(a[1] - ref[1]).max() <= tol
    k = k0.copy()
    k.view(np.uint32)[0, at, 3] = 0x7F800001  # a NaN with a bit below bf16's
    a, lse = _scores(q, k, n_cache, causal)
    sees = (np.arange(c) + n_cache >= at) if causal else np.ones(c, bool)
    assert np.isnan(lse[:2][:, sees]).all() and np.isfinite(lse[:2][:, ~sees]).all()
    assert np.isnan(a[0, : n_cache + 1]).all()
    assert np.abs(a[1] - ref[1]).max() <= tol


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("source", [om.SRC_VALUES, om.SRC_KEYS])
@pytest.mark.parametrize("n", [2, 70, 333])
@pytest.mark.parametrize("kind", ["tiny", "huge", "mixed", "infinite", "nan"])
def test_redundancy_of_extreme_rows(kind, n, source, d):
    rng = np.random.default_rng([n, d, len(kind)])
    x = rng.standard_normal((2, n, d), dtype=np.float32)
    x[:, n // 2] = x[:, 0] + np.float32(0.01) * x[:, n // 2]
    odd = n // 2
    if kind == "tiny":
        x[0, odd] = np.copysign(np.maximum(np.abs(x[0, odd]), 2.0**-8), x[0, odd])
        x[0, odd] *= np.float32(2.0**-115)  # (normal numbers)
    elif kind == "huge":
        x[0, odd] *= np.float32(2.0**100)
    elif kind == "mixed":
        x[0] *= np.exp2(rng.integers(-55, 55, size=(n, 1))).astype(np.float32)
    mod = (np.arange(n) % 4 == 3).astype(np.uint8)
    ref = orc.redundancy(x.astype(np.float64), mod, "max")
    keep = np.ones(n, bool)
    if kind in ("infinite", "nan"):
        x[0, odd, 5] = np.inf if kind == "infinite" else np.nan
        keep[odd] = False
        rest = orc.redundancy(x[:, keep].astype(np.float64), mod[keep], "max")
        ref[0, keep] = rest[0]
    t = torch.from_numpy(x).cuda()
    other = torch.zeros_like(t)
    ctx = om.Context(1, 4, 2, d, n + 3, n, dtype=om.F32, sim_source=source)
    s = torch.full((1, 2, n + 3), 7.0, device="cuda")
    kv = (other, t) if source == om.SRC_VALUES else (t, other)
    ctx.omnimem_redundancy([om.make_layer(None, *kv, torch.from_numpy(mod).cuda(), 0)], s)
    got = s[0].double().cpu().numpy()
    ctx.close()
    assert (got[:, n:] == 7.0).all()
    assert np.abs(got[0, :n][keep] - ref[0][keep]).max() <= 6e-7
    assert np.abs(got[1, :n] - ref[1]).max() <= 6e-7


@pytest.mark.parametrize("d", [64, 128])
def test_redundancy_of_many_heads(d):
    # 9 layers x 2 heads (the work dealt to the eight XCDs); a tiny row, an infinity and a NaN in some of them
    rng = np.random.default_rng(d)
    layers, n = 9, 300
    x = rng.standard_normal((layers, 2, n, d), dtype=np.float32)
    x[:, :, 250] = x[:, :, 3] + np.float32(0.01) * x[:, :, 250]
    mod = (np.arange(n) % 4 == 3).astype(np.uint8)
    refs = [orc.redundancy(x[l].astype(np.float64), mod, "max") for l in range(layers)]
    x[2, 1, 100] *= np.float32(2.0**-70)
    x[4, 0, 7, 0], x[7, 1, 8, 1] = np.inf, np.nan
    keep = np.ones((layers, 2, n), bool)
    keep[4, 0, 7], keep[7, 1, 8] = False, False
    for l, g in ((4, 0), (7, 1)):
        rows = keep[l, g]
        refs[l][g, rows] = orc.redundancy(x[l, g, rows][None].astype(np.float64), mod[rows], "max")[0]
    t, m = torch.from_numpy(x).cuda(), torch.from_numpy(mod).cuda()
    ctx = om.Context(layers, 4, 2, d, n, n, dtype=om.F32)
    s = torch.zeros(layers, 2, n, device="cuda")
    ctx.omnimem_redundancy([om.make_layer(None, t[l], t[l], m, 0) for l in range(layers)], s)
    got = s.double().cpu().numpy()
    ctx.close()
    assert np.abs(got - np.stack(refs))[keep].max() <= 6e-7
