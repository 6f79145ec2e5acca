"""In-place compaction whose staging workgroups take several tiles each (many (layer, KV head) pairs, a long run of rows
that move back): the kept rows of the out-of-place call, bit for bit."""
import pytest
import torch

from paper_2606_07577_amd import omnimem as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("layers,h_kv,kept_audio,reserve", [
    (64, 4, 650, 700),   # four workgroups per pair, eleven tiles, the last of ten slots
    (64, 4, 513, 513),   # the run ends one slot into a tile, at the reserve
    (128, 2, 64, 64),    # one whole tile
    (64, 4, 650, 600),   # longer than the reserve: nothing moves, and the call says so
])
def test_long_runs_of_many_pairs(dtype, d, layers, h_kv, kept_audio, reserve):
    n, audio = 1400, 700     # the audio rows first: every kept one moves behind the visual rows
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(3)
    k, v = (torch.randn(layers, h_kv, n, d, generator=g, device="cuda").to(td) for _ in range(2))
    a = torch.rand(layers, h_kv, n, generator=g, device="cuda") + 0.1
    s = torch.rand(layers, h_kv, n, generator=g, device="cuda")
    mod = (torch.arange(n, device="cuda") < audio).to(torch.uint8)
    budgets = torch.tensor([[n - audio, kept_audio]] * layers, dtype=torch.int32, device="cuda")
    ctx = om.Context(layers, h_kv, h_kv, d, n, n, dtype=om.BF16 if dtype == "bf16" else om.F32,
                     inplace_stage_rows=reserve)

    def call(k, v, ko, vo):
        idx = torch.full((layers, h_kv, n), -1, dtype=torch.int32, device="cuda")
        ctx.omnimem_select_compact([om.make_layer(None, k[l], v[l], mod, 0, k_out=ko[l], v_out=vo[l])
                                    for l in range(layers)], a, s, budgets, idx)
        torch.cuda.synchronize()
        return idx

    ko, vo, ki, vi = torch.zeros_like(k), torch.zeros_like(v), k.clone(), v.clone()
    idx = call(k, v, ko, vo)
    assert torch.equal(call(ki, vi, ki, vi), idx)
    m = n - audio + kept_audio
    if reserve < kept_audio:
        with pytest.raises(om.OmnimemError):
            ctx.omnimem_inplace_status()
        assert torch.equal(ki, k) and torch.equal(vi, v)
    else:
        assert ctx.omnimem_inplace_status() == 0
        assert torch.equal(ki[:, :, :m], ko[:, :, :m]) and torch.equal(vi[:, :, :m], vo[:, :, :m])
    ctx.close()
