"""Adapter operands that are copied, transposed and summed eight or four elements at a time, and one by one where ranks, widths or addresses do not allow it."""
import pytest
import torch

from paper_2506_03077_amd import binding as sb

pytestmark = pytest.mark.gpu

MATS = ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown")


def _shifted(t, by):
    """The same values, `by` elements behind a 16-byte boundary."""
    flat = torch.zeros(t.numel() + by, dtype=t.dtype, device=t.device)
    flat[by:] = t.reshape(-1)
    return flat[by:].view(t.shape)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rank,hidden,mlp", [(8, 256, 512), (12, 256, 512), (1, 64, 172), (3, 72, 90), (40, 128, 100)])
def test_the_same_at_any_address(rank, hidden, mlp, dtype):
    """Gradients do not depend on where the adapters and their gradients lie, so the forms for one element and for several agree bit for bit."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(rank)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    hq, hkv, dh, T = 4, 2, 16, 70
    dims = dict(wq=(hq * dh, hidden), wk=(hkv * dh, hidden), wv=(hkv * dh, hidden), wo=(hidden, hq * dh), wgate=(mlp, hidden), wup=(mlp, hidden), wdown=(hidden, mlp))
    w = {n: (r(*s) * 0.05).to(dt) for n, s in dims.items()}
    w.update(g1=torch.ones(hidden, device="cuda", dtype=dt), g2=torch.ones(hidden, device="cuda", dtype=dt))
    ad = {n: ((r(rank, s[1]) * 0.05).to(dt), (r(s[0], rank) * 0.05).to(dt)) for n, s in dims.items()}
    x, dy = r(1, T, hidden).to(dt), (r(1, T, hidden) * 0.1).to(dt)
    cfg = sb.layer_cfg(sb.SBP_BF16 if dtype == "bf16" else sb.SBP_F32, 1, T, 32, hidden, hq, hkv, dh, mlp)
    got = []
    for by in (0, 1):
        a = {n: (_shifted(p, by), _shifted(q, by)) for n, (p, q) in ad.items()}
        start = {n: (r(rank, s[1]), r(s[0], rank)) for n, s in dims.items()} if not got else start
        da, db = {n: _shifted(p, by) for n, (p, _) in start.items()}, {n: _shifted(q, by) for n, (_, q) in start.items()}
        dx = torch.empty_like(x)
        ws = torch.empty(sb.streambp_layer_lora_workspace_bytes(cfg, a, rank, 2.0), dtype=torch.uint8, device="cuda")
        sb.streambp_layer_lora_backward(cfg, w, a, rank, 2.0, x, dy, dx=dx, da=da, db=db, workspace=ws)
        torch.cuda.synchronize()
        got.append([dx] + [da[n] for n in MATS] + [db[n] for n in MATS])
        assert all(torch.isfinite(t).all() for t in got[-1]) and any(not torch.equal(da[n], start[n][0]) for n in MATS)
    assert all(torch.equal(p, q) for p, q in zip(*got))
