"""fp32 scoring of 513 to 1024 keys of 64 components, whose products are taken by thirds of the operands: against 64 bits on
ordinary and on far apart values, and with infinities, which have no thirds.

The tolerance: a logit of 64 products carries at most 64 roundings of 2^-24 of the sum of their sizes, a few units of x = 2^-20 |q| |k| / 8;
the in-degree's and the entropy's relative error is of that order times the logits' spread (about 45 here): 2e-6 leaves a factor of five over
what is measured, 1e-7 to 4e-7."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def _exact(q, k, w, causal):
    H, G, n = q.shape[0], k.shape[0], k.shape[1]
    x = torch.stack([q[h].double() @ k[h // (H // G)].double().T for h in range(H)]) / math.sqrt(q.shape[2])
    if causal:
        at = n - w + torch.arange(w, device=q.device)
        x = torch.where(torch.arange(n, device=q.device)[None, None] <= at[None, :, None], x, -math.inf)
    p = torch.softmax(x, -1)
    return p.sum((0, 1)), -torch.where(p > 0, p * p.log(), 0.0).sum(-1).mean(-1)


@pytest.mark.parametrize("values", ["normal", "apart", "small", "infinite"])
@pytest.mark.parametrize("H,G,w,n,causal", [(8, 8, 32, 1024, False), (8, 2, 8, 513, False), (4, 2, 9, 700, True), (2, 2, 33, 1023, True)])
def test_products_by_thirds(H, G, w, n, causal, values):
    from paper_2604_06746_amd.sweep import LayerSweep
    g = torch.Generator(device="cuda")
    g.manual_seed(n + w)
    q = torch.randn(H, w, 64, generator=g, device="cuda")
    k = torch.randn(G, n, 64, generator=g, device="cuda")
    if values == "apart":      # components of 2^-20 to 2^20, those of queries and keys the other way round
        e = torch.randint(-20, 21, (64,), generator=g, device="cuda").float().exp2()
        q, k = q * e, k / e
    if values == "small":      # keys whose lower thirds lie near the smallest normal numbers, and the queries that make up for it
        q, k = q * 2.0 ** 100, k * 2.0 ** -100
    if values == "infinite":   # a key that no row sees anything of, far from any other
        q[..., 5] = q[..., 5].abs() + 0.1
        k[:, n // 3, 5] = -math.inf
    sw = LayerSweep(H, G, 64, w, torch.float32, [n], [n // 8], causal=causal)
    sw.score(q[None].contiguous(), k)
    torch.cuda.synchronize()
    D, ent = _exact(q, k, w, causal)
    if values == "infinite":
        assert float(sw.indeg[n // 3]) == 0.0
    assert float((sw.indeg.double() - D).norm() / D.norm()) < 2e-6
    if values == "infinite":   # (an entropy term of 0 times infinity is not a number)
        return
    assert float((sw.entropy_per_head[0].double() - ent).norm() / ent.norm()) < 2e-6


@pytest.mark.parametrize("side", ["keys", "queries"])
@pytest.mark.parametrize("exponent", [60, 89, 91, 108, 112, 115, 118, 122, 124])
def test_products_by_thirds_of_tiny_operands(side, exponent):
    """One side so small that its lower thirds, or all of them, lie below the smallest bf16 number, the other as much larger: the same
    logits, and the same tolerance.  The small side holds zeros and ordinary numbers too.  (The fp32 instruction takes over at 2^90.)"""
    from paper_2604_06746_amd.sweep import LayerSweep
    H, G, w, n = 8, 2, 8, 900
    g = torch.Generator(device="cuda")
    g.manual_seed(exponent)
    q = torch.randn(H, w, 64, generator=g, device="cuda")
    k = torch.randn(G, n, 64, generator=g, device="cuda")
    up = torch.full((64,), float(exponent), device="cuda")
    up[::7] = 0.0                       # (components that both sides have in full)
    up = torch.exp2(up)
    k[:, ::5, ::3] = 0.0
    q, k = (q * up, k / up) if side == "keys" else (q / up, k * up)
    sw = LayerSweep(H, G, 64, w, torch.float32, [n], [n // 8])
    sw.score(q[None].contiguous(), k)
    torch.cuda.synchronize()
    D, ent = _exact(q, k, w, False)
    assert float((sw.indeg.double() - D).norm() / D.norm()) < 2e-6
    assert float((sw.entropy_per_head[0].double() - ent).norm() / ent.norm()) < 2e-6


def test_products_by_thirds_of_tiny_keys_under_a_large_scale():
    from paper_2604_06746_amd import binding as B
    from paper_2604_06746_amd.sweep import LayerSweep
    H, G, w, n = 8, 2, 8, 900
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q = torch.randn(H, w, 64, generator=g, device="cuda")
    k = torch.randn(G, n, 64, generator=g, device="cuda") * 2.0 ** -118
    sw = LayerSweep(H, G, 64, w, torch.float32, [n], [n // 8])
    shape = B.make_shape(H, G, 64, w, B.STRUCTKV_DTYPE_F32, scale=2.0 ** 115)   # (2^118 / 8)
    B.structkv_score_layer(shape, q[None].contiguous(), k, sw.cu, sw.indeg, sw.entropy, sw.entropy_per_head, sw.workspace)
    torch.cuda.synchronize()
    D, ent = _exact(q, k * 2.0 ** 118, w, False)
    assert float((sw.indeg.double() - D).norm() / D.norm()) < 2e-6
    assert float((sw.entropy_per_head[0].double() - ent).norm() / ent.norm()) < 2e-6
