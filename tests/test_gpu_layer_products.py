"""The layer's projections at the edges of their tiles: widths that fill no tile, reductions that end
inside a block, one token, token counts on both sides of the tile sizes, and a width that goes to
the vendor library.  Reference: the products in float32, rounded to bf16 where the layer rounds
them, around the operator's own forward.  Both sides round the same products to bf16 (2^-9 relative
each, once before and once after the operator), so they may differ by a few 2^-9 in the norm."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # B, L, H, d
    (1, 1, 1, 32), (1, 63, 3, 32), (1, 65, 5, 32), (2, 127, 1, 64), (1, 129, 2, 128), (3, 171, 3, 64),
    (1, 5000, 3, 32), (2, 4097, 4, 64), (1, 3000, 4, 128), (1, 40, 16, 128), (1, 2100, 8, 128),
]


@pytest.mark.parametrize("B,L,H,d", CASES)
def test_projections(B, L, H, d):
    import paper_2606_09862_amd as bla
    print(f"layer products: tokens {B}x{L} width {H * d}", flush=True)
    D, M, S = H * d, 8, 15
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    x, wq, wo = (torch.randn(*s, generator=g, device="cuda").mul_(c).to(torch.bfloat16)
                 for s, c in (((B, L, D), 1.0), ((D, 3 * D), D ** -0.5), ((D, D), D ** -0.5)))
    T = [15.0 * (1 + h % 2) for h in range(H)]
    y, sk, sv = bla.layer_forward(x, wq, wo, T, H, M, S)
    qkv = (x.float().view(-1, D) @ wq.float()).to(torch.bfloat16).view(B, L, 3, H, d).permute(2, 0, 3, 1, 4)
    o, rk, rv = bla.forward(*(t.contiguous() for t in qkv), T, M, S)
    ref = (o.permute(0, 2, 1, 3).reshape(-1, D).float() @ wo.float()).view(B, L, D)
    torch.cuda.synchronize()
    for a, b in ((y, ref), (sk, rk), (sv, rv)):
        a, b = a.double(), b.double()
        assert torch.isfinite(a).all()
        assert ((a - b).norm() / b.norm().clamp_min(1e-30)).item() < 4 * 2.0 ** -9
