"""The matrix-core routers' tiles against each other and against plain float64:
token counts at the edges of their 32- and 128-token tiles, expert counts of
every kernel choice, with and without stored logits (bf16, through the C ABI).

A logit is summed in one order whichever tile its token is in (E > 64: one chain
of matrix instructions over K; else the sums of four K quarters, added in
order), so a token routed alone gives the bits it gives in any batch."""
import numpy as np
import pytest
import torch

from gpu_helpers import log

pytestmark = pytest.mark.gpu


def _route(B, desc, x, gain, Wg, bias, T, want_z):
    E, k, H, dev = desc.E, desc.k, desc.H, x.device
    out = dict(a=torch.empty(T, H, dtype=torch.bfloat16, device=dev),
               z=torch.full((T, E), float("nan"), device=dev) if want_z else None,
               idx=torch.full((T, k), -1, dtype=torch.int32, device=dev),
               w=torch.full((T, k), float("nan"), device=dev),
               counts=torch.full((E,), -1, dtype=torch.int32, device=dev))
    B.easybalance_route(desc, 0, T, x, gain, Wg, bias, out["a"], out["z"], out["idx"], out["w"], out["counts"])
    return out


@pytest.mark.parametrize("E,k,H", [(20, 2, 256), (64, 6, 512), (65, 4, 256), (100, 16, 512), (129, 8, 256),
                                   (200, 12, 512), (256, 8, 768)])
def test_route_tiles(E, k, H, device):
    from paper_2608_07964_amd import binding as B
    g = torch.Generator(device=device).manual_seed(E)
    Tmax = 8200
    x = torch.randn(Tmax, H, generator=g, device=device)
    gain = 1 + 0.1 * torch.randn(H, generator=g, device=device)
    Wg = (torch.randn(E, H, generator=g, device=device) * H ** -0.5).bfloat16()
    bias = torch.randn(E, generator=g, device=device)
    desc = B.make_desc(1, H, 128, E, k, 0, 1, "bf16", norm_topk=E % 2)
    ref = None
    # one workgroup per entry, several 32-token tiles, two expert halves, 128-token tiles
    for T in (Tmax, 4097, 4096, 129, 128, 33, 32, 31, 1):
        for want_z in (True, False):
            log(f"route tiles E {E} T {T} z {want_z}")
            o = _route(B, desc, x, gain, Wg, bias, T, want_z)
            torch.cuda.synchronize()
            if ref is None:
                ref = o
                z64 = o["a"].double() @ Wg.double().t() + bias.double()
                # fp32 accumulation of H products: error below H * 2^-24 * sum |a w|
                bound = H * 2.0 ** -24 * (o["a"].double().abs() @ Wg.double().abs().t()) + 1e-6
                assert ((o["z"].double() - z64).abs() <= bound).all()
                top = torch.sort(o["z"], dim=1, descending=True, stable=True).indices[:, :k]
                assert torch.equal(o["idx"].long(), top)
                p = torch.gather(torch.softmax(o["z"].double(), 1), 1, top)
                if desc.norm_topk:
                    p = p / p.sum(1, keepdim=True)
                assert np.abs((o["w"].double() - p).cpu().numpy()).max() <= 1e-5
            for key in ("a", "idx", "w") + (("z",) if want_z else ()):
                got, want = o[key], ref[key][:T]
                if key == "a":
                    got, want = got.view(torch.int16), want.contiguous().view(torch.int16)
                assert torch.equal(got, want), (key, T, want_z)
            assert torch.equal(o["counts"].long(), torch.bincount(ref["idx"][:T].reshape(-1).long(), minlength=E))


# (E, T, stored logits) -> launches of the router and of separate top-k and count kernels
@pytest.mark.parametrize("E,T,want_z,logits,topk", [(64, 32, True, 1, 0), (64, 33, True, 1, 1), (100, 16, True, 1, 0),
                                                    (256, 16, False, 1, 0), (256, 16, True, 1, 2), (256, 64, False, 1, 1)])
def test_profile_counts_the_launches(E, T, want_z, logits, topk, device):
    from paper_2608_07964_amd import binding as B
    log(f"profile E {E} T {T} z {want_z}")
    H, k = 256, 4
    g = torch.Generator(device=device).manual_seed(1)
    desc = B.make_desc(1, H, 128, E, k, 0, 1, "bf16")
    B.easybalance_profile_begin()
    _route(B, desc, torch.randn(T, H, generator=g, device=device), torch.ones(H, device=device),
           torch.randn(E, H, generator=g, device=device).bfloat16(), torch.zeros(E, device=device), T, want_z)
    torch.cuda.synchronize()
    p = B.easybalance_profile_end()
    assert (p["route_norm"][1], p["route_logits"][1], p["route_topk"][1]) == (1, logits, topk)
    assert (p["route_topk"][0] > 0) == (topk > 0)
