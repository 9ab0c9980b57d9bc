"""Every column of the z pass is the same 1D transform whatever the width of
its pencil: H psi with rows of 16 complex (SGW_FORCE_VARIANT pencil=0) is
bitwise H psi with the wide rows, at each length that has both, on cubic grids
and on one whose planes are shorter than its z lines."""
import pytest
import torch

from paper_2601_21005_amd import sgw

pytestmark = pytest.mark.gpu
WIDE = [(40, 40, 40), (48, 48, 48), (56, 56, 56), (64, 64, 64), (80, 80, 80), (96, 96, 96),
        (128, 128, 128), (32, 32, 96)]


@pytest.mark.parametrize("prec", [sgw.SGW_C64, sgw.SGW_C128])
@pytest.mark.parametrize("n", WIDE)
def test_pencil_width_changes_no_bit(n, prec, monkeypatch):
    N = n[0] * n[1] * n[2]
    g = torch.Generator(device="cuda").manual_seed(n[2])
    v = -torch.rand(N, generator=g, device="cuda", dtype=torch.float64).cpu().numpy()
    x = torch.randn((3, N), generator=g, device="cuda", dtype=torch.complex64)
    out = []
    for forced in (False, True):
        if forced:
            monkeypatch.setenv("SGW_FORCE_VARIANT", "pencil=0")
        ctx = sgw.Context(n, 0.6, v, None, precision=prec, ecut=28.0, max_nvec=3)
        y = torch.zeros_like(x.to(ctx.cdtype))
        ctx.apply_H(x.to(ctx.cdtype), y)
        torch.cuda.synchronize()
        ctx.close()
        out.append(y)
    assert torch.isfinite(torch.view_as_real(out[0])).all()
    assert torch.equal(out[0], out[1])
