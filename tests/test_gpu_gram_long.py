"""Batched Gram products of many rows whose blocks together exceed the 256 MB
memory-side cache: one, two and three or more objects take different kernels,
whose needs of LDS must stay within a CU at every depth.

Against float64 products with the exported library, to the bar of the other
Gram tests: 1e-5 of the product, or of z where z - A^T A z cancels."""
import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


def normal64(op, z):
    """A^T A z in float64 of [nz, ny, nx] z."""
    g = op.geom
    H = op.export_H().double()                                       # [nk, nz, nt]
    u = torch.fft.rfft2(z.double()).reshape(g.nz, -1).t()
    u = torch.view_as_real(u.contiguous())                           # [nk, nz, 2]
    r = torch.matmul(H, torch.matmul(H.transpose(1, 2).contiguous(), u))
    c = torch.view_as_complex(r.contiguous()).t().reshape(g.nz, g.ny, -1)
    return torch.fft.irfft2(c, s=(g.ny, g.nx))


@pytest.mark.parametrize("nx,ny,nz", [(48, 48, 608), (48, 48, 640), (64, 64, 409), (64, 64, 992), (64, 32, 641)])
@pytest.mark.parametrize("B", [1, 2, 3, 5])
def test_many_rows(nx, ny, nz, B):
    op = Operator(Geometry.paper_like(nx, ny, nz, 6))
    assert op.info()["gram_bytes"] > 256 << 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx * 10000 + nz + B)
    z = torch.randn((B,) + op.x_shape, generator=gen, device="cuda")
    x, zero, z0 = torch.zeros_like(z), torch.zeros_like(z), z.clone()
    op.fista_step_normal(zero, x, z, [0.0] * B, [1.0] * B, [0.0] * B, [False] * B)   # x = z - A^T A z
    for b in range(B):
        ref = normal64(op, z0[b])
        tol = 1e-5 * max(float(ref.norm()), float(z0[b].norm()))
        assert float(((z0 - x)[b].double() - ref).norm()) <= tol, b


@pytest.mark.parametrize("nx,ny,nz", [(72, 72, 373), (72, 72, 374), (128, 128, 217), (96, 64, 262), (48, 32, 1030), (64, 32, 777)])
def test_broken_lines(nx, ny, nz):
    # blocks whose rows are not whole 128-byte lines: one object, classes of
    # eight members and (on the vector units) of two, odd and even rows, rows over
    # one and two workgroups, with and without the subtracted spectrum
    op = Operator(Geometry.paper_like(nx, ny, nz, 6))
    i = op.info()
    assert i["gram_bytes"] > 256 << 20
    H = op.export_H().double()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx * 10000 + nz)
    z0 = torch.randn(op.x_shape, generator=gen, device="cuda")
    z, x, zero = z0[None].clone(), torch.zeros_like(z0)[None], torch.zeros_like(z0)[None]
    op.fista_step_normal(zero, x, z, [0.0], [1.0], [0.0], [False])   # x = z - A^T A z
    ref = normal64(op, z0)
    assert float(((z0 - x[0]).double() - ref).norm()) <= 1e-5 * max(float(ref.norm()), float(z0.norm()))

    d = torch.randn(op.d_shape, generator=gen, device="cuda")
    u = torch.view_as_real(torch.fft.rfft2(d.double()).reshape(op.geom.nt, -1).t().contiguous())
    c = torch.view_as_complex(torch.matmul(H, u).contiguous()).t().reshape(nz, ny, -1)
    b, tau = torch.fft.irfft2(c, s=(ny, nx)), 0.25
    xk, zk, t = torch.zeros_like(b), torch.zeros_like(b), 1.0
    for _ in range(3):
        v = zk - tau * (normal64(op, zk) - b)
        tn = (1.0 + (1.0 + 4.0 * t * t) ** 0.5) / 2.0
        xn = v.clamp_min(0.0)
        zk, xk, t = xn + (t - 1.0) / tn * (xn - xk), xn, tn
    got = op.recon_fista(d, 3, tau, 0.0, nonneg=True).double()
    assert float((got - xk).norm()) <= 1e-5 * float(xk.norm())
