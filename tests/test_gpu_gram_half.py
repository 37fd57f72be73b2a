"""Gram products of one object from half of each symmetric block, at the edges
of its tiles (16 rows) and loads (32 columns), with 8 and with 2 members per
group, and where the rule for more than 64 rows lets them in (for one object rows
of whole 64 bytes; at least 1,024 units of 8 pairs).

Against float64 products with the exported library, to the bars of the other
Gram tests: 1e-5 of the product, or of z where z - A^T A z cancels."""
import numpy as np
import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu

SMALL = [(16, ny, nz) for ny in (16, 32) for nz in (1, 4, 15, 16, 17, 31, 33, 47, 48, 49, 63, 64)]
LARGE = [(96, 96, nz) for nz in (77, 80, 96, 109, 112, 125, 128)] + [(64, 96, 80), (64, 96, 127)]


def exact(op):
    """A^T A, A^T as float64 functions of [n, ny, nx] arrays."""
    g = op.geom
    H = op.export_H().double()                       # [nk, nz, nt]
    Ht = H.transpose(1, 2).contiguous()

    def spectrum(v):
        return torch.view_as_real(torch.fft.rfft2(v.double()).reshape(v.shape[0], -1).t().contiguous())

    def back(u):
        c = torch.view_as_complex(u.contiguous()).t().reshape(u.shape[1], g.ny, -1)
        return torch.fft.irfft2(c, s=(g.ny, g.nx))

    return (lambda v: back(torch.matmul(H, torch.matmul(Ht, spectrum(v)))),
            lambda d: back(torch.matmul(H, spectrum(d))))


@pytest.mark.parametrize("nx,ny,nz", SMALL + LARGE)
def test_half_blocks(nx, ny, nz):
    op = Operator(Geometry(nx, ny, nz, 12, 1e-4, 1e-4 if nx == ny else 1.1e-4, 1e-4, 2e-7, 1500.0))
    ata, at = exact(op)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx * 10000 + ny * 100 + nz)
    z = torch.randn((1,) + op.x_shape, generator=gen, device="cuda")
    x, zero, z0 = torch.zeros_like(z), torch.zeros_like(z), z.clone()
    op.fista_step_normal(zero, x, z, [0.0], [1.0], [0.0], [False])   # x = z - A^T A z
    ref = ata(z0[0])
    tol = 1e-5 * max(float(ref.norm()), float(z0.norm()))
    assert float(((z0 - x)[0].double() - ref).norm()) <= tol

    # three iterations, the subtracted spectrum of A^T d among them
    d = torch.randn(op.d_shape, generator=gen, device="cuda")
    tau = float(np.float32(0.5 / op.power_norm(z0[0], 20)[0]))
    b, xk, zk, t = at(d), torch.zeros_like(ref), torch.zeros_like(ref), 1.0
    for _ in range(3):
        v = zk - tau * (ata(zk) - b)
        tn = (1.0 + (1.0 + 4.0 * t * t) ** 0.5) / 2.0
        xn = v.clamp_min(0.0)
        zk, xk, t = xn + (t - 1.0) / tn * (xn - xk), xn, tn
    got = op.recon_fista(d, 3, tau, 0.0, nonneg=True).double()
    assert float((got - xk).norm()) <= 1e-5 * float(xk.norm())


@pytest.mark.parametrize("nx,ny,nz,B", [(16, 16, 1, 2), (16, 16, 15, 3), (16, 16, 33, 5), (16, 16, 64, 32), (16, 32, 33, 3),
                                        (16, 32, 64, 4), (16, 32, 47, 9), (96, 96, 77, 2), (96, 96, 80, 3), (64, 64, 80, 2),
                                        (64, 64, 127, 3), (64, 96, 128, 5),
                                        (96, 96, 65, 2), (96, 96, 105, 3), (64, 96, 114, 2)])
def test_half_blocks_of_several_objects(nx, ny, nz, B):
    # objects that start at odd multiples of 8 bytes in a spectrum row, pairs
    # that fill a wave's columns in part, more units than groups
    op = Operator(Geometry(nx, ny, nz, 12, 1e-4, 1e-4 if nx == ny else 1.1e-4, 1e-4, 2e-7, 1500.0))
    ata, _ = exact(op)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx * 10000 + ny * 100 + nz + B)
    z = torch.randn((B,) + op.x_shape, generator=gen, device="cuda")
    x, zero, z0 = torch.zeros_like(z), torch.zeros_like(z), z.clone()
    op.fista_step_normal(zero, x, z, [0.0] * B, [1.0] * B, [0.0] * B, [False] * B)
    for b in range(B):
        ref = ata(z0[b])
        tol = 1e-5 * max(float(ref.norm()), float(z0[b].norm()))
        assert float(((z0 - x)[b].double() - ref).norm()) <= tol, b
