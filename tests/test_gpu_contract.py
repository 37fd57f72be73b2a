"""Per-frequency contraction at the edges of its tiles and row blocks, against
float64 products with the exported library.

The float32 sums of K products are held to the rounding bound of any summation
order, (K + 4) 2^-24 sum |h| |x| per value (one rounding per product and per
addition, and two more for the 16-bit scales)."""
import numpy as np
import pytest
import torch

from paper_2603_28150_amd import inputs
from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


def geometry(square, nz, nt):
    # square: radial classes of up to 8 members; otherwise 2 members
    return Geometry.paper_like(16, 16 if square else 32, nz, nt)


def contract64(op, spec, K, adjoint):
    """(sum_k h x, sum_k |h| |x|) per frequency: spec [nk][K] complex128."""
    H = op.export_H().double()                                   # [nk, nz, nt]
    M = H if adjoint else H.transpose(1, 2).contiguous()         # [nk, n_out, K]
    X = torch.view_as_real(spec)                                 # [nk, K, 2]
    return (torch.matmul(M, X.contiguous()), torch.matmul(M.abs(), X.abs().contiguous()))


@pytest.mark.parametrize("square", [True, False])
@pytest.mark.parametrize("kind", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("nz,nt", [(1, 1), (7, 8), (8, 65), (9, 63), (16, 64), (63, 129), (65, 257), (130, 66), (33, 512)])
def test_contraction_edges(square, kind, nz, nt):
    op = Operator(geometry(square, nz, nt), kind)
    rows = torch.tensor(op.spectrum_rows(), device="cuda")
    used = rows >= 0
    k = rows[used]
    for adjoint in (False, True):
        K, N = (nt, nz) if adjoint else (nz, nt)
        spec = op.spectrum_buffer(K)
        spec.fill_(float("nan"))                                 # padding and unused rows must not leak
        g = torch.Generator(device="cuda")
        g.manual_seed(100 * nz + nt)
        vals = torch.randn((int(used.sum()), K, 2), generator=g, device="cuda")
        buf = spec[used]
        buf[:, :K] = vals
        spec[used] = buf
        out = op.spectrum_buffer(N)
        op.contract(spec, out, adjoint)
        got = out[used][:, :N].double()
        full = torch.zeros((op.nk, K), dtype=torch.complex128, device="cuda")
        full[k] = torch.view_as_complex(vals.double())
        ref, mag = contract64(op, full, K, adjoint)
        err = (got - ref[k]).abs()
        assert torch.isfinite(got).all()
        assert (err <= (K + 4) * 2.0 ** -24 * mag[k] + 1e-37).all(), (adjoint, float(err.max()))


@pytest.mark.parametrize("square", [True, False])
@pytest.mark.parametrize("nz", [5, 16, 61, 128])
@pytest.mark.parametrize("B", [2, 3, 5, 9, 17, 32])
def test_batched_normal_step_equals_single(square, nz, B):
    # pairs (member, object) beyond one, two and four column groups
    op = Operator(geometry(square, nz, 40))
    z0 = torch.from_numpy(np.stack([inputs.gaussian_random(op.x_shape, seed=2300 + b) for b in range(B)])
                          .astype(np.float32)).cuda()
    atd = torch.flip(z0, [0]).contiguous()

    def step(z, a):
        n = z.shape[0]
        x, zz = torch.zeros_like(z), z.clone()
        op.fista_step_normal(a, x, zz, [0.0] * n, [0.5] * n, [0.0] * n, [False] * n)
        return x
    xb = step(z0, atd)
    for b in (0, B // 2, B - 1):
        xs = step(z0[b:b + 1].contiguous(), atd[b:b + 1].contiguous())[0]
        assert float(torch.linalg.norm(xb[b] - xs) / torch.linalg.norm(xs)) <= 1e-6, b
