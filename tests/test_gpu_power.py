"""Normalisation of the power iteration at its edges: volumes with 0 to 3
values beyond the last 16 bytes, volumes below one block and above one stride
of the whole grid (524,288 values), a volume of one slice.

Against the same operator's A and A^T with float64 products and norms.  The
float32 sums run through at most 32 roundings per value, normalisation adds
three and one rounding of v per step moves later quotients by at most as much
again, all relative to |A^T A v|: (64 + 16 i) 2^-24 of the largest one at step i."""
import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(16, 16, 1), (17, 19, 3), (18, 21, 5), (17, 17, 7), (16, 20, 9), (64, 64, 130)])
def test_quotients_match_float64_sums(nx, ny, nz):
    op = Operator(Geometry(nx, ny, nz, 24, 1e-4, 1.1e-4, 1e-4, 2e-8, 1500.0, boundary="linear"))
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 100 + nz)
    v = torch.randn(op.x_shape, generator=g, device="cuda")
    L, trace = op.power_norm(v, 5)
    ref, top = [], 0.0
    v = (v.double() / v.double().norm()).float()
    for _ in range(5):
        u = op.apply_AT(op.apply_A(v)).double()
        ref.append(float((v.double() * u).sum()))
        top = max(top, float(u.norm()))
        v = (u / u.norm()).float()
    assert L == trace[-1]
    for i, (a, b) in enumerate(zip(trace, ref)):
        assert abs(a - b) <= (64 + 16 * i) * 2.0 ** -24 * top
