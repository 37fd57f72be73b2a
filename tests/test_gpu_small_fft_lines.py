"""One-kernel and two-pass transforms on both sides of the lines between them,
which the forward and the inverse transform have at different slice counts.

Against torch's float64 transforms; split transforms of N points keep the
normwise error of an axis below (8 + 4 log2 N) 2^-24."""
import math

import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,S", [((48, 48), 1024), ((48, 48), 1025), ((48, 48), 1365), ((48, 48), 1366), ((64, 64), 576),
                                 ((64, 64), 577), ((64, 48), 1024), ((64, 48), 1025), ((48, 32), 1536), ((48, 32), 1537),
                                 ((48, 32), 2731), ((32, 32), 4096), ((32, 32), 4097)])
def test_both_sides(n, S):
    nx, ny = n
    op = Operator(Geometry(nx, ny, 2, 3, 1e-4, 1.1e-4, 1e-4, 2e-8, 1500.0))
    g = torch.Generator(device="cuda")
    g.manual_seed(S)
    f = torch.randn((S, ny, nx), generator=g, device="cuda")
    B = -(-S // 3)
    bound = sum((8 + 4 * math.log2(k)) * 2.0 ** -24 for k in n)
    spec = op.spectrum_buffer(S)
    spec.fill_(float("nan"))
    op.spectrum(f, S, spec, B_ws=B)
    rows = torch.tensor(op.spectrum_rows(), device="cuda")
    live = rows >= 0
    got = torch.view_as_complex(spec[live][:, :S].double().contiguous())
    ref = torch.fft.rfft2(f.double()).reshape(S, -1).t()[rows[live]]
    assert float((got - ref).norm() / ref.norm()) <= bound
    spec.fill_(float("nan"))
    spec[live, :S] = torch.view_as_real(ref.contiguous()).float()
    out = torch.full_like(f, float("nan"))
    op.inverse_spectrum(spec, S, out, B_ws=B)
    assert float((out.double() - f.double()).norm() / f.double().norm()) <= bound + 2.0 ** -23
