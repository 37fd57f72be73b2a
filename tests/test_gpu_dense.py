"""Dense transforms (axis lengths without a fast FFT) at the edges of their
tiles: K = N/2 + 1 around multiples of 4 and 16, slice counts around 16, the
subtrahend of the inverse pass, slices beyond the column order's switch.

Against torch's float64 transforms; the float32 sums of K products per axis,
in groups of 32, keep the normwise error below (8 + 4 log2 K) 2^-24 per axis."""
import math

import pytest
import torch

from paper_2603_28150_amd import _lib
from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


def bound(*ns):
    return sum((8 + 4 * math.log2(n / 2 + 1)) * 2.0 ** -24 for n in ns)


@pytest.mark.parametrize("nx,ny", [(18, 18), (30, 34), (62, 66), (190, 22), (194, 16), (16, 254), (382, 18), (18, 510), (510, 30)])
@pytest.mark.parametrize("S", [1, 15, 17, 33])
def test_transform_and_inverse(nx, ny, S):
    op = Operator(Geometry(nx, ny, 2, 3, 1e-4, 1.1e-4, 1e-4, 2e-8, 1500.0))
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 1000 + ny + S)
    f = torch.randn((S, ny, nx), generator=g, device="cuda")
    B = -(-S // 3)
    spec = op.spectrum_buffer(S)
    op.spectrum(f, S, spec, B_ws=B)
    rows = torch.tensor(op.spectrum_rows(), device="cuda")
    live = rows >= 0
    got = torch.view_as_complex(spec[live][:, :S].double().contiguous())
    ref = torch.fft.rfft2(f.double()).reshape(S, -1).t()[rows[live]]
    assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) <= bound(nx, ny)
    # f - sub from the float64 spectrum rounded once (2^-24), and the two passes
    spec[live, :S] = torch.view_as_real(ref.contiguous()).float()
    sub = torch.randn((S, ny, nx), generator=g, device="cuda")
    back = torch.empty_like(f)
    op.inverse_spectrum(spec, S, back, sub=sub, B_ws=B)
    want = f.double() - sub.double()
    assert float(torch.linalg.norm(back.double() - want) / torch.linalg.norm(f.double())) <= bound(nx, ny) + 2.0 ** -22


def test_many_slices():
    # 2,100 slices: the column pass takes slice blocks fastest
    op = Operator(Geometry(50, 22, 2, 3, 1e-4, 1.1e-4, 1e-4, 2e-8, 1500.0))
    S = 2100
    f = torch.randn((S, 22, 50), device="cuda")
    spec = op.spectrum_buffer(S)
    op.spectrum(f, S, spec, B_ws=S // 3)
    back = torch.empty_like(f)
    op.inverse_spectrum(spec, S, back, B_ws=S // 3)
    assert float(torch.linalg.norm(back - f) / torch.linalg.norm(f)) <= 2 * bound(50, 22)


def test_scan_grid_stays_refused():
    with pytest.raises(RuntimeError):
        Operator(Geometry.paper_like(202, 32, 4, 8, sx=2))
    assert _lib.load() is not None
