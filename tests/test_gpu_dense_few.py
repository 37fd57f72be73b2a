"""Dense transforms of few slices, where the output tiles of a workgroup's
slices are dealt to several workgroups and, under nine slices, further rows and
frequencies take the columns that no slice fills: axis lengths with one to four
rounds of tiles, slice counts around the powers of two, rows and frequencies
that do not fill the last workgroup.

Against torch's float64 transforms; the float32 sums of K products per axis,
in groups of 32, keep the normwise error below (8 + 4 log2 K) 2^-24 per axis."""
import math

import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


def bound(*ns):
    return sum((8 + 4 * math.log2(n / 2 + 1)) * 2.0 ** -24 for n in ns)


@pytest.mark.parametrize("nx,ny", [(510, 510), (506, 382), (382, 506), (450, 18), (18, 450), (254, 256), (300, 302), (202, 202), (490, 512)])
@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 8, 9, 16, 18])
def test_few_slices(nx, ny, S):
    op = Operator(Geometry(nx, ny, 2, 3, 1e-4, 1e-4, 1e-4, 2e-8, 1500.0))
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 1000 + ny + S)
    f = torch.randn((S, ny, nx), generator=g, device="cuda")
    B = -(-S // 3)
    spec = op.spectrum_buffer(S)
    spec.fill_(float("nan"))
    op.spectrum(f, S, spec, B_ws=B)
    rows = torch.tensor(op.spectrum_rows(), device="cuda")
    live = rows >= 0
    got = torch.view_as_complex(spec[live][:, :S].double().contiguous())
    ref = torch.fft.rfft2(f.double()).reshape(S, -1).t()[rows[live]]
    assert float(torch.linalg.norm(got - ref) / torch.linalg.norm(ref)) <= bound(nx, ny)
    # f - sub from the float64 spectrum rounded once (2^-24), and the two passes
    spec.fill_(float("nan"))
    spec[live, :S] = torch.view_as_real(ref.contiguous()).float()
    sub = torch.randn((S, ny, nx), generator=g, device="cuda")
    back = torch.full_like(f, float("nan"))
    op.inverse_spectrum(spec, S, back, sub=sub, B_ws=B)
    want = f.double() - sub.double()
    assert float(torch.linalg.norm(back.double() - want) / torch.linalg.norm(f.double())) <= bound(nx, ny) + 2.0 ** -22
