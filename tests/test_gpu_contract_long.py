"""Contraction of one object with libraries beyond the 256 MB memory-side cache,
where slab loads, staging of the spectra and stores take other forms than on
small libraries: rows of whole and of broken 64-byte pieces, summed lengths that
end inside a block of rows, one, two and more tiles of outputs, with and without
the 16-bit scales.

Sampled frequencies against float64 products with the exported library, to the
rounding bound of any summation order, (K + 4) 2^-24 sum |h| |x| per value."""
import pytest
import torch

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu

#        n  nz  nt  library    (both row lengths and summed lengths in turn)
CASES = [
    (192, 77, 229, "f32"),     # A^T: staged, 320-byte rows, two tiles
    (192, 80, 337, "f32"),     # A^T: staged, whole 64-byte rows and stores
    (256, 33, 419, "f32"),     # broken rows, short sums
    (144, 213, 211, "f32"),    # 864- and 848-byte rows: plain, staged
    (144, 208, 195, "f32"),    # rows of 195 values: plain; A^T: staged, 832-byte rows, four tiles
    (96, 208, 334, "f32"),     # A: six tiles in one workgroup; A^T: four
    (96, 333, 784, "f32"),     # A^T: six tiles of broken rows; A: thirteen in two workgroups
    (128, 131, 300, "f32"),    # plain, A direct and A^T staged
    (128, 66, 777, "f32"),     # A^T: plain, staged, two tiles of which the second has two outputs
    (128, 213, 350, "bf16"),   # A: scales, 704-byte rows, three tiles
    (144, 93, 389, "bf16"),    # A^T: 192-byte rows, one tile shared by four waves
    (128, 203, 389, "f16"),    # broken rows
]


def check_contraction(op, adjoint, blocks):
    nz, nt = op.geom.nz, op.geom.nt
    K, N = (nt, nz) if adjoint else (nz, nt)
    rows = torch.tensor(op.spectrum_rows(), device="cuda")
    used = torch.nonzero(rows >= 0)[:, 0]
    spec = op.spectrum_buffer(K)
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * nz + nt)
    spec.normal_(generator=g)
    spec[:, K:] = float("nan")                                       # padding must not leak
    out = op.spectrum_buffer(N)
    op.contract(spec, out, adjoint)
    assert torch.isfinite(out[used][:, :N]).all()
    row_of = torch.empty(op.nk, dtype=torch.long, device="cuda")
    row_of[rows[used].long()] = used
    for k0 in blocks:
        H = op.export_H(k0, 40).double()                             # [40, nz, nt]
        M = H if adjoint else H.transpose(1, 2).contiguous()
        r = row_of[k0:k0 + 40]
        x = spec[r][:, :K].double().contiguous()
        err = (out[r][:, :N].double() - torch.matmul(M, x)).abs()
        assert (err <= (K + 4) * 2.0 ** -24 * torch.matmul(M.abs(), x.abs())).all(), (k0, float(err.max()))


@pytest.mark.parametrize("n,nz,nt,kind", CASES)
@pytest.mark.parametrize("adjoint", [False, True])
def test_contraction_of_large_libraries(n, nz, nt, kind, adjoint):
    op = Operator(Geometry.paper_like(n, n, nz, nt), kind)
    i = op.info()
    assert 2 * min(i["slab_bytes_A"], i["slab_bytes_AT"]) > 256 << 20
    check_contraction(op, adjoint, (0, 1, op.nk // 3 - 7, op.nk // 2, op.nk - 40))


# 16-bit rows of up to 32, 64, 128 and more values (loads of 4, 8 and 16 bytes),
# long sums shared by the waves of a workgroup, ends inside a block of rows
@pytest.mark.parametrize("nz,nt", [(260, 391), (257, 129), (300, 31), (32, 303), (512, 64), (33, 1100), (128, 777), (2, 263)])
@pytest.mark.parametrize("kind", ["bf16", "f16"])
@pytest.mark.parametrize("n", [16, 48])
def test_contraction_of_16_bit_rows(n, nz, nt, kind):
    op = Operator(Geometry.paper_like(n, n, nz, nt), kind)
    for adjoint in (False, True):
        check_contraction(op, adjoint, range(0, op.nk - 39, 40 if n == 16 else 400))


@pytest.mark.parametrize("n,nz,B", [(256, 113, 1), (256, 113, 2), (256, 127, 1), (512, 62, 1), (256, 121, 3)])
def test_half_blocks_beyond_the_cache(n, nz, B):
    op = Operator(Geometry.paper_like(n, n, nz, 6))
    assert op.info()["gram_bytes"] > 256 << 20
    H = op.export_H().double()
    g = torch.Generator(device="cuda")
    g.manual_seed(n + nz + B)
    z = torch.randn((B,) + op.x_shape, generator=g, device="cuda")
    x, zero, z0 = torch.zeros_like(z), torch.zeros_like(z), z.clone()
    op.fista_step_normal(zero, x, z, [0.0] * B, [1.0] * B, [0.0] * B, [False] * B)   # x = z - A^T A z
    for b in range(B):
        u = torch.view_as_real(torch.fft.rfft2(z0[b].double()).reshape(nz, -1).t().contiguous())
        r = torch.matmul(H, torch.matmul(H.transpose(1, 2).contiguous(), u))
        ref = torch.fft.irfft2(torch.view_as_complex(r.contiguous()).t().reshape(nz, n, -1), s=(n, n))
        tol = 1e-5 * max(float(ref.norm()), float(z0[b].norm()))     # z - A^T A z cancels
        assert float(((z0 - x)[b].double() - ref).norm()) <= tol, b
