"""The library bytes that one apply of one object reads, as pat_get_info reports
them: a slab per group of up to eight frequencies of a class, whatever the
work items of batches hold."""
import pytest

from paper_2603_28150_amd.op import Geometry, Operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("nx,ny", [(16, 16), (48, 48), (72, 72), (16, 32)])
def test_read_bytes(kind, nx, ny):
    nh = nx // 2 + 1
    members = {}
    for k in range(ny * nh):
        m, p = k % nh, min(k // nh, ny - k // nh)
        c = m * m + p * p if nx == ny else (m, p)
        members[c] = members.get(c, 0) + 1
    groups = sum(-(-n // 8) for n in members.values())
    i = Operator(Geometry.paper_like(nx, ny, 24, 40), kind).info()
    assert i["nclass"] == len(members)
    assert i["read_bytes_A"] == i["slab_bytes_A"] // i["nclass"] * groups
    assert i["read_bytes_AT"] == i["slab_bytes_AT"] // i["nclass"] * groups
