"""One plan over arrays back to back (wsfft_execute_many) against
wsfft_execute_batched over the same entries, bit for bit, and the C2R call that
keeps its input against the one that overwrites it."""
import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def bits(t):
    return torch.view_as_real(t).view(torch.int32)


@pytest.mark.parametrize("shape,count", [((256, 1, 1), 5), ((256, 1, 1), 1), ((27, 6, 1), 9), ((48, 36, 4), 3),
                                         ((65536, 1, 1), 2), ((1, 1, 1), 4), ((512, 512, 96), 1)], ids=str)
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("in_place", [False, True])
def test_many_matches_batched(ws, shape, count, adjoint, in_place):
    nx, ny, nz = shape
    g = torch.Generator(device="cuda").manual_seed(nx + count)
    x = torch.view_as_complex(torch.randn((count, nz, ny, nx, 2), generator=g, device="cuda"))
    p = ws.Plan(nx, ny, nz, "c64", -1)
    want, got = x.clone(), x.clone()
    src_w, src_g = (want, got) if in_place else (x, x)
    if in_place and p.work_bytes:   # entries would share the plan's work buffer
        for call in (lambda: ws.execute_many(p, got, got, count, adjoint),
                     lambda: ws.execute_batched([p] * count, list(want), list(want), adjoint)):
            with pytest.raises(ws.WsfftError) as e:
                call()
            assert e.value.status == 1
        return
    ws.execute_batched([p] * count, list(src_w), list(want), adjoint)
    ws.execute_many(p, src_g, got, count, adjoint)
    assert torch.equal(bits(want), bits(got))


def test_many_of_no_arrays_and_of_16bit(ws):
    p = ws.Plan(64, 1, 1, "fp16", -1)
    e = torch.empty((0, 64, 2), dtype=torch.float16, device="cuda")
    ws.execute_many(p, e, e.clone(), 0)
    x = torch.randn((7, 64, 2), device="cuda").half()
    y = ws.execute_many(p, x, torch.empty_like(x), 7)
    z = torch.stack([p.execute(r.contiguous()) for r in x])
    assert torch.equal(y.view(torch.int16), z.view(torch.int16))


# one axis, two, three; a split y or z axis; unaligned rows
@pytest.mark.parametrize("shape", [(512, 1, 1), (36, 27, 1), (64, 1, 96), (48, 36, 32), (8, 2048, 6), (16, 3, 2048),
                                   (4, 2048, 2048)], ids=str)
def test_c2r_keep(ws, shape):
    nx, ny, nz = shape
    g = torch.Generator(device="cuda").manual_seed(nx)
    X = torch.view_as_complex(torch.randn((nz, ny, nx // 2 + 1, 2), generator=g, device="cuda"))
    before = X.clone()
    got = ws.irfftn(X, nx)
    assert torch.equal(bits(X), bits(before))
    want = ws.RealPlan(nx, ny, nz).c2r(X.clone(), inverse=True)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


def test_c2r_keep_argument_checks(ws):
    p = ws.RealPlan(8, 4, 2)
    buf = torch.zeros(4096, dtype=torch.float32, device="cuda")
    a = buf.data_ptr()
    call = ws._execute_c2r_inverse_keep
    assert call(p.handle, a, None, a + 8192, None) == 3
    assert call(p.handle, a, a, a + 8192, None) == 1
    assert call(p.handle, a, a + 8192, a + 8192, None) == 1
    assert call(p.handle, a, a + 4, a + 8192, None) == 4
    assert call(p.handle, None, a, a + 8192, None) == 3
    assert call(ws.Plan(8, 4, 2).handle, a, a + 4096, a + 8192, None) == 1
