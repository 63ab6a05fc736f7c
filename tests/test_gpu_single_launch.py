"""Launches of one direct pass carry 64 bytes of arguments; a merged launch of
the same plan twice carries the full ones.  Both give the same bits: every
layout, storage type and tile form, unaligned and run-on rows, XCD order,
scales of the inverse, the plane pass, real rows with a pitch."""
import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1, 1), (27, 36, 8), (243, 32, 6), (96, 64, 9), (512, 8, 2), (3, 512, 4), (32, 32, 32), (128, 96, 2)]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


@pytest.mark.parametrize("kind,flags", [("c64", 0), ("c64", 8), ("c64", 16), ("fp16", 0), ("bf16", 0), ("fp16", 4)],
                         ids=["c64", "no-plane", "streaming", "fp16", "bf16", "fp16-math"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("adjoint", [False, True])
def test_single_matches_merged(ws, shape, kind, flags, adjoint):
    nx, ny, nz = shape
    dt = {"c64": torch.float32, "fp16": torch.float16, "bf16": torch.bfloat16}[kind]
    g = torch.Generator(device="cuda").manual_seed(nx)
    x = (0.5 * torch.randn((nz, ny, nx, 2), generator=g, device="cuda")).to(dt)
    if kind == "c64":
        x = torch.view_as_complex(x)
    p = ws.Plan(nx, ny, nz, kind, -1, flags)
    one = p.execute_adjoint(x) if adjoint else p.execute(x)
    outs = [torch.empty_like(x), torch.empty_like(x)]
    ws.execute_batched([p, p], [x, x], outs, adjoint=adjoint)
    for o in outs:
        assert torch.equal(o.view(torch.uint8) if kind != "c64" else torch.view_as_real(o).view(torch.uint8),
                           one.view(torch.uint8) if kind != "c64" else torch.view_as_real(one).view(torch.uint8))
    back = p.execute_inverse(one)
    if not adjoint and kind == "c64":
        assert float(torch.linalg.vector_norm(back - x) / torch.linalg.vector_norm(x)) <= 2e-6


@pytest.mark.parametrize("nx,ny,nz,pitch", [(54, 12, 6, 0), (54, 12, 6, 48), (512, 9, 4, 0), (64, 1, 1, 0)])
def test_real_pass_by_pass(ws, nx, ny, nz, pitch):
    p = ws.RealPlan(nx, ny, nz, pitch=pitch)
    x = torch.randn((nz, ny, nx), generator=torch.Generator(device="cuda").manual_seed(nx), device="cuda")
    h = p.r2c(x)
    want = torch.fft.rfftn(x.double(), dim=(0, 1, 2))
    got = h[..., :nx // 2 + 1]
    assert float(torch.linalg.vector_norm(got - want) / torch.linalg.vector_norm(want)) <= 1e-6
    back = p.c2r(h, inverse=True)
    assert float(torch.linalg.vector_norm(back - x) / torch.linalg.vector_norm(x)) <= 2e-6
