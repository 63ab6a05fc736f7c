"""Merged levels that mix arrays whose rows are whole cache lines with arrays
whose rows are not: bitwise each plan's own call, for few small arrays (one
launch), for aligned arrays too large to join (a launch of their own), more
arrays than one launch holds, and both signs."""
import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu

BATCHES = {
    "small": [(64, 64, 32), (27, 27, 32), (48, 64, 16), (36, 64, 16), (27, 64, 16)],
    "large aligned": [(256, 256, 128), (243, 243, 16), (256, 256, 144), (81, 128, 16)],
    "many": [((24, 32, 48)[i % 3], 64, 6 + 2 * (i % 2)) for i in range(45)] + [(27, 64, 9), (81, 64, 2)],
}


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


@pytest.mark.parametrize("kind", ["c64", "fp16"])
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("name", BATCHES)
def test_mixed_rows(ws, name, adjoint, kind):
    g = torch.Generator(device="cuda").manual_seed(7)
    plans = [ws.Plan(nx, ny, nz, kind, -1, ws.FLAG_NO_PLANE) for nx, ny, nz in BATCHES[name]]
    xs = [0.5 * torch.randn((nz, ny, nx, 2), generator=g, device="cuda") for nx, ny, nz in BATCHES[name]]
    xs = [torch.view_as_complex(x) if kind == "c64" else x.half() for x in xs]
    ys = [torch.empty_like(x) for x in xs]
    ws.execute_batched(plans, xs, ys, adjoint=adjoint)
    for p, x, y in zip(plans, xs, ys):
        want = p.execute_adjoint(x) if adjoint else p.execute(x)
        a, b = (torch.view_as_real(y), torch.view_as_real(want)) if kind == "c64" else (y, want)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), p.describe()
