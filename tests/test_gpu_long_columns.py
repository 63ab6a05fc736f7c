"""1024-point strided passes of complex64: half-width tiles where rows are less
than 64 KiB apart or the full-width ones would leave CUs idle in the last round; both sides of the line, ragged column
counts, rows of no whole cache lines, in place, stacks, and merged launches that
mix the two.  Against the FP64 oracle at 1e-6 and, where one tile serves both,
bit for bit; the rounding of the full-width tile as in test_gpu_rounding."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import need_gpu, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

# (nx, ny, nz), whether the 1024-point pass halves its tiles
SHAPES = [((64, 1024, 3), True), ((27, 1024, 4), True), ((4096, 1024, 1), True), ((6912, 1024, 1), True),
          ((8192, 1024, 1), False), ((64, 64, 1024), True), ((128, 81, 1024), True), ((128, 64, 1024), False),
          ((27, 27, 1024), True), ((243, 32, 1024), True), ((13122, 1024, 3), False), ((324, 27, 1024), True)]
ids = ["x".join(map(str, s)) for s, _ in SHAPES]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def same(a, b):
    return torch.equal(torch.view_as_real(a), torch.view_as_real(b))


@pytest.mark.parametrize("shape,half", SHAPES, ids=ids)
def test_both_tiles(ws, shape, half):
    nx, ny, nz = shape
    a = synth.uniform_c((nz, ny, nx), seed=nx + ny).astype(np.complex64)
    x = to_dev(a)
    p = ws.Plan(nx, ny, nz, "c64", -1, ws.FLAG_NO_PLANE)
    assert ("n=1024 v0 half" in p.describe()) == half, p.describe()
    y = p.execute(x)
    assert rel_l2(to_host(y), oracle.fftn(a.astype(np.complex128), -1)) <= 1e-6
    assert same(y, ws.Plan(nx, ny, nz, "c64", -1, ws.FLAG_NO_PLANE | ws.FLAG_STREAMING).execute(x))
    z = x.clone()
    p.execute(z, z)
    assert same(y, z)
    xs = torch.stack([x, -x])
    ys = ws.execute_many(p, xs, torch.empty_like(xs), 2)
    assert same(ys[0], y) and same(ys[1], -y)
    assert rel_l2(to_host(p.execute_inverse(y)), a) <= 2e-6


@pytest.mark.parametrize("adjoint", [False, True])
def test_merged_launches_of_both(ws, adjoint):
    shapes = [s for s, _ in SHAPES if s[0] * s[1] * s[2] < 1 << 24] * 2
    plans = [ws.Plan(*s, "c64", -1, ws.FLAG_NO_PLANE) for s in shapes]
    xs = [to_dev(synth.uniform_c((nz, ny, nx), seed=i)) for i, (nx, ny, nz) in enumerate(shapes)]
    ys = [torch.empty_like(x) for x in xs]
    ws.execute_batched(plans, xs, ys, adjoint=adjoint)
    for p, x, y in zip(plans, xs, ys):
        assert same(y, p.execute_adjoint(x) if adjoint else p.execute(x)), p.describe()


def test_rounding_of_the_full_width_tile(ws):
    nx = 8192
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.view_as_complex(torch.randn((1, 1024, nx, 2), generator=g, device="cuda"))
    y = x.clone()
    ws.Plan(nx, 1024, 1, "c64", -1).execute_pass(1, x, y)
    want = torch.fft.fft(x.to(torch.complex128), dim=1)
    assert float((y.to(torch.complex128) - want).norm() / want.norm()) <= 1.005 * 1.091e-7
