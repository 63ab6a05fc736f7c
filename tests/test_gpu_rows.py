"""Strided passes over rows of no whole cache lines, ragged column counts run
on across planes, and half-width tiles: against the FP64 oracle, and bitwise
against the streaming schedule, whose tiles are the same per column.  Shapes
straddle the rules: aligned and unaligned rows, columns that fill no tile, one
and many planes, few and many tiles; alone, as a stack of arrays in one call
and merged with other shapes.  Tolerance against the oracle: complex64 1e-6."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import c16_to_dev, need_gpu, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPES = [(27, 48, 6), (36, 72, 32), (81, 54, 8), (96, 64, 9), (72, 216, 3), (243, 32, 6), (48, 96, 36), (3, 128, 54),
          (162, 162, 4), (24, 2048, 2), (27, 1536, 3), (9, 27, 243), (64, 64, 64), (144, 36, 128)]
ids = ["x".join(map(str, s)) for s in SHAPES]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_c64(ws, shape):
    nx, ny, nz = shape
    a = synth.uniform_c((nz, ny, nx), seed=nx + ny).astype(np.complex64)
    x = to_dev(a)
    p = ws.Plan(nx, ny, nz, "c64", -1, ws.FLAG_NO_PLANE)
    y = p.execute(x)
    assert rel_l2(to_host(y), oracle.fftn(a.astype(np.complex128), -1)) <= 1e-6, p.describe()
    s = ws.Plan(nx, ny, nz, "c64", -1, ws.FLAG_NO_PLANE | ws.FLAG_STREAMING).execute(x)
    assert torch.equal(torch.view_as_real(y), torch.view_as_real(s))
    z = x.clone()
    p.execute(z, z)
    assert torch.equal(torch.view_as_real(y), torch.view_as_real(z))
    if p.work_bytes == 0:
        xs = torch.stack([x, 2 * x, -x])
        ys = ws.execute_many(p, xs, torch.empty_like(xs), 3)
        assert torch.equal(torch.view_as_real(ys[0]), torch.view_as_real(y))
        assert torch.equal(torch.view_as_real(ys[2]), torch.view_as_real(-y))


@pytest.mark.parametrize("kind,flags", [("fp16", 0), ("bf16", 0), ("fp16", 4)], ids=["fp16", "bf16", "fp16-math"])
@pytest.mark.parametrize("shape", SHAPES, ids=ids)
def test_16bit_bitwise(ws, shape, kind, flags):
    nx, ny, nz = shape
    rnd = synth.to_fp16_pairs if kind == "fp16" else synth.to_bf16_pairs
    x = c16_to_dev(rnd(synth.normal_c((nz, ny, nx), seed=nx + ny, scale=0.5)), kind)
    y = ws.Plan(nx, ny, nz, kind, -1, flags).execute(x)
    s = ws.Plan(nx, ny, nz, kind, -1, flags | ws.FLAG_STREAMING).execute(x)
    assert torch.isfinite(y.float()).all()
    assert torch.equal(y.view(torch.int16), s.view(torch.int16))


def test_merged_batch_of_ragged_shapes(ws):
    shapes = [(27, 64, 6), (36, 64, 32), (81, 64, 8), (96, 64, 3), (243, 64, 6), (48, 64, 36), (72, 64, 1)]
    xs = [to_dev(synth.uniform_c((nz, ny, nx), seed=nx)) for nx, ny, nz in shapes]
    plans = [ws.Plan(*s, "c64", -1, ws.FLAG_NO_PLANE) for s in shapes]
    outs = [torch.empty_like(x) for x in xs]
    ws.execute_batched(plans, xs, outs)
    for p, x, y in zip(plans, xs, outs):
        assert torch.equal(torch.view_as_real(p.execute(x)), torch.view_as_real(y)), p.describe()


@pytest.mark.parametrize("shape", [(36, 81, 9), (64, 27, 81), (96, 54, 6), (12, 6, 243)],
                         ids=lambda s: "x".join(map(str, s)))
def test_real_unaligned_z(ws, shape):
    nx, ny, nz = shape
    a = synth.normal_c((nz, ny, nx), seed=nx).real.astype(np.float32)
    p = ws.RealPlan(nx, ny, nz)
    x = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    h = p.r2c(x)
    assert rel_l2(to_host(h), oracle.rfftn(a.astype(np.float64))) <= 1e-6
    assert rel_l2(to_host(p.c2r(h, inverse=True)), a) <= 2e-6
