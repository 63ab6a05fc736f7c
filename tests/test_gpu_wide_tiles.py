"""The 64-column strided tiles of the 4-byte types, which only launches of 512
tiles and more take (smaller ones run half-width tiles): every length that has
one, as the z axis over aligned columns and over columns of no whole cache lines
(the cached kernels), and as the y axis.  Sampled columns, the last tile's among
them, against the FP64 oracle at the 16-bit bounds (3e-3; BF16 with rounded
twiddles: 3 one-rounding floors), and whole slices with FP32 arithmetic bit for
bit against calls so small that they take half-width tiles, where the length has
them.  Then the
16-bit arrays that take the cached passes, bitwise against the streaming schedule
and against an FP64 transform."""
import re

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import c16_to_c128, need_gpu, rel_l2

pytestmark = pytest.mark.gpu

FP32_MATH = [24, 27, 32, 36, 54, 64, 81, 96, 128, 144, 162, 243, 256]
FP16_MATH = [24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 256, 288, 384, 512, 1024]
CASES = [("fp16", 0, n) for n in FP32_MATH] + [("bf16", 0, n) for n in FP32_MATH] + [("fp16", 4, n) for n in FP16_MATH]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def data(shape, kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = 0.5 * torch.randn(tuple(shape) + (2,), generator=g, device="cuda")
    return x.to(torch.float16 if kind == "fp16" else torch.bfloat16)


def tile(p, axis):
    """Label, columns per tile and words of the pass along `axis`."""
    m = re.search(r" %s\[([^\]]*)\]" % axis, p.describe())
    words = m.group(1).split(" ")
    return words[0], int(next(w for w in words if w.startswith("per="))[4:]), words


def check(got, x, kind, sp, n):
    """(columns, n, 2) device tensors, the pass's output and input."""
    rnd = synth.to_fp16_pairs if kind == "fp16" else synth.to_bf16_pairs
    want = oracle.fft1d_batch(c16_to_c128(x, kind), -1)
    s = 2.0 ** -sp
    floor = rel_l2(synth.pairs_to_c128(rnd(want * s), kind), want * s)
    e = rel_l2(c16_to_c128(got, kind), want * s)
    assert e <= (3.0 * floor if kind == "bf16" else 3e-3), (n, e, floor)


@pytest.mark.parametrize("kind,flags,n", CASES, ids=str)
def test_z_axis(ws, kind, flags, n):
    sp = int(np.ceil(np.log2(n) / 2))
    for nx, ny, few, label in ((192, 192, 192, "strided"), (243, 162, 27, "cached-strided")):
        p = ws.Plan(nx, ny, n, kind, -1, flags)
        lab, per, words = tile(p, "z")
        assert per == 64 and "half" not in words, p.describe()
        if nx == 243:
            assert lab == label, p.describe()
        x = data((n, ny * nx), kind, n)
        y = x.clone()
        p.execute_pass(2, y, y)
        q = ws.Plan(few, 1, n, kind, -1, flags)
        for c0 in (0, 64 * 7, ny * nx - few):
            part = x[:, c0:c0 + few].contiguous()
            q.execute_pass(1, part, part)
            if not flags:   # FP16 arithmetic: the compiler fuses other packed multiply-adds in each tile
                assert torch.equal(part.view(torch.int16), y[:, c0:c0 + few].contiguous().view(torch.int16)), (nx, c0)
            check(y[:, c0:c0 + few].transpose(0, 1).contiguous(), x[:, c0:c0 + few].transpose(0, 1).contiguous(), kind,
                  sp, n)
        g = torch.Generator().manual_seed(n)
        cols = torch.cat([torch.randint(ny * nx, (120,), generator=g), torch.arange(ny * nx - 40, ny * nx)]).cuda()
        check(y[:, cols].transpose(0, 1).contiguous(), x[:, cols].transpose(0, 1).contiguous(), kind, sp, n)


@pytest.mark.parametrize("kind,flags,n", CASES, ids=str)
def test_y_axis(ws, kind, flags, n):
    sp = int(np.ceil(np.log2(n) / 2))
    for nx, nz in ((192, 192), (162, 216)):
        p = ws.Plan(nx, n, nz, kind, -1, flags)
        assert tile(p, "y")[1] == 64 and "half" not in tile(p, "y")[2], p.describe()
        x = data((nz, n, nx), kind, n + 1)
        y = x.clone()
        p.execute_pass(1, y, y)
        q = ws.Plan(nx, n, 1, kind, -1, flags)
        for z in (0, nz // 2, nz - 1):
            part = x[z].clone()
            q.execute_pass(1, part, part)
            if not flags:
                assert torch.equal(part.view(torch.int16), y[z].view(torch.int16)), (nx, z)
            check(y[z].transpose(0, 1).contiguous(), x[z].transpose(0, 1).contiguous(), kind, sp, n)


# arrays of 64 MiB up to 128 MiB: cached x stores, cached y and z; streaming below
@pytest.mark.parametrize("kind,flags", [("fp16", 0), ("bf16", 0), ("fp16", 4)], ids=["fp16", "bf16", "fp16-math"])
@pytest.mark.parametrize("shape,cached", [((256, 256, 256), True), ((512, 512, 64), True), ((512, 512, 96), True),
                                          ((256, 256, 243), False)], ids=str)
def test_cached_range_equals_streaming(ws, kind, flags, shape, cached):
    nx, ny, nz = shape
    x = data((nz, ny, nx), kind, nx + nz)
    p = ws.Plan(nx, ny, nz, kind, -1, flags)
    q = ws.Plan(nx, ny, nz, kind, -1, flags | ws.FLAG_STREAMING)
    want = ("cached-store-contig", "cached-strided", "cached-strided") if cached else ("contig", "strided", "strided")
    assert tuple(part.split(" ")[0] for part in p.describe().split("[")[1:]) == want, p.describe()
    assert "cached" not in q.describe()
    for call in ("execute", "execute_adjoint", "execute_inverse"):
        got, ref = getattr(p, call)(x), getattr(q, call)(x)
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), call
    y, r = x.clone(), x.clone()
    p.execute(y, out=y)
    q.execute(r, out=r)
    assert torch.equal(y.view(torch.int16), r.view(torch.int16))
    want = torch.view_as_real(torch.fft.fftn(torch.view_as_complex(x.double()))) * 2.0 ** -p.scale_log2
    floor = float((want.to(x.dtype).double() - want).norm() / want.norm())
    e = float((p.execute(x).double() - want).norm() / want.norm())
    assert e <= (3.0 * floor if kind == "bf16" else 3e-3), (e, floor)
