"""Contiguous passes whose tiles go through LDS as one range (and the measured
contiguous geometries), against the FP64 oracle: every length of the tables,
with fewer pencils than a tile, several tiles and a ragged one, packed rows on
16-byte boundaries and rows that start one element past one; half spectra with
compact and padded rows.  Tolerances: complex64 1e-6 (round trip 2e-6); 16-bit
storage as in the precision tests, 3e-3 (BF16 with rounded twiddles: 3
one-rounding floors), one pass here."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import c16_to_c128, c16_to_dev, need_gpu, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 4, 6, 8, 9, 12, 16, 18, 24, 27, 32, 36, 48, 54, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256,
           288, 324, 384, 432, 486, 512, 576, 648, 729, 768, 864, 972, 1024, 1296, 1458, 1728, 1944, 2048, 2187, 2304,
           2592, 2916, 3456, 3888, 4096, 4374, 4608, 5184, 6561, 7776, 8192, 8748, 9216, 10368, 11664,
           12288, 13122, 15552]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def offset(t, off):
    """The same values in a buffer that starts `off` complex elements past an aligned address."""
    flat = t.reshape(-1)
    per = 2 if t.dtype != torch.complex64 and t.shape[-1] == 2 else 1
    buf = torch.empty(flat.numel() + off * per, dtype=t.dtype, device=t.device)
    view = buf[off * per:].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("n", LENGTHS)
def test_c64(ws, n):
    for rows in (1, 5, 300 if n <= 512 else 11):
        a = synth.uniform_c((rows, n), seed=n + rows).astype(np.complex64)
        want = oracle.fft1d_batch(a.astype(np.complex128), -1)
        p = ws.Plan(n, 1, 1, "c64", -1)
        for off in (0, 1):
            x = offset(to_dev(a), off)
            y = offset(torch.zeros_like(x), off)
            ws.execute_many(p, x, y, rows)
            e = rel_l2(to_host(y), want)
            assert e <= 1e-6, (n, rows, off, e, p.describe())


@pytest.mark.parametrize("kind,flags", [("fp16", 0), ("bf16", 0), ("fp16", 4)], ids=["fp16", "bf16", "fp16-math"])
@pytest.mark.parametrize("n", [m for m in LENGTHS if m <= 2048])
def test_16bit(ws, n, kind, flags):
    rnd = synth.to_fp16_pairs if kind == "fp16" else synth.to_bf16_pairs
    for rows in (5, 131):
        pairs = rnd(synth.normal_c((rows, n), seed=n + rows, scale=0.5))
        p = ws.Plan(n, 1, 1, kind, -1, flags)
        X = oracle.fft1d_batch(synth.pairs_to_c128(pairs, kind), -1)
        floor = rel_l2(synth.pairs_to_c128(rnd(X * 2.0 ** -p.scale_log2), kind) * 2.0 ** p.scale_log2, X)
        for off in (0, 1):
            x = offset(c16_to_dev(pairs, kind), off)
            y = offset(torch.zeros_like(x), off)
            ws.execute_many(p, x, y, rows)
            e = rel_l2(c16_to_c128(y, kind) * 2.0 ** p.scale_log2, X)
            assert e <= (3.0 * floor if kind == "bf16" else 3e-3), (n, rows, off, e, floor, p.describe())


@pytest.mark.parametrize("n", [m for m in LENGTHS if m <= 1458 or m in (5184, 8192, 9216, 12288, 13122)])
def test_real(ws, n):
    nx = 2 * n
    for rows, pitch in ((1, 0), (36, 0), (18, (n + 1 + 15) // 16 * 16), (6, n + 4)):
        a = synth.normal_c((rows, nx), seed=n + rows).real.astype(np.float32)
        p = ws.RealPlan(nx, 1, rows, pitch=pitch)
        x = torch.from_numpy(a).cuda().reshape(rows, 1, nx)
        want = oracle.rfftn(a.astype(np.float64).reshape(rows, 1, nx))
        h = p.r2c(x)
        e = rel_l2(to_host(h)[..., :n + 1], want)
        assert e <= 1e-6, (nx, rows, pitch, e, p.describe())
        back = p.c2r(h, inverse=True)
        e = rel_l2(to_host(back), a.reshape(rows, 1, nx))
        assert e <= 2e-6, (nx, rows, pitch, e, p.describe())
