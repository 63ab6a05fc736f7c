"""Strided passes with a measured launch geometry, against the FP64 oracle.

Every length of the geometry tables runs as the y axis (a ragged last tile of
columns at each plane) and as the z axis (flattened columns), both with fewer
columns than a tile and with a tile and a remainder.  Tolerances: complex64
1e-6; 16-bit storage as in the precision tests, 3e-3 (BF16 with rounded
twiddles: 3 one-rounding floors), two passes here."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import c16_to_c128, c16_to_dev, need_gpu, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LENGTHS = [36, 48, 64, 72, 81, 96, 108, 128, 144, 162, 192, 216, 243, 256, 288, 324, 384, 432, 486, 576, 648, 729, 768,
           864, 972, 1024]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def shapes(n):
    """(nx, ny, nz): y axis with 6 and 72 columns, z axis with 27 and 96."""
    return [(6, n, 2), (72, n, 1), (9, 3, n), (48, 2, n)]


@pytest.mark.parametrize("n", LENGTHS)
def test_c64(ws, n):
    for nx, ny, nz in shapes(n):
        a = synth.uniform_c((nz, ny, nx), seed=n + nx).astype(np.complex64)
        p = ws.Plan(nx, ny, nz, "c64", -1)
        got = to_host(p.execute(to_dev(a)))
        e = rel_l2(got, oracle.fftn(a.astype(np.complex128), -1))
        assert e <= 1e-6, (nx, ny, nz, e, p.describe())


@pytest.mark.parametrize("kind,flags", [("fp16", 0), ("bf16", 0), ("fp16", 4)], ids=["fp16", "bf16", "fp16-math"])
@pytest.mark.parametrize("n", LENGTHS)
def test_16bit(ws, n, kind, flags):
    rnd = synth.to_fp16_pairs if kind == "fp16" else synth.to_bf16_pairs
    for nx, ny, nz in shapes(n):
        pairs = rnd(synth.normal_c((nz, ny, nx), seed=n + nx, scale=0.5))
        p = ws.Plan(nx, ny, nz, kind, -1, flags)
        got = c16_to_c128(p.execute(c16_to_dev(pairs, kind)), kind) * 2.0 ** p.scale_log2
        X = oracle.fftn(synth.pairs_to_c128(pairs, kind), -1)
        floor = rel_l2(synth.pairs_to_c128(rnd(X * 2.0 ** -p.scale_log2), kind) * 2.0 ** p.scale_log2, X)
        e = rel_l2(got, X)
        assert e <= (3.0 * floor if kind == "bf16" else 3e-3), (nx, ny, nz, e, floor, p.describe())
