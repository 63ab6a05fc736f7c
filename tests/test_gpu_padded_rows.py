"""C2R x passes over half-spectrum rows with a pitch: even and odd pitches, and
buffers that start one element past an aligned address; fewer rows than a tile
and a tile with a remainder.  NaN in the padding.  Bitwise the compact plan's
result."""
import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu

LENGTHS = [2, 3, 9, 16, 27, 32, 81, 96, 128, 192, 243, 256, 384, 486, 512, 729, 972, 1296, 1944, 2592]


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", LENGTHS)
def test_c2r_rows_with_a_pitch(ws, n, offset):
    nx, w = 2 * n, n + 1
    for rows in (1, 36, 256 if n <= 64 else 27):
        g = torch.Generator(device="cuda").manual_seed(n + rows)
        X = torch.view_as_complex(torch.randn((rows, 1, w, 2), generator=g, device="cuda"))
        want = ws.RealPlan(nx, 1, rows).c2r(X.clone(), inverse=True)
        for pitch in sorted({w + w % 2, w + w % 2 + 2, w + 1 - w % 2, (w + 15) // 16 * 16 + 16}):
            if pitch == w:
                continue
            p = ws.RealPlan(nx, 1, rows, pitch=pitch)
            buf = torch.full((rows * pitch + offset,), float("nan"), dtype=torch.complex64, device="cuda")
            H = buf[offset:].view(rows, 1, pitch)
            H[..., :w] = X
            got = p.c2r(H, inverse=True)
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (n, rows, pitch, offset)
            assert torch.isfinite(got).all()
