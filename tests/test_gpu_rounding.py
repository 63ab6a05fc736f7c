"""Rounding error of single complex64 (and FP16-arithmetic) passes, relative L2
against FP64 over 2^21 values: no larger than that of the length's schedule
under the radix rules, which the figures below are (two seeds each, within 0.2%
of each other).  The bound allows 0.5%."""
import math

import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu

CONTIG = {108: 9.395e-08, 486: 1.176e-07, 576: 1.075e-07, 648: 1.144e-07, 729: 1.218e-07, 972: 1.211e-07,
          1296: 1.187e-07, 1728: 1.177e-07, 2187: 1.331e-07, 3888: 1.347e-07, 4374: 1.398e-07, 6561: 1.464e-07,
          7776: 1.407e-07, 8748: 1.433e-07}
STRIDED = {324: 1.097e-07, 576: 1.102e-07, 864: 1.138e-07, 1024: 1.091e-07}
SLACK = 1.005


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def normal(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(tuple(shape) + (2,), generator=g, device="cuda")


def error(got, want):
    return float((got.to(torch.complex128) - want).norm() / want.norm())


@pytest.mark.parametrize("n", CONTIG)
def test_contiguous_pass(ws, n):
    rows = (1 << 21) // n
    x = torch.view_as_complex(normal((rows, n), n))
    y = ws.execute_many(ws.Plan(n, 1, 1, "c64", -1), x, torch.empty_like(x), rows)
    assert error(y, torch.fft.fft(x.to(torch.complex128))) <= SLACK * CONTIG[n]


@pytest.mark.parametrize("n", STRIDED)
def test_strided_pass(ws, n):
    m = 1 << int(math.log2((1 << 21) / (32 * n)))
    p = ws.Plan(32, n, m, "c64", -1, ws.FLAG_NO_PLANE)
    x = torch.view_as_complex(normal((m, n, 32), n))
    y = x.clone()
    p.execute_pass(1, x, y)   # the y pass alone, in place on y
    assert error(y, torch.fft.fft(x.to(torch.complex128), dim=1)) <= SLACK * STRIDED[n]


def test_contiguous_pass_fp16_arithmetic(ws):
    n, bound = 729, 1.085e-3
    rows = (1 << 21) // n
    x = (0.5 * normal((rows, n), n)).half()
    p = ws.Plan(n, 1, 1, "fp16", -1, ws.FLAG_FP16_MATH)
    y = ws.execute_many(p, x, torch.empty_like(x), rows)
    want = torch.fft.fft(torch.view_as_complex(x.double())) * 2.0 ** -p.scale_log2
    assert error(torch.view_as_complex(y.double()), want) <= SLACK * bound
