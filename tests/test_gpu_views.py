"""irfftn of inputs whose conjugation, negation or strides are still pending (a
lazily conjugated tensor is contiguous and shares its memory with the one that
is not): bitwise the result of the materialised input, and complex64 within
1e-6 of the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import need_gpu, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


VIEWS = {
    "conj": lambda X: X.conj(),
    "neg": lambda X: torch._neg_view(X),
    "conj of neg": lambda X: torch._neg_view(X).conj(),
    "transposed": lambda X: X.transpose(0, 1).contiguous().transpose(0, 1),
    "conj transposed": lambda X: X.transpose(0, 1).contiguous().transpose(0, 1).conj(),
    "sliced": lambda X: torch.cat([X, X], dim=-1)[..., :X.shape[-1]],
    "conj sliced": lambda X: torch.cat([X, X], dim=-1)[..., :X.shape[-1]].conj(),
}


@pytest.mark.parametrize("view", VIEWS, ids=str)
@pytest.mark.parametrize("shape", [(64, 1, 1), (36, 27, 4), (512, 6, 2)], ids=str)
def test_irfftn_of_views(ws, shape, view):
    nx, ny, nz = shape
    a = synth.normal_c((nz, ny, nx // 2 + 1), seed=nx).astype(np.complex64)
    X = VIEWS[view](to_dev(a))
    before = X.clone()
    got = ws.irfftn(X, nx)
    assert torch.equal(torch.view_as_real(X.clone()), torch.view_as_real(before))
    want = ws.irfftn(before, nx)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    ref = oracle.irfftn(before.cpu().numpy().astype(np.complex128), nx) / (nx * ny * nz)
    assert rel_l2(to_host(got), ref) <= 1e-6
