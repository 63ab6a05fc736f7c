"""Performance cases: the transforms that programs run with this library, over the range of sizes it takes.

Every case names a family (``kind``), its sizes and its options:

* ``c2c``      one 3D complex transform on a kept plan (complex64, or FP16 / BF16 storage): ``forward`` alone or
               a ``round trip`` (forward, then the exact inverse), into buffers the program keeps;
* ``grad``     the differentiable transform inside a training step: the value and the input gradient;
* ``image``    one 2D plan over a stack of complex64 images stored back to back;
* ``signal``   one 1D plan over a stack of complex64 signals stored back to back;
* ``real``     a real FP32 array to its half spectrum and back: ``plan`` on a kept plan, where the inverse
               consumes the spectrum (it overwrites it), or ``function``, the functional pair that keeps it;
* ``poisson``  the spectral Poisson solve and its gradient (the paper's transform inside a loss);
* ``batch``    many arrays of uneven shapes in one call.

Sizes are nx (fastest), ny, nz.  Every axis length of the library is 2^a 3^b, so the odd sizes are those with
radix-3 factors and rows that are no whole cache lines.
"""
import math

import torch

from paper_2209_15040_amd import binding as wsfft

# 2^a 3^b up to 2^18
SMOOTH = sorted(2 ** a * 3 ** b for a in range(19) for b in range(12) if 2 ** a * 3 ** b <= 1 << 18)
# the lengths programs choose most: powers of two and three times one
COMMON = [n for n in SMOOTH if n & (n - 1) == 0 or (n % 3 == 0 and (n // 3) & (n // 3 - 1) == 0)]
# axis lengths of the uneven batches
BATCH_AXES = (32, 64, 96, 128, 256)


def listed():
    return [
        # the smallest array the library is used on alone (latency and launches count): the paper's 32^3
        {"name": "c64-32cubed", "kind": "c2c", "dtype": "c64", "nx": 32, "ny": 32, "nz": 32, "op": "round trip"},
        # an ordinary simulation grid, one step of a spectral solver
        {"name": "c64-128cubed", "kind": "c2c", "dtype": "c64", "nx": 128, "ny": 128, "nz": 128, "op": "round trip"},
        # a grid with radix-3 axes and rows of no whole cache lines, inside a training step
        {"name": "grad-324x288x216", "kind": "grad", "nx": 324, "ny": 288, "nz": 216},
        # the paper's headline size: 512^3 forward and back
        {"name": "c64-512cubed", "kind": "c2c", "dtype": "c64", "nx": 512, "ny": 512, "nz": 512, "op": "round trip"},
        # the largest cube (8 GiB per array)
        {"name": "c64-1024cubed", "kind": "c2c", "dtype": "c64", "nx": 1024, "ny": 1024, "nz": 1024, "op": "forward"},
        # 16-bit storage with FP32 arithmetic at the headline size
        {"name": "fp16-512cubed", "kind": "c2c", "dtype": "fp16", "nx": 512, "ny": 512, "nz": 512, "op": "round trip"},
        # 16-bit storage on a grid of odd and radix-3 axes
        {"name": "bf16-288x243x256", "kind": "c2c", "dtype": "bf16", "nx": 288, "ny": 243, "nz": 256, "op": "round trip"},
        # one large image; its y axis takes two passes
        {"name": "image-8192sq", "kind": "image", "nx": 8192, "ny": 8192, "count": 1},
        # long signals, each in two passes
        {"name": "signal-65536x1024", "kind": "signal", "nx": 65536, "count": 1024},
        # real data at the headline size, to the half spectrum and back
        {"name": "real-512cubed", "kind": "real", "api": "plan", "nx": 512, "ny": 512, "nz": 512},
        # the Poisson loss: solution and gradient on a 256^3 grid
        {"name": "poisson-256cubed", "kind": "poisson", "nx": 256, "ny": 256, "nz": 256},
        # many uneven arrays side by side in one call (1 GiB of input)
        {"name": "batch-96", "kind": "batch", "count": 96, "shapes": 3},
    ]


def _axis(rng, lo, hi, even=False):
    """A length in [lo, hi], spread over its logarithm: half of them common ones, half any 2^a 3^b."""
    t = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    ok = [n for n in (COMMON if rng.random() < 0.5 else SMOOTH) if lo <= n <= hi and not (even and n % 2)]
    return min(ok, key=lambda n: abs(math.log(n / t)))


def _grid(rng, lo, hi, most, even_x=False):
    while True:
        nx, ny, nz = _axis(rng, lo, hi, even_x), _axis(rng, lo, hi), _axis(rng, lo, hi)
        if nx * ny * nz <= most:
            return {"nx": nx, "ny": ny, "nz": nz}


def draw(rng):
    kind = rng.choice(("c2c", "c2c", "c2c16", "c2c16", "grad", "image", "signal", "real", "real", "poisson", "batch"))
    if kind == "c2c":
        return {"kind": "c2c", "dtype": "c64", **_grid(rng, 32, 1024, 1 << 27), "op": rng.choice(("forward", "round trip"))}
    if kind == "c2c16":
        return {"kind": "c2c", "dtype": rng.choice(("fp16", "bf16", "fp16-math")), **_grid(rng, 32, 512, 1 << 27),
                "op": rng.choice(("forward", "round trip"))}
    if kind == "grad":
        return {"kind": "grad", **_grid(rng, 32, 512, 1 << 26)}
    if kind == "image":
        nx, ny = _axis(rng, 128, 8192), _axis(rng, 128, 8192)
        most = max(1, (1 << 26) // (nx * ny))
        return {"kind": "image", "nx": nx, "ny": ny, "count": min(64, max(1, round(math.exp(rng.uniform(0, math.log(most))))))}
    if kind == "signal":
        nx = _axis(rng, 64, 262144)
        most = (1 << 26) // nx
        return {"kind": "signal", "nx": nx, "count": max(1, round(most * math.exp(-rng.uniform(0, math.log(256)))))}
    if kind == "real":
        return {"kind": "real", "api": rng.choice(("plan", "function")), **_grid(rng, 32, 768, 1 << 27, even_x=True)}
    if kind == "poisson":
        return {"kind": "poisson", **_grid(rng, 32, 512, 1 << 25, even_x=True), "nz": rng.choice((32, 64, 128, 256))}
    return {"kind": "batch", "count": rng.randint(6, 96), "shapes": rng.randint(4, 1 << 20)}


def _batch_shapes(case):
    """(nx, ny, nz) of each array: axes drawn from BATCH_AXES, cubes drawn again."""
    g = torch.Generator().manual_seed(case["shapes"])
    out = []
    while len(out) < case["count"]:
        s = [BATCH_AXES[i] for i in torch.randint(len(BATCH_AXES), (3,), generator=g).tolist()]
        if len(set(s)) > 1:
            out.append(tuple(s))
    return out


def _normal(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


def _complex(shape, seed):
    return torch.view_as_complex(_normal(tuple(shape) + (2,), seed))


def _inputs(case, seed):
    kind = case["kind"]
    if kind == "image":
        return _complex((case["count"], case["ny"], case["nx"]), seed)
    if kind == "signal":
        return _complex((case["count"], case["nx"]), seed)
    if kind == "batch":
        return _complex((sum(x * y * z for x, y, z in _batch_shapes(case)),), seed)
    shape = (case["nz"], case["ny"], case["nx"])
    if kind in ("real", "poisson"):
        return _normal(shape, seed)
    if case.get("dtype", "c64") == "c64":
        return _complex(shape, seed)
    return (0.5 * _normal(shape + (2,), seed)).to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float16)


def _plan16(case):
    math16 = case["dtype"] == "fp16-math"
    return wsfft.Plan(case["nx"], case["ny"], case["nz"], "bf16" if case["dtype"] == "bf16" else "fp16", -1,
                      wsfft.FLAG_FP16_MATH if math16 else 0)


def prepare(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    s = {"case": case, "x": x}
    if kind == "c2c":
        s["plan"] = wsfft.Plan(case["nx"], case["ny"], case["nz"], "c64", -1) if case["dtype"] == "c64" else _plan16(case)
        s["y"] = torch.empty_like(x)
        if case["op"] == "round trip":
            s["back"] = torch.empty_like(x)
    elif kind == "grad":
        s["w"] = _complex(x.shape, seed + (1 << 30))
        x.requires_grad_(True)
    elif kind == "image":
        s["plan"], s["y"] = wsfft.Plan(case["nx"], case["ny"], 1, "c64", -1), torch.empty_like(x)
    elif kind == "signal":
        s["plan"], s["y"] = wsfft.Plan(case["nx"], 1, 1, "c64", -1), torch.empty_like(x)
    elif kind == "real" and case["api"] == "plan":
        s["plan"] = wsfft.RealPlan(case["nx"], case["ny"], case["nz"])
        s["half"] = torch.empty(s["plan"].half_shape(x.shape), dtype=torch.complex64, device=x.device)
        s["back"] = torch.empty_like(x)
    elif kind == "poisson":
        s["w"] = _normal(x.shape, seed + (1 << 30))
        x.requires_grad_(True)
    elif kind == "batch":
        shapes = _batch_shapes(case)
        plans = {q: wsfft.Plan(*q, "c64", -1) for q in sorted(set(shapes))}
        y = torch.empty_like(x)
        s["y"], s["plans"], s["ins"], s["outs"] = y, [plans[q] for q in shapes], [], []
        at = 0
        for nx, ny, nz in shapes:
            n = nx * ny * nz
            s["ins"].append(x[at:at + n].view(nz, ny, nx))
            s["outs"].append(y[at:at + n].view(nz, ny, nx))
            at += n
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "c2c":
        s["plan"].execute(s["x"], s["y"])
        if case["op"] == "forward":
            return s["y"]
        s["plan"].execute_inverse(s["y"], s["back"])
        return s["y"], s["back"]
    if kind == "grad":
        y = wsfft.FFTn.apply(s["x"], -1)
        (g,) = torch.autograd.grad(y, s["x"], s["w"])
        return y, g
    if kind in ("image", "signal"):
        return wsfft.execute_many(s["plan"], s["x"], s["y"], case["count"])
    if kind == "real" and case["api"] == "plan":
        s["plan"].r2c(s["x"], s["half"])
        return s["plan"].c2r(s["half"], s["back"], inverse=True)   # the spectrum is consumed
    if kind == "real":
        half = wsfft.rfftn(s["x"])
        return half, wsfft.irfftn(half, case["nx"])
    if kind == "poisson":
        u = wsfft.poisson_solve(s["x"])
        (g,) = torch.autograd.grad(u, s["x"], s["w"])
        return u, g
    wsfft.execute_batched(s["plans"], s["ins"], s["outs"])
    return s["y"]


def work(case):
    """Bytes of every input read once and every output written once per call, and 5 N log2 N per complex transform."""
    kind = case["kind"]
    if kind == "batch":
        n = [x * y * z for x, y, z in _batch_shapes(case)]
        return {"bytes": 16 * sum(n), "flops": sum(5 * m * math.log2(m) for m in n)}
    axes = case["nx"] * case.get("ny", 1) * case.get("nz", 1)
    flops = 5 * axes * math.log2(axes)
    if kind in ("image", "signal"):
        return {"bytes": 16 * axes * case["count"], "flops": flops * case["count"]}
    if kind == "grad":
        return {"bytes": 2 * 16 * axes, "flops": 2 * flops}
    if kind == "real":
        half = (case["nx"] // 2 + 1) * case["ny"] * case["nz"]
        return {"bytes": 2 * (4 * axes + 8 * half), "flops": flops}
    if kind == "poisson":
        return {"bytes": 2 * 8 * axes, "flops": 2 * flops}
    calls = 2 if case["op"] == "round trip" else 1
    return {"bytes": calls * (16 if case["dtype"] == "c64" else 8) * axes, "flops": calls * flops}


def _poisson64(f):
    """Re(IFFT(-FFT(f) / |k|^2)) on [0, 2 pi)^3, the k = 0 mode dropped."""
    nz, ny, nx = f.shape
    k = [torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=f.device) for n in (nz, ny, nx)]
    k2 = k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2
    m = torch.where(k2 > 0, -1.0 / k2, torch.zeros_like(k2))
    return torch.fft.ifftn(torch.fft.fftn(f) * m).real.contiguous()


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "batch":
        out, at = [], 0
        for nx, ny, nz in _batch_shapes(case):
            n = nx * ny * nz
            out.append(torch.fft.fftn(x[at:at + n].view(nz, ny, nx).to(torch.complex128)).reshape(-1))
            at += n
        return torch.cat(out)
    if kind == "poisson":
        return _poisson64(x.double()), _poisson64(_normal(x.shape, seed + (1 << 30)).double())
    if kind == "real":
        x64 = x.double()
        return x64 if case["api"] == "plan" else (torch.fft.rfftn(x64), x64)
    if kind == "image":
        return torch.fft.fft2(x.to(torch.complex128))
    if kind == "signal":
        return torch.fft.fft(x.to(torch.complex128))
    if kind == "grad":
        w = _complex(x.shape, seed + (1 << 30))
        n = x.numel()
        return torch.fft.fftn(x.to(torch.complex128)), torch.fft.ifftn(w.to(torch.complex128)) * n
    if case["dtype"] == "c64":
        x64 = x.to(torch.complex128)
        y = torch.fft.fftn(x64)
        return y if case["op"] == "forward" else (y, x64)
    # 16-bit plans store 2^-S times the transform, S the sum of ceil(log2(n) / 2) over the axes
    S = sum(math.ceil(math.log2(case[a]) / 2) for a in ("nx", "ny", "nz"))
    y = torch.view_as_real(torch.fft.fftn(torch.view_as_complex(x.double())) * 2.0 ** -S)
    return y if case["op"] == "forward" else (y, x.double())
