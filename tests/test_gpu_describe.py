"""Plan descriptions name what a call launches: half-width tiles, columns run on
across planes, and the tiles of one launch (of one plane chunk where x and y run
in chunks)."""
import re

import pytest

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return need_gpu()


def passes(desc):
    """(label, per, grid, words) of each pass."""
    out = []
    for part in re.findall(r"\[([^\]]*)\]", desc):
        words = part.split(" ")
        num = {k: int(v) for k, v in (w.split("=") for w in words if "=" in w)}
        out.append((words[0], num.get("per"), num["grid"], words))
    return out


def ceil_div(a, b):
    return -(-a // b)


# x, y, z axes; storage; words that the y and z passes carry or not
CASES = [
    ((32, 32, 32), "c64", 8, {"y": {"half"}, "z": {"half"}}),
    ((96, 144, 16), "fp16", 0, {"y": {"half"}, "z": set()}),
    ((96, 54, 64), "c64", 8, {"y": set(), "z": set()}),
    ((324, 96, 96), "fp16", 0, {"y": {"flat", "xcd"}, "z": set()}),
    ((27, 48, 64), "c64", 8, {"y": {"flat", "xcd"}, "z": set()}),
    ((512, 512, 512), "c64", 0, {"y": set(), "z": set()}),
]


@pytest.mark.parametrize("shape,kind,flags,want", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else None)
def test_launches(ws, shape, kind, flags, want):
    nx, ny, nz = shape
    d = ws.Plan(nx, ny, nz, kind, -1, flags).describe()
    m = re.search(r"chunks of (\d+) planes", d)
    planes = int(m.group(1)) if m else nz
    x, y, z = passes(d)
    assert x[2] == ceil_div(ny * planes, x[1]), d
    cols = {"y": (nx, planes), "z": (nx * ny, 1)}
    for name, (label, per, grid, words) in (("y", y), ("z", z)):
        c, outer = cols[name]
        assert grid == (ceil_div(c * outer, per) if "flat" in words else ceil_div(c, per) * outer), (name, d)
        assert want[name] <= set(words), (name, d)
        if "half" in words:
            assert per >= 32 and ceil_div(c, 2 * per) * outer < 512, (name, d)


def test_plane_plan_of_32_cubed(ws):
    plane, z = passes(ws.Plan(32, 32, 32, "c64", -1).describe())
    assert plane[2] == 32
    assert z[1] == 32 and z[2] == 32 and "half" in z[3]   # 1024 columns
