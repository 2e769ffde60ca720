import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

GOLDEN = os.path.join(ROOT, "tests", "golden")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


def read_golden(name):
    """key = values fixture -> dict of float lists (comments start with #)."""
    out = {}
    with open(os.path.join(GOLDEN, name)) as f:
        for line in f:
            line = line.split("#", 1)[0].strip()
            if not line or "=" not in line:
                continue
            k, v = line.split("=", 1)
            out[k.strip()] = [float(t) for t in v.split()]
    return out


@pytest.fixture
def golden():
    return read_golden


def training_path(pop, train):
    """Runs train(), the first training of a new population, and names the
    kernels that it ran on, from the launches that the library counts: "fused"
    (whole steps in one launch), "streamed n" (n hidden layers on the streaming
    kernel, which has two launches for each layer's register image and mask
    words made first) or "tiles"."""
    pop.set_profiling(True)
    before = pop.kernel_stats()
    train()
    after = pop.kernel_stats()
    pop.set_profiling(False)
    n = {k: after[k][1] - before[k][1] for k in after}
    if n["fused_train"]:
        return "fused"
    assert n["layer_train"] > 0
    images = n["aux"] - 1                                # beside the launch that clears the epoch's sums
    return "streamed %d" % (images // 2) if images else "tiles"
