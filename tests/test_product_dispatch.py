"""Which kernel, tile and load width a product of any size runs on: the dispatch is host code, so it is asked on the
CPU (``tests/host/product_plan.cpp`` linked against the library; nothing is launched)."""
import os
import subprocess

import pytest

import paper_2105_14450_amd as c3
from paper_2105_14450_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYOUT = {c3.FORM_AB: (1, 0), c3.FORM_ABT: (1, 1), c3.FORM_ATB: (0, 0)}

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="ROCm compiler not found")


@pytest.fixture(scope="session")
def plans(tmp_path_factory):
    c3.binding.load()
    exe = str(tmp_path_factory.mktemp("plan") / "product_plan")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(ROOT, "tests", "host", "product_plan.cpp"), "-x", "none", build.LIB,
                    "-Wl,-rpath," + os.path.dirname(build.LIB), "-Wl,-rpath,/opt/rocm/lib", "-o", exe],
                   check=True, capture_output=True)

    def ask(lines):
        res = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True, timeout=60)
        return [tuple(map(int, line.split())) for line in res.stdout.splitlines()]
    return ask


def plain(dtype, form, m, n, k, batch=1, out=c3.BF16):
    return "plain %d %d %d %d %d %d %d %d" % (dtype, out, *LAYOUT[form], batch, m, n, k)


def test_launches_stay_below_the_grid_limit(plans):
    # 64000 blocks of 1 x 33600: 2^24 tiles of 256 work-items and more do not fit one grid dimension, the element-wise
    # kernel has the batch in another one
    assert plans([plain(c3.BF16, form, 1, 33600, 1, batch=64000) for form in LAYOUT]) == [(0, 0)] * 3
    for tile, piece in plans([plain(c3.BF16, form, 8, 64, 4096, batch=64000) for form in LAYOUT]):
        assert tile and -(-8 // tile) * -(-64 // tile) * 64000 < 1 << 24
