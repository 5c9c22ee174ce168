"""The plan of the single-pass kernels on the host (CPU): block tables, variants
and admission as fdtd_create makes them, read through the runtime's own source
without a device (tests/plan/plan_driver.cpp)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    from paper_2609_30039_amd import build as B
    if not os.path.exists(B.LIB):
        B.build()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC,
                        os.path.join(ROOT, "tests", "plan", "plan_driver.cpp"), "-x", "none", B.LIB,
                        "-Wl,-rpath," + os.path.dirname(B.LIB), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def _check(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("ok"), (r.stdout + r.stderr)[-4000:]


def test_blocks_take_a_variant_that_covers_their_nodes(driver):
    """Every node of a block and every neighbour it reads, across a seam too:
    slabs, seams and dispersive cells are in the block's variant; each node has
    one owner; tiles keep the kernels' limits."""
    _check(driver, "masks")


def test_admitted_absorber_memories_fit_their_descriptors(driver):
    """Domains whose absorber memories, rounded up to pairs of x nodes, reach
    2 GiB stay off the single pass (its dropped accesses use that offset); those
    below take it."""
    _check(driver, "spans")


def test_auto_takes_the_measured_route(driver):
    """Which kernels AUTO takes on either side of each line of its rule."""
    _check(driver, "routes")
