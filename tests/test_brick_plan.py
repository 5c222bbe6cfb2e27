"""Tiles of cells as the host plans them (brick_plan_host.cpp, linked with the
library's objects): run on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    from paper_1105_5613_amd import build, md
    if not os.path.exists(md.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("plan") / "brick_plan_host")
    pkg = os.path.dirname(md.LIB_PATH)
    common = [f for f in build.COMMON if f != "-Werror" and not f.startswith("-O")]
    r = subprocess.run([build.HIPCC, "-O1", *common, "-Wno-unused-function",
                        os.path.join(ROOT, "tests", "brick_plan_host.cpp"), "-x", "none",
                        md.LIB_PATH, f"-Wl,-rpath,{pkg}", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, (args, r.returncode, r.stdout, r.stderr)
        return r.stdout
    return run


@pytest.mark.parametrize("n,rho,fill", [(131072, 1.0, 0.85), (262144, 1.0, 0.9),
                                        (65536, 1.2, 0.84), (1048576, 0.9, 0.88)])
def test_empty_tiles_read_no_particle(plan, n, rho, fill):
    """Boxes with a void at the top: their last tiles hold no home particles and
    their home rows start past the last particle."""
    print(plan("empty", n, rho, fill))


@pytest.mark.parametrize("n,rho,tiles", [(1 << 20, 1.2, True), (1 << 20, 0.05, True),
                                         (900000000, 1.2, True), (1 << 30, 0.05, False)])
def test_list_free_launches_fit_a_grid(plan, n, rho, tiles):
    """At 900,000,000 particles the threads of a launch pass 2^31; a dilute box
    of 2^30 would pass 2^32 and takes row tiles."""
    out = plan("grid", n, rho)
    print(out)
    assert ("tiles of" in out) == tiles


@pytest.mark.parametrize("n,rho,cap,tiles", [
    (4000, 1.2, 0, True), (1 << 20, 1.2, 0, True), (1 << 24, 1.2, 0, True),
    (1 << 26, 1.2, 0, True), (1 << 26, 0.6, 0, True), (6000, 1.2, 2400000, True),
    (1 << 20, 1.2, 2 ** 31 - 1, True), (1 << 26, 1.2, 4000, False)])
def test_rows_of_a_tile_within_32_bits(plan, n, rho, cap, tiles):
    """The force kernel addresses the list from a tile's first row with 32
    bits: rows are never given more chunks than a neighbourhood has entries
    for, and boxes where that is not enough keep gather lists."""
    out = plan("span", n, rho, cap)
    print(out)
    assert ("tiles of" in out) == tiles
