"""The C ABI's host code (cmflb_capi.hip) against a runtime without a device
(capi_host_driver.hip): what it allocates, captures and launches for calls
whose effect a GPU test does not show.  CPU only; built with the address
sanitizer where the toolchain has it."""
import os
import subprocess

import pytest

from paper_2602_16486_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    try:
        cxx = build.clangxx()
    except RuntimeError as e:
        pytest.skip(str(e))
    tmp = tmp_path_factory.mktemp("capi_host")
    exe = str(tmp / "driver")
    flags = ["-x", "hip", "--offload-host-only", f"--offload-arch={build.ARCH}", "-O1", "-g",
             "-std=c++17", "-Wno-unused-function", "-Wno-option-ignored"]
    objs = []
    # one cuid-less object may hold the fat binary's plain symbol names
    for src, cuid in ((os.path.join(ROOT, "paper_2602_16486_amd", "csrc", "cmflb_capi.hip"), "none"),
                      (os.path.join(ROOT, "tests", "capi_host_driver.hip"), "hash")):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        subprocess.run([cxx, *flags, "-Xarch_host", "-fsanitize=address", f"-fuse-cuid={cuid}",
                        "-c", src, "-o", objs[-1]], check=True)
    subprocess.run([cxx, "-Xarch_host", "-fsanitize=address", *objs, "-o", exe, "-lpthread"], check=True)

    def run(what):
        r = subprocess.run([exe, what], capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1:exitcode=23"))
        assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
        lines = r.stdout.split("\n")
        # graph executables, streams, events, device and pinned bytes at the end
        assert "left 0 0 0 0 0" in lines, r.stdout
        return lines
    return run


def test_graphs_are_captured_at_most_once_per_parity(driver):
    """A lattice or ensemble whose captured graphs were dropped by a new shape
    takes direct steps from then on: at most one capture per buffer parity
    in its life, every step taken, and graphs as before where the shape was
    set before the first run."""
    out = dict(line.split(" captures ") for line in driver("graphs") if " captures " in line)
    assert int(out["lattice"]) <= 2 and int(out["ensemble"]) <= 2
    assert out["tuned"] == "1 launches 10"


def test_untuned_launches_and_their_partial_sums_are_bounded(driver):
    """One tile per workgroup only while the grid is one that the runtime
    launches (below 2^32 threads) and the partial sums take at most 256 MB or
    1/64 of the populations: boxes of one or few sites per row have as many
    tiles as rows.  The tuner launches no larger grid either."""
    boxes = [line.split() for line in driver("shapes") if line.startswith("box ")]
    assert len(boxes) > 80
    for b in boxes:
        v = dict(zip(b[5::2], map(int, b[6::2])))
        assert 0 < v["threads"] < 2 ** 32 and v["tuner"] < 2 ** 32, b
        # (and series, second-level rows and the step counter: under 2 MB)
        assert v["beside"] <= max(256 << 20, v["population"] // 64) + (2 << 20), b
    full = [b for b in boxes if b[1:5] == ["27", "1024", "1024", "1024"] and b[6] == "1" and b[8] == "0"]
    assert full and all(b[12] == str(1024 ** 3 // 256) for b in full)  # one tile per workgroup


def test_large_copies_survive_failing_allocations(driver):
    """Whichever host allocation of a large copy fails, the copy is made (by
    fewer threads or the runtime alone) and nothing is thrown."""
    out = dict(line.split(" failed ") for line in driver("allocations") if " failed " in line)
    assert int(out["allocations"]) >= 6  # the chunk flags, the thread list, four threads


def test_pinned_memory_is_bounded_and_given_back(driver):
    """Forty lattices and an ensemble share the pinned chunks of their large
    copies: one set of 24 MB in turn, at most four sets in ten threads, none
    once all of them are destroyed."""
    out = dict(line[7:].rsplit(" ", 1) for line in driver("pinned") if line.startswith("pinned "))
    assert int(out["in turn"]) == 24 << 20
    assert int(out["at once"]) <= 4 * (24 << 20)
    assert int(out["after"]) == 0


def test_workgroup_sizes_of_untuned_lattices(driver):
    """Ragged D2Q9 boxes keep 256 threads unless a tenth and more of the lanes
    would idle, and 3-D boxes of few tiles take 64: both measured faster than
    the fewest lanes."""
    got = {tuple(line.split()[1:4]): int(line.split()[4]) for line in driver("blocks") if line.startswith("block ")}
    want = {("9", "1030x900x1", "0"): 256, ("9", "1030x900x1", "1"): 256, ("9", "600x600x1", "0"): 128,
            ("27", "64x64x1", "1"): 64, ("27", "32x32x32", "1"): 64, ("19", "12x14x17", "2"): 64,
            ("27", "50x50x50", "1"): 256, ("27", "256x256x256", "1"): 256}
    assert {k: got[k] for k in want} == want
    assert got["9", "1290x800x1", "0"] != 64
