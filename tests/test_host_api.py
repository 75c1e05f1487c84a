"""Host side of the C ABI without a GPU: its sources linked with a stand-in
for the HIP runtime and the launchers (tests/host_runtime.h), where failures
can be forced and calls counted."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_03920_amd", "csrc")


def run(tmp_path, program, sources):
    exe = str(tmp_path / "program")
    # launchers that a program does not define are not called by it
    subprocess.run(["g++", "-std=c++17", "-O1", "-no-pie", "-D__HIP_PLATFORM_AMD__", "-isystem",
                    "/opt/rocm/include", os.path.join(ROOT, "tests", program),
                    *(os.path.join(CSRC, s) for s in sources), "-o", exe, "-lquadmath", "-pthread",
                    "-Wl,--unresolved-symbols=ignore-all"], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=60)


def test_readings_without_pinned_memory(tmp_path):
    """A reading never fails for want of pinned memory: groups are copied one
    by one, with the same result."""
    r = run(tmp_path, "host_readings.cpp", ["qsg_api.cpp", "qsg_tables.cpp"])
    assert r.returncode == 0, r.stdout


def test_eigensolves_keep_their_pinned_memory(tmp_path):
    """To give pinned memory back waits for all streams of the device, so it
    is not done from solve to solve; a solve can do without."""
    r = run(tmp_path, "host_lanczos.cpp", ["qsg_transfer_api.cpp"])
    assert r.returncode == 0, (r.returncode, r.stdout)


def test_level_entries_are_handlers(tmp_path):
    """The colour pass jumps to the offsets of a slot's level entries: the
    host builds none but starts of handlers, and runs no slot without."""
    r = run(tmp_path, "host_ladders.cpp", ["qsg_api.cpp", "qsg_tables.cpp"])
    assert r.returncode == 0, (r.returncode, r.stdout)


def test_energy_walk_depths(tmp_path):
    """Few large slots get deep walks: their waves add to the same counters."""
    r = run(tmp_path, "host_energy_walks.cpp", [])
    assert r.returncode == 0, (r.returncode, r.stdout)
