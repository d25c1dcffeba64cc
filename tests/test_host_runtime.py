"""What the library asks the HIP runtime for when it reads results back, on the CPU: a C
program links libodb.so and stands in for the runtime's functions (tests/host/host_runtime.c)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2606_19989_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def asked(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_runtime")
    r = subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-Wextra", "-Werror", "-D_GNU_SOURCE",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROCM, "include"),
                        os.path.join(HERE, "host", "host_runtime.c"), "-o", exe, "-rdynamic", "-pthread",
                        "-L", PKG, "-l:libodb.so", "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                        "-Wl,-rpath," + PKG, "-Wl,-rpath," + os.path.join(ROCM, "lib")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(mode):
        r = subprocess.run([exe, mode], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
        return {k: int(v) for k, v in (line.split() for line in r.stdout.splitlines())}
    return run


def test_read_page_is_coherent(asked):
    """The page that kernels write and the host reads behind an event is coherent memory: its
    visibility then rests on the kernel's system-scope fence, not on an environment variable
    or on what an event releases.  The page and the event go when their thread ends."""
    a = asked("page")
    assert a["status"] == 0
    assert a["page_coherent"] == 1 and a["page_portable"] == 1 and a["event_untimed"] == 1
    assert (a["pages"], a["pages_freed"], a["events"], a["events_freed"]) == (1, 1, 1, 1)
    assert a["event_waits"] == 2 and a["stream_waits"] == 1 and a["copies"] == 0


def test_reads_without_a_pinned_page(asked):
    """Without pinned memory every result comes by a pageable copy and a wait for the stream."""
    a = asked("nopage")
    assert a["status"] == 0
    assert (a["pages"], a["pages_freed"], a["events"]) == (0, 0, 0)
    assert a["event_waits"] == 0 and a["copies"] == 3 and a["stream_waits"] == 3
