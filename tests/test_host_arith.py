"""Host checks of the device code's index arithmetic at the edges of the accepted sizes: a small program on the
library's own headers, compiled for the host alone."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(tmp_path, body, includes):
    """Output of a program that includes `includes` and runs `body` in its main()."""
    src, exe = tmp_path / "check.hip", tmp_path / "check"
    src.write_text("".join(f'#include "{i}"\n' for i in includes)
                   + "#include <cstdio>\nusing namespace tcx;\nint main() {\n" + body + "\nreturn 0; }\n")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "paper_1804_06926_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True, capture_output=True, text=True, timeout=110)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()


M_MAX = (1 << 31) - (1 << 20)   # kept edges at most


@pytest.mark.parametrize("form,ends", [
    ("false", [0, 1, 1 << 30, M_MAX - 1, M_MAX]),                                   # the oriented columns
    ("true", [0, 1, (1 << 31) - 1, 1 << 31, (1 << 31) + 1900, (1 << 32) - (1 << 21)]),   # the symmetric adjacency, 2m
])
def test_entry_ends(tmp_path, form, ends):
    """An in-edge entry gives back the start and the end it was made of: positions in the oriented columns beside
    the group mark, positions in the symmetric adjacency over their whole range."""
    body = ""
    for end in ends:
        start = max(end - 400, 0)
        for mark in (["0ull"] if form == "true" else ["0ull", "CSC_FOLLOWS"]):
            body += (f"{{ const uint64_t e = ({start}ull | {end}ull << 32) | {mark};"
                     f' printf("%u %u\\n", tail_start(e), tail_end(e, {form})); }}\n')
    got = [int(x) for x in run_host(tmp_path, body, ["internal.h"])]
    want = []
    for end in ends:
        want += [max(end - 400, 0), end] * (1 if form == "true" else 2)
    assert got == want


def test_stretches_of_a_bucket(tmp_path):
    """Stretches of a bucket of endpoints: the exact quotient rounded up, up to all 2E endpoints of the largest
    edge list in one bucket and the stretch length that it gets."""
    largest = 2 * M_MAX
    sizes = [0, 1, 8191, 8192, 8193, 1 << 31, largest - 1, largest]
    chunks = [8192, 8193, 3 * largest // 512, 3 * largest // (2 * 8192)]
    body = "".join(f'printf("%u\\n", stretches({s}u, {c}u));\n' for s in sizes for c in chunks)
    assert [int(x) for x in run_host(tmp_path, body, ["internal.h"])] == [-(-s // c) for s in sizes for c in chunks]
