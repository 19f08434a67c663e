"""Checks of the native library on the host, by a program that stands in for the HIP runtime (host_checks.cpp)."""

import os
import re
import struct
import subprocess
import tempfile

import pytest

import paper_2411_15100_amd as xgm
from paper_2411_15100_amd import build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_checks(tmp_path_factory):
    xgm.load_library()  # (built if it is not)
    out = str(tmp_path_factory.mktemp("host_checks") / "host_checks")
    include = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-Wall", "-rdynamic", "-pthread", "-D__HIP_PLATFORM_AMD__", "-isystem", include,
                    os.path.join(HERE, "host_checks.cpp"), "-o", out, "-ldl"], check=True)

    def run(*what, text=""):
        done = subprocess.run([out, lib_build.LIB, *map(str, what)], input=text, capture_output=True, text=True, timeout=120)
        assert done.returncode == 0, done.stdout + done.stderr
        return done.stdout

    return run


def test_a_build_ends_where_a_copy_cannot_be_launched(host_checks):
    host_checks("moves")


def test_copies_that_are_too_many_for_a_launch_are_refused(host_checks):
    host_checks("too_many_moves")


def nested_grammar(rules, digits=0):
    """Nested brackets, next to a chain of rules that does nothing but make the tables larger: 42 bytes a rule."""
    text = 'root ::= n | "<" c0 | "=" e\nn ::= "(" m ")"\nm ::= n | [a-z]* | "1"\ne ::= "e"' + " ([0-9] | n)" * digits + "\n"
    return text + "".join(f'c{k} ::= "a" c{k + 1}\n' for k in range(rules)) + f'c{rules} ::= "z"\n'


# (rules, digits) of which the tables in front of the headers are exactly as large as the room that a fill (31 KB) or an
# accept (64 KB) has for tables
EXACT = {31 * 1024: (743, 0), 64 * 1024: (1547, 1)}


def test_tables_that_count_as_staged_have_a_header_staged(host_checks):
    host_checks("staging")


@pytest.mark.parametrize("room", EXACT)
def test_grammars_whose_tables_fill_the_room_exactly(host_checks, room):
    assert int(host_checks("headers", text=nested_grammar(*EXACT[room])).split()[0]) == room


def many_rules(n):
    return "root ::= " + " | ".join(f"f{k}" for k in range(n)) + "\n" + "".join(f'f{k} ::= "{chr(97 + k % 26) * 110}{k}"\n' for k in range(n))


@pytest.mark.parametrize("cpus, callers, most", [(1, 1, 0), (1, 3, 0), (2, 1, 1), (2, 2, 1), (2, 4, 1), (4, 1, 3), (4, 4, 3)])
def test_compiles_start_no_more_threads_than_there_are_cpus(host_checks, cpus, callers, most):
    """Callers and helpers together: a compile that is alone for a moment may start one while others have not begun."""
    started, at_once = map(int, host_checks("threads", cpus, callers, text=many_rules(200)).split()[:2])
    if started < 0:
        pytest.skip("not as many CPUs")
    assert at_once <= most
    assert (started > 0) == (most > 0) or callers > 1


# Rules of so many bytes each: the largest decides how long determinising takes, and helpers are for what is left.
@pytest.mark.parametrize("sizes, helpers", [([9000], 0), ([9000] + [100] * 4, 0), ([5000] * 2, 1), ([4500, 4500, 2900], 1), ([3000] * 3, 2), ([2500] * 4, 3), ([1000] * 12, 3)])
def test_compiles_start_as_many_threads_as_there_is_work_for(host_checks, sizes, helpers):
    text = "root ::= " + " | ".join(f"f{k}" for k in range(len(sizes))) + "\n"
    text += "".join(f'f{k} ::= "' + "".join(chr(97 + (5 * j + j // 26 + k) % 26) for j in range(n)) + '"\n' for k, n in enumerate(sizes))
    started, at_once = map(int, host_checks("threads", 4, 1, text=text).split()[:2])
    if started < 0:
        pytest.skip("not as many CPUs")
    assert started == 20 * (helpers + 1)  # (20 compiles; one thread more makes what is not in the tables)
    assert at_once <= max(helpers, 1)


def test_kernels_keep_their_registers():
    """No kernel keeps vector registers in memory; the fills that walk move a few dozen scalar registers to lanes of vector
    registers and back (up to 38 today), not a hundred: their walks wait for every instruction."""
    readelf = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
    if not os.path.exists(readelf):
        pytest.skip("no llvm-readelf")
    data = open(lib_build.LIB, "rb").read()
    bundle = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    at, code = bundle + 32, b""
    for _ in range(struct.unpack_from("<Q", data, bundle + 24)[0]):
        offset, size, length = struct.unpack_from("<QQQ", data, at)
        if data[at + 24 : at + 24 + length].endswith(b"gfx950"):
            code = data[bundle + offset : bundle + offset + size]
        at += 24 + length
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(code)
        f.flush()
        notes = subprocess.run([readelf, "--notes", f.name], capture_output=True, text=True, check=True).stdout
    kernels = re.findall(r"\.name: +(\S+).*?\.sgpr_spill_count: (\d+).*?\.vgpr_spill_count: (\d+)", notes, re.S)
    fills = [int(sgpr) for name, sgpr, _ in kernels if "11fill_kernel" in name]
    assert len(kernels) > 50 and len(fills) > 20
    assert all(int(vgpr) == 0 for _, _, vgpr in kernels)
    assert max(fills) <= 48
