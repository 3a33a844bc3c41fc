"""The arithmetic by which launches of many workgroups are cut, compiled by itself for the
CPU: a HIP launch stays below 2^32 threads, its documented limit, and what one launch cannot
hold is still done."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_23115_amd", "csrc")
THREADS, WAVES = 256, 4
MOST = 2**24 - 1  # workgroups of 256 threads


def compiled(tmp_path, body):
    cxx = shutil.which("g++")
    assert cxx, "g++ not found"
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "launch_shape.h"\n'
                   "using namespace gleam;\nint main(int argc, char** argv) {\n"
                   "auto arg = [&](int i) { return strtoull(argv[i], nullptr, 10); };\n" + body + "}\n")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True, text=True).stdout
        return [int(x) for x in out.split()]

    return run


@pytest.fixture(scope="module")
def copy_shape(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("copy"),
                    "(void)argc; const CopyShape c = copy_shape(arg(1), (uint32_t)arg(2), arg(3) != 0);\n"
                    'printf("%d %u %u\\n", c.large ? 1 : 0, c.per_log2, c.groups);\n')


@pytest.mark.parametrize("block", [4096 << k for k in range(13)])
@pytest.mark.parametrize("sparse", [0, 1])
def test_copy_shape(copy_shape, block, sparse):
    large = sparse and block >= 65536
    per = block // (16384 if large else 4096)
    at_limit = MOST * WAVES // per  # blocks that fill the largest launch, and those around them
    for n in {1, 2, 5, 1000, 65_535, 65_536, 8_388_608, at_limit - 1, at_limit, at_limit + 1, 2 * at_limit + 7, 2**40}:
        got_large, per_log2, groups = copy_shape(n, block, sparse)
        assert got_large == (1 if large else 0) and 1 << per_log2 == per, (n, block)
        assert groups == min(-(-n * per // WAVES), MOST), (n, block)
        assert 0 < groups * THREADS < 2**32


def test_launch_in_parts(tmp_path):
    """Parts in order, none larger than the limit, that make up every workgroup once; a failed
    one is the last."""
    run = compiled(tmp_path,
                   "const uint64_t fail = argc > 3 ? arg(3) : ~0ull;\n"
                   "const int32_t st = launch_in_parts(arg(1), arg(2), [&](uint64_t first, uint32_t count) -> int32_t {\n"
                   '  printf("%llu %u\\n", (unsigned long long)first, count);\n'
                   "  return first >= fail ? -4 : 0;\n});\n"
                   'printf("%d\\n", st);\n')
    for groups in (0, 1, MOST - 1, MOST, MOST + 1, 2 * MOST, 2**24, 2**31 - 1):
        *parts, status = run(groups, MOST)
        at = 0
        for first, count in zip(parts[::2], parts[1::2]):
            assert first == at and 0 < count <= MOST
            at += count
        assert at == groups and status == 0 and len(parts) // 2 == -(-groups // MOST)
    assert run(50, 20, 20) == [0, 20, 20, 20, -4]
