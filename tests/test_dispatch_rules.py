"""The rules that choose kernels and launch shapes by sizes (csrc/vnm_rules.h), compiled for the host and compared with
the measurements their comments state."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16135_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule("f(1, 2)") evaluates an expression on the rules and returns it as an integer."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    tmp = tmp_path_factory.mktemp("rules")

    def run(expr):
        src = tmp / "rule.cpp"
        src.write_text('#include "vnm_rules.h"\n#include <cstdio>\nusing namespace vnm;\n'
                       'int main() { std::printf("%%lld", (long long)(%s)); }\n' % expr)
        exe = str(tmp / "rule")
        res = subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        return int(subprocess.run([exe], capture_output=True, text=True, check=True).stdout)
    return run


# small matrices: a pass over the rows no wider than they need, a workgroup per row; tall ones: wide passes, 16 rows
@pytest.mark.parametrize("out,inn,aligned,waves,flight,rows", [
    (1, 64, 1, 4, 1, 1), (33, 64, 1, 4, 4, 1), (200, 304, 1, 4, 4, 1), (384, 11008, 1, 4, 4, 8), (500, 4096, 1, 4, 8, 4), (1000, 1000, 1, 4, 8, 1),
    (1024, 1024, 1, 4, 8, 1), (1025, 1025, 0, 16, 8, 4), (2048, 4096, 1, 8, 8, 8), (4096, 4096, 1, 16, 8, 16),
    (16, 1031, 0, 16, 8, 1), (11008, 64, 1, 16, 8, 8)])
def test_ria_score_shapes(rule, out, inn, aligned, waves, flight, rows):
    assert rule("colsum_shape(%d, %d).waves" % (out, aligned)) == waves
    assert rule("colsum_shape(%d, %d).flight" % (out, aligned)) == flight
    assert rule("score_rows(%d, %d)" % (out, inn)) == rows
