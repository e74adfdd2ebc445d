"""The rule that says which one-read passes a workgroup's LDS holds, on the
host: at the last beamlet count that it takes and the next one, with what the
compiled kernels hold beside the launch's own bytes (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_0908_4421_amd")
MAX_LDS = 160 << 10   # of a gfx950 workgroup

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "quad_layout.h"
using namespace imrt;
int main() {
  for (int nt : {1, 2, 4})
    for (int ns : {1, 4, 16, 256})
      for (int mode : {QM_SOLVE, QM_GRAD, QM_POWER, QM_EVAL, QM_PLAIN}) {
        int nb = 1;
        while (nb < 20000 && quad_fits(MAX_LDS, quad_lds_bytes(nb + 1, nt, ns, mode))) ++nb;
        std::printf("%d %d %d %d %zu %zu\n", nt, ns, mode, nb, quad_lds_bytes(nb, nt, ns, mode),
                    quad_lds_bytes(nb + 1, nt, ns, mode));
      }
  std::printf("fixed %zu whole %zu %zu\n", kQuadFixedLds, kWholeFixedLds, quad_lds_bytes(1024, 1, 256, QM_WHOLE));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("layout")
    (d / "layout.cpp").write_text(PROGRAM.replace("MAX_LDS", str(MAX_LDS)))
    subprocess.run([cxx, "-std=c++17", "-I", os.path.join(PKG, "csrc"), str(d / "layout.cpp"), "-o", str(d / "layout")],
                   check=True)
    out = subprocess.run([str(d / "layout")], check=True, stdout=subprocess.PIPE, text=True).stdout
    rows = [tuple(map(int, ln.split())) for ln in out.splitlines() if ln[0].isdigit()]
    fixed, whole, whole_bytes = map(int, re.search(r"fixed (\d+) whole (\d+) (\d+)", out).groups())
    return rows, fixed, whole, whole_bytes


def test_both_sides_of_the_edge(rule):
    rows, fixed, whole, whole_bytes = rule
    assert len(rows) == 3 * 4 * 5
    for nt, ns, mode, nb, last, beyond in rows:
        assert last + fixed <= MAX_LDS, (nt, ns, mode, nb)
        assert nb == 20000 or beyond + fixed > MAX_LDS, (nt, ns, mode, nb)
        # a vector's bytes and its column sums', at least
        assert last >= nt * nb * (12 if mode in (0, 2, 4) else 4) + (nb if mode in (0, 2, 4) else 0) + 32 * ns
    assert whole_bytes + whole <= 64 << 10


def test_the_compiled_kernels_hold_no_more(rule, tmp_path):
    """Group segment of every kernel of the built one-read pass, as the
    compiler states it."""
    _, fixed, whole, _ = rule
    obj = os.path.join(PKG, "_build", "onepass.o")
    objdump, readelf = ("/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readelf")
    if not all(os.path.exists(p) for p in (obj, objdump, readelf)):
        pytest.skip("one-read pass not built here")
    shutil.copy(obj, tmp_path / "onepass.o")
    subprocess.run([objdump, "--offloading", "onepass.o"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert len(code) == 1
    notes = subprocess.run([readelf, "--notes", str(tmp_path / code[0])], check=True, stdout=subprocess.PIPE,
                           text=True).stdout
    sizes = re.findall(r"\.group_segment_fixed_size: (\d+).*?\.name: +(\w+)", notes, re.S)
    quads = {name: int(n) for n, name in sizes if re.search("quad_(kernel|batch|shared)", name)}
    wholes = {name: int(n) for n, name in sizes if "whole_kernel" in name}
    assert len(quads) > 50 and len(wholes) == 3
    assert max(quads.values()) <= fixed and max(wholes.values()) <= whole
