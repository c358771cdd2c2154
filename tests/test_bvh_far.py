"""CPU: the tree builder ends on meshes whose boxes' areas overflow FP64."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2309_12496_amd", "csrc")

MAIN = r"""
#include "bvh_build.cpp"
#include <cstdio>
using namespace rich;
int main() {
    // two flat mirrors, which are sheets at this t_min, and two far patches of an absorber
    std::vector<BuildTri> tris;
    auto patch = [&](double x, double y, int group, bool mirror) {
        for (int i = 0; i < 40; ++i) {
            BuildTri t{};
            const double a = i % 8, b = i / 8;
            const double v[3][3] = {{x + a, y + b, 0}, {x + a + 1, y + b, 0}, {x + a, y + b + 1, 0}};
            for (int m = 0; m < 3; ++m)
                for (int q = 0; q < 3; ++q) t.v[m][q] = v[m][q];
            t.n[2] = 1.0;
            t.index = (uint32_t)tris.size();
            t.group = group;
            t.mirror = mirror;
            tris.push_back(t);
        }
    };
    patch(0.0, 0.0, 0, true);
    patch(1000.0, 0.0, 1, true);
    patch(1e200, 1e200, 2, false);
    patch(-1e200, -1e200, 3, false);
    std::vector<Node4> nodes;
    std::vector<Tri> out;
    std::vector<Sheet> sheets;
    BuildBox box;
    int depth = 0;
    const uint32_t root = build_mesh_bvh4(tris, nodes, out, &depth, &box, SheetBudget{1e300, 1e200, 1e200, false}, sheets);
    std::printf("%d %zu %zu\n", root != kEmpty, out.size(), sheets.size());
}
"""


def test_overflowing_areas(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                    os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), str(tmp_path / "main.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.split() == ["1", "160", "2"], (r.returncode, r.stdout)
