"""CPU: the error budget of the mirror sheets bounds what FP32 makes of a reflection point.

The queries' arithmetic in numpy (products and sums rounded one by one, fused
ones once, reciprocals off by up to one unit in the last place): rays from up
to the budget's reach away are traced to facets, and the reflection point, once
more in the facet's frame, is compared with the facet's plane in FP64.
"""

import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2309_12496_amd", "csrc")
U = 2.0 ** -24
F = np.float32


@pytest.fixture(scope="module")
def point_error(tmp_path_factory):
    """point_error of bvh_build.cpp, in units of 2^-24."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("sheet")
    (d / "main.cpp").write_text(
        '#include "bvh_build.cpp"\n#include <cstdio>\n#include <cstdlib>\n'
        "int main(int, char **v) {\n"
        "    rich::SheetBudget b{1.0, atof(v[1]), atof(v[2]), atoi(v[3]) != 0};\n"
        '    std::printf("%.17g\\n", std::ldexp(rich::point_error(b, atof(v[4]), atof(v[5])), 24));\n}\n')
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                    "-I", os.path.join(rocm, "include"), str(d / "main.cpp"), "-o", exe], check=True)
    return lambda reach, far, moving, rho, longest: float(subprocess.run(
        [exe, *map(str, (reach, far, int(moving), rho, longest))], check=True, capture_output=True, text=True).stdout)


def fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(F)


def rotation(rng):
    a = rng.normal(size=(3, 3))
    q, r = np.linalg.qr(a)
    return q * np.sign(np.diag(r))


@pytest.mark.parametrize("moving", [False, True])
@pytest.mark.parametrize("reach, rho, longest", [(6000.0, 2100.0, 5.0), (3000.0, 2100.0, 5.0), (3000.0, 150.0, 1.5),
                                                 (3000.0, 150.0, 60.0), (100.0, 3000.0, 60.0)])
def test_reflection_points(point_error, reach, rho, longest, moving):
    rng = np.random.default_rng(int(reach + rho + longest) + moving)
    worst, n = 0.0, 200_000
    for _ in range(4):
        org = rng.uniform(-1500.0, 1500.0, 3).astype(F)
        rot = rotation(rng) if moving else np.eye(3)
        scale = rng.uniform(0.9, 1.0) if moving else 1.0
        m = (rot.T / scale).astype(F)                          # local = m (world - org)
        back = np.linalg.inv(m.astype(np.float64))             # what FP32 made of the frame, exactly undone

        def local(x):
            if not moving:
                return x
            return np.stack([fma(m[i, 0], x[:, 0], fma(m[i, 1], x[:, 1], (m[i, 2] * x[:, 2]).astype(F)))
                             for i in range(3)], 1)

        def rcp(x):
            r = (1.0 / np.float64(x)).astype(F)
            return np.nextafter(r, r * F(1 + rng.choice([-1.0, 0.0, 1.0])), dtype=F)

        def unit(x):
            return x / np.linalg.norm(x, axis=1, keepdims=True)

        # facets: right triangles at up to rho from the frame's origin, met at cosines of 0.5 to 1
        nrm = unit(rng.normal(size=(n, 3)))
        a = unit(np.cross(nrm, rng.normal(size=(n, 3))))
        b = np.cross(nrm, a)
        leg = longest / np.sqrt(2.0)
        at = unit(rng.normal(size=(n, 3))) * (rho - longest) * rng.uniform(0.3, 1.0, (n, 1))
        V = [(at + leg * (x * a + y * b)).astype(F) for x, y in ((-0.3, -0.3), (0.7, -0.3), (-0.3, 0.7))]
        V64 = [v.astype(np.float64) for v in V]
        nrm = unit(np.cross(V64[1] - V64[0], V64[2] - V64[0]))
        p = (rng.dirichlet((2, 2, 2), n)[:, :, None] * np.stack(V64, 1)).sum(1)
        az, c = rng.uniform(0.0, 2.0 * np.pi, (n, 1)), rng.uniform(0.5, 1.0, (n, 1))
        d_loc = -c * nrm + np.sqrt(1.0 - c * c) * (np.cos(az) * a + np.sin(az) * b)
        d = unit(d_loc @ back.T).astype(F)
        o = (p @ back.T + org - reach * rng.uniform(0.5, 1.0, (n, 1)) * d.astype(np.float64)).astype(F)
        # the query
        ol, dl = local((o - org).astype(F)), local(d)
        kz = np.argmax(np.abs(dl), axis=1)
        kx, ky = (kz + 1) % 3, (kz + 2) % 3
        take = lambda v, k: np.take_along_axis(v, k[:, None], 1)[:, 0]
        sz = rcp(take(dl, kz))
        sx, sy = (take(dl, kx) * sz).astype(F), (take(dl, ky) * sz).astype(F)
        P = [(v - ol).astype(F) for v in V]
        X = [fma(-sx, take(q, kz), take(q, kx)) for q in P]
        Y = [fma(-sy, take(q, kz), take(q, ky)) for q in P]
        Z = [(sz * take(q, kz)).astype(F) for q in P]
        edge = lambda i, j: ((X[i] * Y[j]).astype(F) - (Y[i] * X[j]).astype(F)).astype(F)
        e = [edge(2, 1), edge(0, 2), edge(1, 0)]
        det = ((e[0] + e[1]).astype(F) + e[2]).astype(F)
        t = (fma(e[0], Z[0], fma(e[1], Z[1], (e[2] * Z[2]).astype(F))) * rcp(det)).astype(F)
        inside = (np.minimum.reduce(e) >= 0) | (np.maximum.reduce(e) <= 0)
        assert inside.mean() > 0.9
        hit = np.stack([fma(t, d[:, i], o[:, i]) for i in range(3)], 1)
        again = local((hit - org).astype(F)).astype(np.float64)   # the next query's origin
        off = np.abs(((again - V64[0]) * nrm).sum(1))[inside] * scale
        worst = max(worst, float(off.max()) / U)
    bound = point_error(reach, np.sqrt(3.0) * 3000.0, moving, rho, longest)
    print(f"worst {worst:.0f}, bound {bound:.0f}, 12 S {12 * 3000}")
    # (the bound adds worst cases and what the next query's own tests add; sliver terms apart)
    assert worst <= bound and worst > 0.05 * bound
