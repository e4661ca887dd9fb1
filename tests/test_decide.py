"""The far-field ray kernel's pixel decision on the CPU, under UndefinedBehaviorSanitizer: positions
far outside the map, infinite and undefined ones are left to the re-check or called out, and never
converted to whole numbers."""
import math
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1005_5198_amd", "csrc")


def _inside(x, m, n):
    """The pixel along one axis, in exact terms: x is farther than m from both its edges."""
    if not math.isfinite(x) or not m >= 0.0:
        return None
    f = math.floor(x)
    return f if 0 <= f < n and x - f > m and (x - f) + m < 1.0 else None


def test_pixel_inside(tmp_path):
    exe = str(tmp_path / "decide_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined,float-cast-overflow",
                    "-fno-sanitize-recover=all", "-I", CSRC, os.path.join(ROOT, "tests", "decide_driver.cpp"), "-o", exe],
                   check=True)
    inf, nan = math.inf, math.nan
    grids = [(1, 1), (3, 5), (1024, 1024), (2 ** 31 - 1, 1), (1, 2 ** 31 - 1), (46340, 46340)]
    cases = []
    for npx, npy in grids:
        xs = [0.5, -0.5, 0.0, -0.0, 1.0, 0.25, npx - 0.5, npx - 1.0, float(npx), npx + 0.5, npx - 2.0 ** -22, -1e-300, 1e-300,
              2.0 ** 31 - 0.5, 2.0 ** 31, -2.0 ** 31, -2.0 ** 31 - 0.5, 2.0 ** 32 + 0.5, 2.0 ** 63, 1e19, 1e300, -1e300, inf, -inf, nan]
        ys = [0.5, npy - 0.5, float(npy), -0.5, 2.0 ** 31 + 0.5, 2.0 ** 32 + 0.5, 1e300, -1e300, inf, nan]
        for x in xs:
            for y in ys:
                for mu, mv in ((0.0, 0.0), (1e-9, 0.3), (0.3, 1e-9), (0.6, 0.6), (inf, 0.0), (0.0, inf), (nan, 0.0), (0.0, nan)):
                    cases.append((x, y, mu, mv, npx, npy))
    text = "".join(" ".join([*(repr(float(v)) for v in c[:4]), str(c[4]), str(c[5])]) + "\n" for c in cases)
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split()
    assert len(out) == len(cases)
    for c, got in zip(cases, out):
        i, j = _inside(c[0], c[2], c[4]), _inside(c[1], c[3], c[5])
        assert int(got) == (-1 if i is None or j is None else j * c[4] + i), c


def test_the_kernel_decides_by_it():
    text = open(os.path.join(CSRC, "farfield.hip")).read()
    body = text[text.index("int patch_decide("):]
    body = body[:body.index("\n}\n")]
    assert "pixel_inside(u, v, Mu, Mv, a.npx, a.npy)" in body and "(int)f" not in body
