"""The host rule that sends calls whose velocity and right-hand side share memory to the
copying paths (extents.hpp), compiled for the CPU, against the sets of elements that the
used extents hold: every offset of one array against the other that can make them meet, in
strides without and with room for rows laid out side by side.
"""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_19061_amd", "csrc")

MAIN = """
#include <cstdio>
#include "extents.hpp"
int main() {
    int nx, ny;
    long ld, es, v[4];
    char* base = (char*)(1l << 40);
    while (std::scanf("%d %d %ld %ld %ld %ld %ld %ld", &nx, &ny, &ld, &es, v, v + 1, v + 2, v + 3) == 8)
        std::putchar('0' + stk::velocity_shares(nx, ny, ld, es, base + v[0] * es, base + v[1] * es, base + v[2] * es,
                                                base + v[3] * es));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("extents")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "extents")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", exe], check=True)
    return lambda lines: subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True,
                                        check=True).stdout


@pytest.mark.parametrize("nx,ny", [(2, 2), (3, 2), (4, 5)])
@pytest.mark.parametrize("es", [4, 8])
def test_shared_memory_is_the_meeting_of_the_used_extents(rule, nx, ny, es):
    def x(at, ld):
        return {at + j * ld + i for j in range(ny) for i in range(nx + 1)}

    def y(at, ld):
        return {at + j * ld + i for j in range(ny + 1) for i in range(nx)}

    lines, want = [], []
    for ld in (nx + 1, nx + 2, 2 * nx + 1, 2 * nx + 2, 2 * nx + 5, 4 * nx + 4):
        far = (ny + 3) * ld
        vx, vy, away = 4 * far, 8 * far, 40 * far
        for d in range(-far, far + 1):
            # one array of the right-hand side moved over one of the velocity, the other apart
            for bx, by in ((vx + d, away), (vy + d, away), (away, vx + d), (away, vy + d)):
                v, b = x(vx, ld) | y(vy, ld), x(bx, ld) | y(by, ld)
                lines.append(f"{nx} {ny} {ld} {es} {vx} {vy} {bx} {by}")
                want.append("1" if v & b else "0")
    assert rule(lines) == "".join(want)
    assert "0" in want and "1" in want
