"""The rules that choose among paths with the same results (csrc/routes.hpp), compiled for the host, as a pytest fixture."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include "routes.hpp"
int main(int argc, char **argv)
{
    long long v[8];
    char what[32];
    while (std::scanf("%31s", what) == 1) {
        if (!std::strcmp(what, "order")) {
            for (int i = 0; i < 5; ++i) if (std::scanf("%lld", v + i) != 1) return 1;
            const hgca::GatherOrder o = hgca::gather_order(v[0], v[1], v[2], v[3] != 0, v[4] != 0);
            std::printf("%d\n", o.keep ? 2 : o.by_group ? 1 : 0);
        } else if (!std::strcmp(what, "first")) {
            for (int i = 0; i < 5; ++i) if (std::scanf("%lld", v + i) != 1) return 1;
            std::printf("%d\n", hgca::window_first(v[0] != 0, v[1], v[2], v[3], v[4] != 0) ? 1 : 0);
        } else if (!std::strcmp(what, "short")) {
            for (int i = 0; i < 7; ++i) if (std::scanf("%lld", v + i) != 1) return 1;
            std::printf("%d\n", hgca::short_step(v[0] != 0, v[1], v[2], v[3], v[4], v[5], v[6]) ? 1 : 0);
        }
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    src, exe = d / "routes.cpp", d / "routes"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2507_03153_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)

    def ask(*lines):
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return ask
