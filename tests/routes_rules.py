"""The rules that choose among paths with the same results (csrc/routes.hpp), compiled for the host, as a pytest fixture."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
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
        } else if (!std::strcmp(what, "queries")) {      // shares as an fp32 append call over one tier makes them
            for (int i = 0; i < 7; ++i) if (std::scanf("%lld", v + i) != 1) return 1;
            const long long pairs = v[1] * v[2], units = pairs * ((v[4] * v[3] + 127) / 128), steps = (v[5] + 63) / 64;
            const int most = (int)std::max(std::max(1LL, 512 / units), (v[5] + 511) / 512);
            const int64_t turns = hgca::line_turns(units, steps, hgca::line_shares(units, steps, most, 256, 1), 256);
            std::printf("%d\n", hgca::query_by_query(v[0], v[1], v[2], v[3], v[4], v[5], v[6], turns) ? 1 : 0);
        }
    }
}
"""


def runs_query_by_query(rules, B, N, Hq, Hkv, d, cap):
    """Whether an fp32 append call over one tier runs query by query; its splits as the call cuts them."""
    blocks, up64 = max(1, B * Hkv * -(-N * Hq // Hkv // 128)), lambda x: (x + 63) // 64 * 64
    most = max(max(1, 512 // blocks), -(-cap // 512))
    chunk = max(min(512, max(64, up64(-(-cap // max(1, 1024 // (B * N * Hkv)))))), up64(-(-cap // most)))
    return rules("queries %d %d %d %d %d %d %d" % (d, B, Hkv, Hq // Hkv, N, cap, -(-cap // chunk))) == [1]


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
