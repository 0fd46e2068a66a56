"""The rule that gives the Sinkhorn rounds of a routing call their work-groups, compiled from its source for the host: work-groups that wait
for each other are at most a quarter of those that the device holds, whatever its size, and their rows fit their registers."""
import os
import subprocess

import pytest

from tests import test_gpu_router

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2604_03260_amd", "csrc", "focus_route.hip")

PROGRAM = """
#include <algorithm>
#include <cstdio>
#include <initializer_list>
struct RouteLayout { int B, n, K, nsink; };
%s
int main(int argc, char**)
{
    if (argc > 1) {                               // of each shape read in: work-groups, padded groups, rows per thread
        int B, K, n;
        while (scanf("%%d %%d %%d", &B, &n, &K) == 3) {
            const int g = sink_groups(RouteLayout{B, n, K, std::min(256, (n + 255) / 256)}, 256);
            printf("%%d %%d %%d\\n", g, sink_kp(K), g ? sink_rows(sink_kp(K), (n + g - 1) / g) : 0);
        }
        return 0;
    }
    long long exchanged = 0, launches = 0;
    for (int units : {8, 20, 32, 64, 128, 256, 304})
        for (int B : {1, 2, 3, 5, 8, 16, 31, 64, 70, 129, 1000})
            for (int K = 1; K <= 32; ++K)
                for (int n = 1; n < (1 << 20); n += 1 + n / 37) {
                    RouteLayout R{B, n, K, std::min(256, (n + 255) / 256)};
                    const int g = sink_groups(R, units), kp = sink_kp(K);
                    if (g == 0) { ++launches; continue; }
                    const int tokens = (n + g - 1) / g, rows = sink_rows(kp, tokens);
                    bool bad = rows <= 0 || rows * kp > 64 || rows * 256 < tokens || kp < K || g > 64;
                    // the kernel's three slots of K sums for each work-group lie in 48 of the 64 * nsink words of partial sums
                    bad = bad || (g > 1 && ((long long)g * B * 4 > (long long)units * sink_resident(kp, rows) || 3LL * g * K > 48LL * R.nsink));
                    if (bad) { printf("units %%d B %%d K %%d n %%d: %%d work-groups of %%d rows\\n", units, B, K, n, g, rows); return 1; }
                    exchanged += g > 1;
                }
    printf("%%lld %%lld\\n", exchanged, launches);
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    text = open(SOURCE).read()
    begin, end = text.index("constexpr int sink_kp("), text.index("// Column sums on their way")
    (tmp / "rule.cpp").write_text(PROGRAM % text[begin:end])
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", str(tmp / "rule"), str(tmp / "rule.cpp")])
    return str(tmp / "rule")


def test_work_groups_of_the_rounds_fit_a_quarter_of_the_device(rule):
    r = subprocess.run([rule], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    exchanged, launches = map(int, r.stdout.split())
    assert exchanged > 1000 and launches > 1000


def test_shapes_of_the_gpu_tests_reach_every_kernel(rule):
    def of(shapes):
        r = subprocess.run([rule, "shapes"], input="".join("%d %d %d\n" % s[:3] for s in shapes), capture_output=True, text=True, check=True)
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]

    one, each = of(test_gpu_router.ROUNDS_IN_ONE_LAUNCH), of(test_gpu_router.A_LAUNCH_PER_ROUND)
    assert all(g > 0 for g, _, _ in one) and all(g == 0 for g, _, _ in each)
    kernels = {(4, 2), (4, 4), (4, 8), (4, 16), (8, 2), (8, 4), (8, 8), (16, 2), (16, 4), (32, 2)}
    assert {(kp, rows) for _, kp, rows in one} == kernels
    assert {kp for g, kp, _ in one if g == 1} == {kp for g, kp, _ in one if g > 1} == {4, 8, 16, 32}
    # a launch per round: all groups of the padding there, and some of them missing
    assert {(kp, K == kp) for (_, kp, _), (_, _, K, _, _) in zip(each, test_gpu_router.A_LAUNCH_PER_ROUND)} == {(kp, whole) for kp in (4, 8, 16, 32) for whole in (True, False)}
