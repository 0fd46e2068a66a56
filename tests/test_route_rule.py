"""The rule that gives the Sinkhorn rounds of a routing call their work-groups, compiled from its source for the host: work-groups that wait
for each other are at most a quarter of those that the device holds, whatever its size, and their rows fit their registers."""
import os
import subprocess


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2604_03260_amd", "csrc", "focus_route.hip")

PROGRAM = """
#include <algorithm>
#include <cstdio>
#include <initializer_list>
struct RouteLayout { int B, n, K, nsink; };
%s
int main()
{
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


def test_work_groups_of_the_rounds_fit_a_quarter_of_the_device(tmp_path):
    text = open(SOURCE).read()
    begin, end = text.index("constexpr int sink_kp("), text.index("// Column sums on their way")
    (tmp_path / "rule.cpp").write_text(PROGRAM % text[begin:end])
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "rule"), str(tmp_path / "rule.cpp")])
    r = subprocess.run([str(tmp_path / "rule")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    exchanged, launches = map(int, r.stdout.split())
    assert exchanged > 1000 and launches > 1000
