"""Which problems the kernel for short 16-bit problems takes, from its source for the host.  The bucketing skips for it what the tiled
kernel needs (key copy, key norms, membership words), so whatever the bucketing does not read must not decide: the softcap."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2604_03260_amd", "csrc", "focus_attn_short.hip")

PROGRAM = """
#include <cstdint>
#include <cstdio>
#include <initializer_list>
struct Layout { int B, Hq, n, d, dtype, NC, masked, dense, soft, local_only, merge_prev, BQ, causal; long long ks[3]; float softcap; };
%s
int main()
{
    long long taken = 0, left = 0;
    for (int d : {64, 80, 96, 128, 256})
        for (int causal : {0, 1})
            for (int dense : {0, 1})
                for (int heads = 1; heads < 1200; heads += 1 + heads / 40)
                    for (int n = 1; n < 6000; n += 1 + n / 30) {
                        Layout L{1, heads, n, d, 1, 1, !dense, dense, 0, 0, 0, 128, causal, {1LL * heads * n * d, 1LL * n * d, d}, 0.f};
                        const bool without = short_attention(L);
                        L.softcap = 50.f;
                        if (short_attention(L) != without) { printf("d %%d causal %%d dense %%d heads %%d n %%d\\n", d, causal, dense, heads, n); return 1; }
                        ++(without ? taken : left);
                    }
    printf("%%lld %%lld\\n", taken, left);
    return 0;
}
"""


def test_the_softcap_does_not_decide(tmp_path):
    text = open(SOURCE).read()
    begin, end = text.index("bool short_attention("), text.index("hipError_t launch_attn_short(")
    (tmp_path / "rule.cpp").write_text(PROGRAM % text[begin:end])
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "rule"), str(tmp_path / "rule.cpp")])
    r = subprocess.run([str(tmp_path / "rule")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    taken, left = map(int, r.stdout.split())
    assert taken > 1000 and left > 1000
