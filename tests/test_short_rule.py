"""Which problems the kernels for rows in position order take, from their sources for the host.  The bucketing skips for the 16-bit one
what the tiled kernel needs (key copy, key norms, membership words), so whatever the bucketing does not read must not decide: the
softcap."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_03260_amd", "csrc")

PROGRAM = """
#include <cstdint>
#include <cstdio>
#include <initializer_list>
struct Layout { int B, Hq, n, d, dtype, NC, masked, dense, soft, local_only, merge_prev, BQ, causal; long long ks[3]; float softcap; int K; };
%s
int main(int argc, char** argv)
{
    int d, n, groups, causal, dense;                  // dense of the soft gate: its groups
    while (argc > 1 && scanf("%%d %%d %%d %%d %%d", &d, &n, &groups, &causal, &dense) == 5) {
        const int per = (n + 31) / 32;
        Layout L{groups / per, 1, n, d, 1, 1, !dense, dense, 0, 0, 0, 128, causal, {1LL * n * d, 1LL * n * d, d}, 0.f, dense};
        const char rule = argv[1][0];
        L.soft = rule == 's';
        printf("%%d\\n", (int)(rule == 'h' ? short_attention(L) : rule == 's' ? short_soft_attention(L) : by_tiles(L)));
    }
    if (argc > 1) return 0;
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


# d, tokens, work-groups of 32 rows, causal, dense; microseconds of bucketing and attention: tiled, short, tiled with a cap of 50, short with it
MEASURED = [
    (64, 512, 1024, 1, 0, 33.1, 31.8, 35.8, 36.2), (64, 4096, 768, 1, 0, 79.5, 71.6, 101, 93.2), (80, 4096, 768, 1, 0, 87.6, 86.7, 110, 109),
    (96, 4096, 768, 1, 0, 90.9, 83.5, 111, 104), (128, 256, 1024, 1, 0, 37.4, 32.3, 38.8, 35.4), (128, 1024, 768, 1, 0, 51.3, 51.2, 56.4, 52.4),
    (128, 4096, 640, 1, 0, 104, 102, 126, 104), (256, 256, 1024, 1, 0, 57.3, 55.2, 58.5, 60.4), (256, 1024, 640, 1, 0, 75.2, 78.5, 79.3, 89.2),
    (256, 4096, 640, 1, 0, 168, 188, 185, 225), (256, 4096, 512, 1, 0, 168, 147, 183, 176),
    (64, 256, 768, 0, 0, 26.6, 22.9, 27.8, 25.5), (64, 256, 896, 0, 0, 27.3, 27.8, 28.7, 31.1), (64, 512, 640, 0, 0, 30.2, 30.3, 32.9, 35.0),
    (96, 512, 752, 0, 0, 39.2, 41.5, 42.2, 45.0), (64, 1024, 512, 0, 0, 35.7, 34.7, 40.8, 40.0), (64, 4096, 512, 0, 0, 75.6, 79.6, 97.3, 105),
    (96, 4096, 384, 0, 0, 90.8, 96.4, 110, 120), (64, 2048, 512, 0, 0, 48.9, 49.4, 59.6, 61.5), (64, 4096, 256, 0, 0, 74.6, 46.8, 96.5, 60.2),
    (64, 4096, 512, 0, 1, 83.3, 69.1, 102, 94.8), (80, 4096, 512, 0, 1, 98.5, 86.8, 116, 111), (128, 4096, 256, 0, 1, 114, 77.8, 133, 80.7),
    (256, 256, 640, 0, 0, 52.4, 51.0, 53.6, 55.2), (256, 512, 512, 0, 0, 59.6, 59.5, 61.3, 66.0), (256, 4096, 256, 0, 0, 169, 146, 185, 171),
]


# d, tokens, work-groups of 32 rows, 1, groups; microseconds of the soft gate: tiled, short
MEASURED_SOFT = [
    (64, 512, 752, 1, 4, 27.7, 21.1), (64, 300, 1000, 1, 4, 22.3, 23.1), (64, 40, 1000, 1, 4, 16.4, 17.3), (96, 40, 1000, 1, 4, 17.3, 18.9),
    (96, 1024, 1024, 1, 4, 44.9, 36.4), (64, 300, 760, 1, 16, 22.5, 24.5), (64, 512, 752, 1, 16, 27.4, 29.3), (128, 300, 760, 1, 8, 25.4, 27.1),
    (128, 300, 760, 1, 16, 25.5, 30.8), (128, 512, 752, 1, 16, 32.1, 37.9), (128, 1000, 736, 1, 16, 46.0, 51.6), (128, 2048, 704, 1, 16, 74.2, 77.0),
    (128, 300, 500, 1, 32, 28.5, 29.8),
]
# d, tokens, work-groups of 32 rows, causal, dense; microseconds in 32 bits: attn_f32_linear_kernel, attn_f32_kernel
MEASURED_F32 = [
    (256, 256, 400, 1, 0, 70.1, 78.5), (256, 512, 800, 0, 1, 259, 248), (256, 512, 800, 1, 0, 153, 168), (256, 700, 198, 1, 1, 114, 109),
    (256, 700, 396, 0, 0, 187, 183), (256, 700, 88, 0, 0, 92.5, 97.4), (256, 1024, 384, 1, 0, 126, 122), (256, 1024, 384, 0, 1, 239, 220),
    (256, 1024, 800, 1, 0, 241, 246), (256, 2048, 768, 1, 0, 375, 350), (256, 2048, 768, 0, 1, 634, 556), (96, 2048, 768, 1, 0, 150, 138),
    (96, 2048, 1600, 1, 0, 1.0, 1.07), (96, 2048, 768, 0, 0, 1.0, 1.26), (96, 1024, 640, 0, 1, 134, 130), (64, 1024, 768, 0, 1, 111, 99.2),
    (64, 2048, 768, 0, 1, 186, 162), (64, 2048, 640, 0, 1, 155, 161), (64, 2048, 768, 0, 0, 189, 210), (64, 700, 748, 0, 1, 91.8, 97.9),
]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    text = open(os.path.join(CSRC, "focus_attn_short.hip")).read()
    source = text[text.index("bool short_attention("):text.index("hipError_t launch_attn_short(")]
    source += text[text.index("bool short_soft_attention("):text.index("hipError_t launch_attn_short_soft(")]
    text = open(os.path.join(CSRC, "focus_attn_f32.hip")).read()
    source += text[text.index("bool by_tiles("):text.index("hipError_t launch_attn_f32(")]
    (tmp / "rule.cpp").write_text(PROGRAM % source)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", str(tmp / "rule"), str(tmp / "rule.cpp")])
    return str(tmp / "rule")


def chosen(rule, which, table):
    r = subprocess.run([rule, which], input="".join("%d %d %d %d %d\n" % m[:5] for m in table), capture_output=True, text=True, check=True)
    return list(zip(map(int, r.stdout.split()), table))


def test_the_softcap_does_not_decide(rule):
    r = subprocess.run([rule], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    taken, left = map(int, r.stdout.split())
    assert taken > 1000 and left > 1000


def test_the_faster_kernel_is_taken(rule):
    """... or one within 5 %, with and without a softcap; the soft gate and 32 bits: within 2.5 %."""
    for short, m in chosen(rule, "hard", MEASURED):
        assert m[5 + short] <= 1.05 * min(m[5:7]) and m[7 + short] <= 1.05 * min(m[7:9]), m
    for short, m in chosen(rule, "soft", MEASURED_SOFT):
        assert m[5 + short] <= (1.025 * min(m[5:7]) if m[6] > m[5] else m[5]), m
    for tiles, m in chosen(rule, "f32", MEASURED_F32):
        assert m[5 + tiles] <= 1.025 * min(m[5:7]), m
