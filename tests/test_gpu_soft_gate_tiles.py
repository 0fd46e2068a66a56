"""The soft gate at the edges of its group padding (16 and 32 columns), head dims and tiles."""
import pytest

from tests import test_gpu_soft_gate as soft
from paper_2604_03260_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 129, 300])
@pytest.mark.parametrize("d,K,dtype", [(64, 16, "bf16"), (80, 1, "f16"), (96, 17, "bf16"), (128, 16, "f16"), (128, 32, "bf16")])
def test_group_padding_and_tiles(n, d, K, dtype):
    wl = soft.case("soft_tiles", n=n, d=d, K=K, dtype=dtype, window=min(40, n))
    inp = workloads.make_inputs(wl, "cuda")
    g = soft.soft_assignment(wl, "cuda")
    out, lse = soft.run_soft(wl, inp, g, 6.0)[:2]
    soft.check_soft(wl, inp, g, 6.0, out, lse)


# the tiled kernel: more work-groups of 32 rows than the kernel for short problems takes
@pytest.mark.parametrize("n,heads", [(64, 640), (129, 208), (300, 104)])
@pytest.mark.parametrize("d,K,dtype", [(64, 16, "bf16"), (80, 1, "f16"), (96, 17, "bf16"), (128, 16, "f16"), (128, 32, "bf16")])
def test_group_padding_and_tiles_of_many_heads(n, heads, d, K, dtype):
    wl = soft.case("soft_tiles", B=heads // 8, Hq=8, Hkv=4, n=n, d=d, K=K, dtype=dtype, window=min(40, n))
    inp = workloads.make_inputs(wl, "cuda")
    g = soft.soft_assignment(wl, "cuda")
    out, lse = soft.run_soft(wl, inp, g, 6.0)[:2]
    soft.check_soft(wl, inp, g, 6.0, out, lse)


# windows inside a unit of 32 keys, over several, nearly everything; a negative slope; groups that end inside a half-wave's eight
@pytest.mark.parametrize("n,w", [(33, 1), (97, 32), (290, 70), (290, 289)])
@pytest.mark.parametrize("d,K,dtype,lam", [(64, 3, "f16", 6.0), (80, 32, "bf16", 2.0), (96, 9, "f16", -4.0), (128, 5, "bf16", 8.0), (128, 20, "f16", 3.0)])
def test_short_soft_gate(n, w, d, K, dtype, lam):
    wl = soft.case("soft_short", B=2, n=n, d=d, K=K, dtype=dtype, window=w)
    inp = workloads.make_inputs(wl, "cuda")
    g = soft.soft_assignment(wl, "cuda")
    out, lse = soft.run_soft(wl, inp, g, lam)[:2]
    soft.check_soft(wl, inp, g, lam, out, lse)
