"""The soft gate at the edges of its group padding (16 and 32 columns), head dims and tiles."""
import pytest
import torch

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


# ... and the cases of the small problems there: no slope, negative slope, windows of one position and of everything, one position, one-hot
@pytest.mark.parametrize("lam,one_hot,kw", [
    (0.0, False, dict(d=128, n=520, B=8)), (-7.0, False, dict(d=64, n=640, K=8, B=5)), (9.0, False, dict(d=128, n=300, window=300, B=12)),
    (4.0, False, dict(d=64, n=513, window=1, K=2, B=9)), (5.0, False, dict(d=64, n=1, B=130, window=1)), (60.0, True, dict(d=128, n=1000, K=8, window=40, B=4)),
    (12.0, False, dict(d=80, n=700, K=32, window=16, B=3)), (20.0, False, dict(d=96, n=512, K=8, window=64, dtype="f16", B=7))])
def test_gates_in_tiles(lam, one_hot, kw):
    wl = soft.case("soft_tiles", Hq=8, Hkv=2, **kw)
    assert wl.B * wl.Hq * -(-wl.n // 32) > (512 if wl.K > 16 else 1024 if wl.K <= 4 and wl.d < 128 else 768)     # else the kernel for short problems
    inp = workloads.make_inputs(wl, "cuda")
    g = soft.soft_assignment(wl, "cuda")
    if one_hot:
        g = torch.nn.functional.one_hot(g.argmax(-1), wl.K).float().contiguous()
    out, lse = soft.run_soft(wl, inp, g, lam)[:2]
    soft.check_soft(wl, inp, g, lam, out, lse)
