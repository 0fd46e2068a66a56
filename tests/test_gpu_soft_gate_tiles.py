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
