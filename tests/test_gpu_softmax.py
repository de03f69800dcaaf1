"""GPU parity of the softmax at the edges of its rows-in-registers variants against the oracle."""
import pytest

from paper_1704_04560_amd import workloads as wl
from tests.test_gpu_train_step import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("classes", [1, 63, 65, 256, 257, 1024, 1025])
def test_softmax_widths_match_oracle(classes, dtype):
    net = wl.Net(f"softmax-{classes}", (1, 1, 24), (wl.fc(classes),), dtype, "normal")
    run_case(net.name, net, 2, 5, 2, 3, 0.05, 0.9)
