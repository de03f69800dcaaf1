"""GPU parity of strided projections, whose data gradient is kept at the positions they read,
against the oracle."""
import pytest

from paper_1704_04560_amd import workloads as wl
from tests.test_gpu_train_step import run_case

pytestmark = pytest.mark.gpu

# source channels, height and width, projection channels, stride: odd sizes whose last rows and
# columns are read or are not, a stride past the kernel, channels off the vectors (full-size share)
PROJECTIONS = [(16, 13, 10, 24, 2), (8, 9, 16, 32, 3), (12, 8, 8, 16, 2), (20, 7, 11, 40, 2)]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("c,h,w,out,stride", PROJECTIONS)
def test_strided_projections_match_oracle(c, h, w, out, stride, dtype):
    net = wl.Net(f"projection-{c}-{out}-{stride}", (3, h, w),
                 (wl.conv(4, 3, pad=1), wl.conv(c, 3, pad=1, relu=True),
                  wl.conv(8, 1, relu=True), wl.conv(out, 3, stride=stride, pad=1),
                  wl.addp(1, out, stride=stride, relu=True), wl.fc(5)), dtype, "normal")
    run_case(net.name, net, 2, 6, 2, 3, 0.02, 0.9)
