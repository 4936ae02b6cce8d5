"""The pair-screen network's kernels at the sample counts where the size of their tiles changes
(16, 32 and 64 samples) and around the smaller tiles' edges, with the bounds of the tests at the
64-sample tiles' edges."""
import pytest

from test_gpu_screen_net import test_forward_and_backward as forward_and_backward
from test_gpu_screen_net import test_training_step_is_forward_backward_adam as training_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 31, 33, 4096, 4097, 8192, 8193])
def test_tiles(n):
    forward_and_backward(n)
    training_step(n)
