"""Running sums of a chunk's query and key rows (bf16, 128-wide heads, chunks of more than 128 tokens): stored mean keys
and selections against the oracle at chunk lengths around their blocks of 128 tokens and 8 tokens per wavefront, and for
group sizes around the four rows that are read at a time."""
import pytest

from tests.test_gpu_parity import _stream_parity
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("whole_step", [True, False])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
def test_running_sums_at_block_edges(gpu_device, group, whole_step):
    sizes = [129, 255, 256, 257, 136, 137, 391]
    w = Workload("mini-sums", 2 * group, 2, 128, "bf16", sum(sizes), 512, 4, 96, 0, 200, "uniform", 16, 96)
    _stream_parity(w, 20 + group, sum(sizes), gpu_device, chunk_sizes=sizes, whole_step=whole_step)
