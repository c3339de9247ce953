"""Step 1 of chunks of up to 128 tokens, which is one launch, and step 2 of chunks whose query rows the scoring workgroups sum:
spans, index vectors, selections and outputs against the oracle around the tile edges (64, 128), for every form of the map."""
import pytest

from oracle import ltri_oracle as O
from tests.test_gpu_parity import _stream_parity
from workloads import Workload

pytestmark = pytest.mark.gpu

SIZES = [128, 2, 63, 64, 65, 127, 128, 3, 129, 100, 1, 128]
FORMS = {
    "logit, means": dict(),
    "logit, means, cap": dict(phi=0.3, max_spans_per_chunk=3),
    "logit, percentile": dict(theta=99.0, theta_quantile=0.97, phi=0.1, max_spans_per_chunk=5, max_spans=2048),
    "logit, index vectors": dict(rep_mode=O.REP_DYNAMIC, lam=1.0, unit_tokens=64, index_block_max=9),
    "softmax, means": dict(seg_map=O.MAP_SOFTMAX, theta=0.0213, phi=0.1, max_spans=2048),
    "softmax, percentile, index vectors": dict(seg_map=O.MAP_SOFTMAX, theta=99.0, theta_quantile=0.9, phi=0.1,
                                               max_spans_per_chunk=4, rep_mode=O.REP_DYNAMIC, lam=3.0, max_spans=2048),
    "softmax, units, index vectors": dict(seg_map=O.MAP_SOFTMAX, theta=99.0, theta_quantile=0.9, max_spans_per_chunk=4,
                                          rep_mode=O.REP_DYNAMIC, lam=2.0, unit_tokens=48, index_block_max=6,
                                          ratio_mode=1, max_spans=2048),
}


@pytest.mark.parametrize("whole_step", [True, False])
@pytest.mark.parametrize("dtype,dim,heads,q_map", [("bf16", 128, 8, False), ("bf16", 128, 4, True), ("f32", 64, 8, True),
                                                   ("f32", 128, 2, False)])
@pytest.mark.parametrize("form", list(FORMS))
def test_short_chunks(gpu_device, form, dtype, dim, heads, q_map, whole_step):
    T = sum(SIZES)
    w = Workload("mini-short", heads, 2, dim, dtype, T, max(SIZES), 4, 150, 6, 200, "uniform", 8, 60)
    _stream_parity(w, 17 + heads, T, gpu_device, chunk_sizes=SIZES, rows=range(0, 128, 9), use_q_seg=q_map, whole_step=whole_step,
                   **FORMS[form])
