"""Chunks of more than 16 tiles a side, whose tiles are given up where a bound on their scores is negative: spans, selections and
outputs against the oracle just past that size, at the largest chunk and with a last tile of one row, where nearly every tile is
given up (short spans), where few are (a low threshold) and where none is (a negative one)."""
import math

import pytest

from oracle import ltri_oracle as O
from tests.test_gpu_parity import _stream_parity
from workloads import Workload

pytestmark = pytest.mark.gpu

SIZES = [1025, 2048, 1089]
FORMS = {
    "short spans": (16, 64, dict()),
    "long spans, low threshold": (64, 900, dict(theta=0.12 * math.sqrt(128))),
    "negative threshold": (16, 64, dict(theta=-0.25)),
    "percentile": (16, 200, dict(theta=99.0, theta_quantile=0.97)),
    "softmax": (16, 200, dict(seg_map=O.MAP_SOFTMAX, theta=0.0213)),
}


@pytest.mark.parametrize("dtype,heads,q_map", [("bf16", 4, False), ("bf16", 4, True), ("f32", 2, False)])
@pytest.mark.parametrize("form", list(FORMS))
def test_given_up_tiles(gpu_device, form, dtype, heads, q_map):
    lo, hi, kw = FORMS[form]
    T = sum(SIZES)
    w = Workload("mini-bound", heads, 2, 128, dtype, T, max(SIZES), 4, 150, 6, 200, "uniform", lo, hi)
    _stream_parity(w, 31 + heads, T, gpu_device, chunk_sizes=SIZES, rows=range(0, 1025, 199), use_q_seg=q_map,
                   **{**dict(phi=0.1, max_spans_per_chunk=24, max_spans=2048), **kw})
