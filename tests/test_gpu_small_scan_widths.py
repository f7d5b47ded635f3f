"""Small scans of the shape-agnostic path at the edges of how a wave's share of Eq. 5 is cut: channel groups of 1, 2, 4, 8 and 16
to a wave (by the number of positions), one, two and three taps past a multiple of the taps in flight, head_dim 64 (a build of
its own) and others, the scan in one launch and step by step."""
import pytest

from paper_2406_05317_amd import inputs
from parity_util import compare_scan, gpu_forward, oracle_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    dict(head_dim=64, M=16, B=16, L=80, conv_width=3),          # 32 positions: eight parts of two channel groups
    dict(head_dim=64, M=16, B=16, L=72, conv_width=1),
    dict(head_dim=64, M=24, B=20, L=75, conv_width=5),          # 44: four parts of four, tap 4 alone behind two pairs
    dict(head_dim=64, M=40, B=24, L=90, conv_width=7),          # 64 positions, three slot tiles
    dict(head_dim=64, M=56, B=40, L=170, conv_width=9),         # 96: two parts of eight
    dict(head_dim=64, M=96, B=90, L=290, conv_width=15),        # 186: one part of sixteen, taps brought in in chunks
    dict(head_dim=64, M=16, B=16, L=64, conv_width=3, conv_in=1),
    dict(head_dim=64, M=24, B=20, L=75, conv_width=5, norm=2, filter_abs=True),  # the rectifier in front of the convolution
    dict(head_dim=56, M=16, B=16, L=64, conv_width=3),          # fourteen channel groups: one and two to a part
    dict(head_dim=24, M=33, B=31, L=101, conv_width=5),
    dict(head_dim=128, M=16, B=16, L=64, conv_width=3),
], ids=str)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_against_the_oracle(case, dtype):
    w = inputs.Workload(**{**dict(name="widths", dtype=dtype, batch=1, n_q_heads=2, n_kv_heads=1, seed=21), **case})
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    compare_scan(w, gpu_forward(w, q, k, v, cw, cb, impl=1, history=True), oracle_forward(w, q, k, v, cw, cb), what=str(case))
