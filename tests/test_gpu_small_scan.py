"""The small-scan kernels of the shape-agnostic path (one workgroup per chain for a whole scan, or one per 16 slots
and step; attention of all blocks in one launch): against the oracle, and bit for bit between the schedules."""
import pytest
import torch

from paper_2406_05317_amd import inputs
from parity_util import compare_scan, gpu_forward, oracle_forward

pytestmark = pytest.mark.gpu

CASES = [
    dict(M=16, B=16, L=256, conv_width=3),                                             # one tile: the whole scan in one launch
    dict(M=1, B=1, L=7, conv_width=1, head_dim=4),                                     # the smallest
    dict(M=17, B=5, L=61, conv_width=5, n_q_heads=4, n_kv_heads=2, head_dim=24),       # a slot past the tile, ragged last block
    dict(M=33, B=31, L=200, conv_width=3, head_dim=60, norm=1, bias_sigma=0.5),        # three tiles in one workgroup, d % 16 != 0
    dict(M=24, B=40, L=170, conv_width=7, head_dim=32, norm=2, filter_abs=True, bias_sigma=0.2),   # block longer than the cache
    dict(M=20, B=16, L=100, conv_width=5, head_dim=16, conv_in=1, batch=2),            # [K | V] filters
    dict(M=96, B=96, L=400, conv_width=15, n_q_heads=2, n_kv_heads=2),                 # a launch per step, six tiles
    dict(M=64, B=40, L=280, conv_width=21, head_dim=128),                              # filters brought in a few taps at a time
    dict(M=40, B=24, L=200, conv_width=5, n_q_heads=2, n_kv_heads=2, per_head_filters=True, bias_sigma=0.4, protect_share=0.2),
    dict(M=16, B=12, L=140, conv_width=5, dtype="bf16", protect_share=0.3, norm=1, bias_sigma=0.5, stop=36),
    dict(M=116, B=116, L=500, conv_width=9),                                           # as many positions as fit, one tap at a time
    dict(M=160, B=128, L=600, conv_width=9),                                           # too many positions: the separate kernels
]


@pytest.mark.parametrize("case", CASES, ids=[str(i) for i in range(len(CASES))])
def test_small_scans(case):
    c = dict(case)
    share, stop = c.pop("protect_share", 0.0), c.pop("stop", None)
    w = inputs.Workload(**{**dict(name="small", dtype="f32", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=64, seed=31,
                                  conv_gain=2.0), **c})
    if stop:                       # rectified sums in bf16: rounding differences grow from step to step (a row sum near zero)
        w = w.replace(L=stop)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    protect = (torch.rand(w.M, generator=torch.Generator().manual_seed(3)) < share) if share else None
    want = oracle_forward(w, q, k, v, cw, cb, **({"protect": protect} if share else {}))
    a = gpu_forward(w, q, k, v, cw, cb, impl=1, history=True, protect=protect)
    compare_scan(w, a, want, what="all blocks at once")
    for other in (gpu_forward(w, q, k, v, cw, cb, impl=1, history=False, protect=protect),
                  gpu_forward(w, q, k, v, cw, cb, impl=1, history=3, protect=protect),
                  gpu_forward(w, q, k, v, cw, cb, impl=1, step_by_step=True, protect=protect)):
        assert a[3:] == other[3:]
        for x, y in zip(a[:3], other[:3]):
            assert torch.equal(x, y)


@pytest.mark.parametrize("case", [
    dict(M=12000, B=16, L=40),                             # the LDS of a compute unit would not hold a row of M + B scores
    dict(M=5000, B=16, L=40, dtype="bf16", n_q_heads=2),   # nor 64 KB four of them
    dict(M=5000, B=700, L=2150, head_dim=16),              # past the 2048 positions a row may have: another kernel
], ids=str)
def test_first_blocks_of_a_large_cache(case):
    """Few live slots in a cache far larger than the row attention's limit: what a block needs goes by what it sees."""
    w = inputs.Workload(**{**dict(name="large", dtype="f32", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=64, seed=37,
                                  conv_width=3), **case})
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    want = oracle_forward(w, q, k, v, cw, cb)
    a = gpu_forward(w, q, k, v, cw, cb, impl=1)
    compare_scan(w, a, want, what="scan")
    b = gpu_forward(w, q, k, v, cw, cb, impl=1, step_by_step=True)
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", [64, 65, 100, 128, 129])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_widths_around_the_columns_of_a_lane(d, dtype):
    """Row attention with one column a lane, with two, the second one cut, and the first width that goes to a workgroup per row
    (bf16 rows are 16-byte aligned: widths rounded up to a multiple of 8)."""
    if dtype == "bf16":
        d = (d + 7) // 8 * 8
    w = inputs.Workload(name="width", dtype=dtype, batch=2, n_q_heads=2, n_kv_heads=1, head_dim=d, M=20, B=12, L=100, seed=41,
                        conv_width=3)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    a = gpu_forward(w, q, k, v, cw, cb, impl=1, history=True)
    compare_scan(w, a, oracle_forward(w, q, k, v, cw, cb), what=f"d = {d}")
    for x, y in zip(a[:3], gpu_forward(w, q, k, v, cw, cb, impl=1, history=False)[:3]):
        assert torch.equal(x, y)
