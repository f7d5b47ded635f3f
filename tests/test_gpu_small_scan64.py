"""The single-precision small-scan kernel for head_dim 64: every filter width it is built for, one to three slot tiles in a
workgroup, the edges of its position tiles and of the four forms of its Eq. 6, addresses that are only 4-byte aligned."""
import pytest
import torch

from paper_2406_05317_amd import inputs
from parity_util import compare_scan, gpu_forward, oracle_forward, to_np

pytestmark = pytest.mark.gpu


def workload(**case):
    return inputs.Workload(**{**dict(name="scan64", dtype="f32", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=64, seed=53,
                                     conv_gain=2.0), **case})


def check(w, protect=None):
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    kw = {} if protect is None else {"protect": protect}
    a = gpu_forward(w, q, k, v, cw, cb, impl=1, history=True, protect=protect)
    compare_scan(w, a, oracle_forward(w, q, k, v, cw, cb, **kw), what="all blocks at once")
    for other in (gpu_forward(w, q, k, v, cw, cb, impl=1, history=False, protect=protect),
                  gpu_forward(w, q, k, v, cw, cb, impl=1, history=2, protect=protect)):
        assert a[3:] == other[3:]
        for x, y in zip(a[:3], other[:3]):
            assert torch.equal(x, y)


@pytest.mark.parametrize("width", [3, 5, 7, 9, 11, 13, 15, 21])
def test_widths(width):
    # two slot tiles, the second with one live slot; the last block shorter, and a first compression on fewer live slots
    check(workload(M=17, B=12, L=111, conv_width=width, n_q_heads=2, n_kv_heads=2, per_head_filters=True))


@pytest.mark.parametrize("M,B", [(16, 16), (17, 15), (16, 17), (32, 32), (33, 31), (33, 32), (48, 16), (48, 17),
                                 (64, 64), (65, 63), (65, 64), (96, 96), (1, 1), (3, 40), (8, 120)])
def test_position_tiles(M, B):
    check(workload(M=M, B=B, L=4 * (M + B) + 5, conv_width=5))


@pytest.mark.parametrize("M,width", [(20, 3), (40, 5), (80, 9)])
@pytest.mark.parametrize("norm", [0, 1, 2])
def test_norms_bias_and_protected_slots(M, width, norm):
    extra = dict(filter_abs=True) if norm == 2 else {}
    w = workload(M=M, B=M - 7, L=5 * M, conv_width=width, norm=norm, bias_sigma=0.3, n_q_heads=2, n_kv_heads=1, batch=2, **extra)
    check(w)
    check(w, protect=torch.rand(M, generator=torch.Generator().manual_seed(5)) < 0.3)


def test_rows_that_start_anywhere():
    """Token strides of 65 floats, a first element and filters that are 4-byte aligned only: the same bits as from whole lines."""
    from paper_2406_05317_amd import binding as lb
    w = workload(M=20, B=18, L=150, conv_width=7, n_q_heads=2, n_kv_heads=2)
    q, k, v = inputs.qkv(w)
    cw, _ = inputs.conv_filters(w)
    want = gpu_forward(w, q, k, v, cw, None, impl=1, history=True)

    def shifted(x):
        wide = torch.full(x.shape[:-1] + (65,), float("nan"), device="cuda").flatten()
        wide = torch.cat([wide, wide.new_full((1,), float("nan"))])[1:].view(x.shape[:-1] + (65,))
        wide[..., :64] = x.to("cuda")
        return wide[..., :64]

    cfg = lb.config_for(w, impl=1)
    filters = torch.cat([torch.zeros(1), cw.flatten()]).to("cuda")[1:].view(cw.shape)
    assert filters.data_ptr() % 16
    cache, o = lb.Cache(cfg, "cuda"), shifted(torch.zeros_like(q))
    ws = lb.workspace(cfg, w.L, w.B, True, "cuda")
    lb.lococo_sequence_forward(cfg, shifted(q), shifted(k), shifted(v), o, filters, None, cache, w.B, ws)
    torch.cuda.synchronize()
    for x, y in zip((o, cache.k, cache.v), want[:3]):
        assert (to_np(x) == to_np(y)).all()
