"""A block step whose attention shares the compression's launch: the same bits as the two launches, and the choice between
the two by the number of workgroups."""
import pytest
import torch

from paper_2406_05317_amd import binding as lb
from paper_2406_05317_amd import inputs
from parity_util import compare_scan, gpu_forward, oracle_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    dict(B=1, M=128, n_kv_heads=32, n_q_heads=32),                       # one token: 128 + 32 workgroups
    dict(B=2, M=512, n_kv_heads=4, n_q_heads=32, len0=511),              # grouped heads, one slot short
    dict(B=2, M=96, n_kv_heads=2, n_q_heads=2, conv_width=21, norm=1),
    dict(B=77, M=256, n_kv_heads=8, n_q_heads=32, conv_width=21, conv_in=1, norm=1),
    dict(B=128, M=64, n_kv_heads=4, n_q_heads=4, conv_in=1),             # one query tile, whole
    dict(B=129, M=32, n_kv_heads=1, n_q_heads=1, len0=0),                # two, the second one row; an empty cache
    dict(B=200, M=256, n_kv_heads=8, n_q_heads=32),
    dict(B=130, M=128, n_kv_heads=16, n_q_heads=96, joint=True),         # 64 + 192: every compute unit of 256
    dict(B=130, M=128, n_kv_heads=16, n_q_heads=112, joint=False),       # 64 + 224: one launch each
    dict(B=1, M=128, n_kv_heads=4, n_q_heads=8, protect=True, joint=False),
], ids=str)
def test_one_launch_or_two_give_the_same_bits(case):
    c = dict(case)
    len0, joint, protect = c.pop("len0", c["M"]), c.pop("joint", True), c.pop("protect", False)
    w = inputs.Workload(**{**dict(name="step", dtype="bf16", batch=1, head_dim=128, L=c["B"], conv_width=15, seed=3), **c})
    cfg = lb.config_for(w)
    if lb.lococo_describe_path(cfg, w.B)["compute_units"] != 256:
        joint = None                                     # (the counts above are for 256)
    g = torch.Generator(device="cuda").manual_seed(8)
    rnd = lambda *s, sd=0.3: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, sd, generator=g)
    q, k, v = rnd(1, w.n_q_heads, w.B, 128), rnd(1, w.n_kv_heads, w.B, 128), rnd(1, w.n_kv_heads, w.B, 128)
    ck, cv = rnd(1, w.n_kv_heads, w.M, 128), rnd(1, w.n_kv_heads, w.M, 128)
    cw = rnd(w.M, 256 if w.conv_in else 128, w.conv_width, sd=0.05)
    out = []
    for one_call in (True, False):
        cache = lb.Cache(cfg, "cuda")
        cache.load(ck, cv, len0)
        if protect:
            cache.set_protect(torch.arange(w.M).view(1, 1, -1).expand(1, w.n_kv_heads, -1).numpy() < 3)
        o = torch.full_like(q, float("nan"))
        ws = lb.workspace(cfg, w.B, w.B, history=False)
        lb.lococo_timing_begin()
        if one_call:
            lb.lococo_segment_step(cfg, q, k, v, o, cw, None, cache, ws)
        else:                                            # a scan of one block: attention, then the compression
            lb.lococo_sequence_forward(cfg, q, k, v, o, cw, None, cache, w.B, ws)
        ran = set(lb.lococo_timing_end()) - {"repack_filters"}
        two = {"compress_mfma", "attn_decode" if w.B == 1 else "attn_mfma"}
        if joint is not None:
            assert ran == ({"compress_mfma"} if one_call and joint else two), ran
        out.append((o, cache.k.clone(), cache.v.clone(), cache.len))
    for x, y in zip(*out):
        assert x == y if isinstance(x, int) else torch.equal(x, y)


@pytest.mark.parametrize("case", [
    dict(M=64, B=64, L=256, conv_width=21, norm=1),          # a block's own tiles and the cache's, two each
    dict(M=32, B=16, L=96),                                  # no tile of the block's own
    dict(M=32, B=1, L=34, conv_width=21),
    dict(M=96, B=160, L=480),                                # an empty cache at the first step
    dict(M=64, B=40, L=190, norm=1, n_kv_heads=1),           # a fill, a partly filled cache, a ragged block
    dict(M=64, B=64, L=256, conv_width=21, protect=True),
], ids=str)
def test_steps_over_keys_and_values_that_wait_for_nobody(case):
    """Filters over [K | V], pairs of workgroups: the first step of a launch walks all its tiles with the key half of the filters
    before it takes the value half, later ones do either for the block's own tiles first.  The same bits, and the oracle's."""
    c = dict(case)
    protect = c.pop("protect", False)
    w = inputs.Workload(**{**dict(name="kvstep", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, conv_width=15,
                                  conv_in=1, seed=5), **c})
    cfg = lb.config_for(w)
    assert lb.lococo_describe_path(cfg, w.B)["step_pipeline"] == 2
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    mask = (torch.arange(w.M) < 5).view(1, 1, -1).expand(1, w.n_kv_heads, -1).numpy() if protect else None
    scan = gpu_forward(w, q, k, v, cw, cb, history=True, protect=mask)
    steps = gpu_forward(w, q, k, v, cw, cb, step_by_step=True, protect=mask)
    for x, y in zip(scan, steps):
        assert x == y if isinstance(x, int) else torch.equal(x, y)
    compare_scan(w, scan, oracle_forward(w, q, k, v, cw, cb, protect=mask), what=str(case))
