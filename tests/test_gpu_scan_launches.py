"""What a scan no longer launches on its own: leading fill blocks go with the filters, the last state goes straight to the caller's
buffer where the attention behind the scan does not read it.  Bit for bit against the step-by-step schedule."""
import pytest
import torch

from paper_2406_05317_amd import binding as lb

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)], ids=["bf16", "f32"])
@pytest.mark.parametrize("cur", [0, 1])
@pytest.mark.parametrize("case", [
    dict(M=96, B=20, L=20 * 4),                  # fill blocks alone
    dict(M=96, B=20, L=20 * 5),                  # one compression
    dict(M=96, B=20, L=20 * 6),                  # two: the last state lands in the buffer the first one came from
    dict(M=96, B=20, L=20 * 7 + 3),              # three and a short block
    dict(M=32, B=7, L=60, len0=9),               # live slots ahead of the fills
    dict(M=64, B=64, L=64 * 3, len0=64),         # none to fill
    dict(M=64, B=16, L=16 * 9, history=3),       # windows of three blocks, fills across two of them
    dict(M=64, B=16, L=16 * 10, history=3),
], ids=str)
def test_schedules_leave_the_same_bits(case, cur, dtype, d):
    c = dict(dict(len0=0, history=1), **case)
    g = torch.Generator(device=DEV).manual_seed(11)
    b, hq, hkv, M, L = 2, 4, 2, c["M"], c["L"]
    rnd = lambda *s: torch.empty(s, dtype=dtype, device=DEV).normal_(0, 0.3, generator=g)
    wide = rnd(b, L, hq + 2 * hkv, d)            # token-major, as a projection leaves them: heads d apart, tokens (hq + 2 hkv) d
    q, k, v = (wide[:, :, i:j].transpose(1, 2) for i, j in ((0, hq), (hq, hq + hkv), (hq + hkv, hq + 2 * hkv)))
    w, ck, cv = rnd(M, d, 15) * 0.2, rnd(b, hkv, M, d), rnd(b, hkv, M, d)
    cfg = lb.make_config(dtype=dtype, batch=b, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, M=M, conv_width=15)
    got = []
    for history in (c["history"], 0):
        cache = lb.Cache(cfg, DEV)
        cache.c.cur = cur
        cache.load(ck, cv, c["len0"])
        assert cache.cur == cur
        o = torch.full((b, hq, L, d), float("nan"), dtype=dtype, device=DEV)
        ws = lb.workspace(cfg, L, c["B"], history, DEV)
        lb.lococo_sequence_forward(cfg, q, k, v, o, w, None, cache, c["B"], ws)
        torch.cuda.synchronize()
        got.append((o, cache.k[:, :, :cache.len].clone(), cache.v[:, :, :cache.len].clone(), cache.len, cache.cur))
    assert got[0][3:] == got[1][3:]
    for x, y in zip(got[0][:3], got[1][:3]):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y)


@pytest.mark.parametrize("blocks", [1, 2, 3])
@pytest.mark.parametrize("cur", [0, 1])
def test_scans_over_keys_and_values_leave_the_same_bits(cur, blocks):
    """Their area for the key-side logits is where scans over the keys are told the place of the last state."""
    g = torch.Generator(device=DEV).manual_seed(12)
    b, h, M, B, d = 1, 4, 64, 50, 128
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0, 0.3, generator=g)
    q, k, v = (rnd(b, h, B * blocks, d) for _ in range(3))
    w, ck, cv = rnd(M, 2 * d, 15) * 0.2, rnd(b, h, M, d), rnd(b, h, M, d)
    cfg = lb.make_config(dtype=torch.bfloat16, batch=b, n_q_heads=h, n_kv_heads=h, head_dim=d, M=M, conv_width=15, conv_in=1, norm=1)
    got = []
    for history in (1, 0):
        cache = lb.Cache(cfg, DEV)
        cache.c.cur = cur
        cache.load(ck, cv, M)
        o = torch.full_like(q, float("nan"))
        lb.lococo_sequence_forward(cfg, q, k, v, o, w, None, cache, B, lb.workspace(cfg, B * blocks, B, history, DEV))
        torch.cuda.synchronize()
        got.append((o, cache.k.clone(), cache.v.clone(), cache.len, cache.cur))
    assert got[0][3:] == got[1][3:]
    for x, y in zip(got[0][:3], got[1][:3]):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y)


@pytest.mark.parametrize("steps", [2, 3])
@pytest.mark.parametrize("case", [
    dict(M=64, heads=4, width=21),               # two workgroups a pair that take the steps in turn
    dict(M=64, heads=4, width=15),               # so, few positions: the build that can tell its last step
    dict(M=512, heads=4, width=15),              # more, but few steps
    dict(M=512, heads=4, width=15, steps=11),    # and so many that the state is copied
    dict(M=96, heads=64, width=21),              # one, a chain each
    dict(M=96, heads=96, width=15),              # several chains a workgroup
    dict(M=128, heads=128, width=15),            # 64 slots a workgroup
    dict(M=128, heads=160, width=15),            # and several chains
    dict(M=96, heads=64, width=15),              # one chain each, width 15: the state is copied
], ids=str)
def test_builds_whose_last_step_writes_to_the_caller(case, steps):
    g = torch.Generator(device=DEV).manual_seed(13)
    h, M, B, d, steps = case["heads"], case["M"], 40, 128, case.get("steps", steps)
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0, 0.3, generator=g)
    q, k, v = (rnd(1, h, B * steps - 3, d) for _ in range(3))
    w, ck, cv = rnd(M, d, case["width"]) * 0.2, rnd(1, h, M, d), rnd(1, h, M, d)
    cfg = lb.make_config(dtype=torch.bfloat16, batch=1, n_q_heads=h, n_kv_heads=h, head_dim=d, M=M, conv_width=case["width"])
    got = []
    for history in (1, 0):
        cache = lb.Cache(cfg, DEV)
        cache.load(ck, cv, M)
        o = torch.full_like(q, float("nan"))
        lb.lococo_sequence_forward(cfg, q, k, v, o, w, None, cache, B, lb.workspace(cfg, q.shape[2], B, history, DEV))
        torch.cuda.synchronize()
        got.append((o, cache.k.clone(), cache.v.clone(), cache.len, cache.cur))
    assert got[0][3:] == got[1][3:]
    for x, y in zip(got[0][:3], got[1][:3]):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y)


@pytest.mark.parametrize("steps", [1, 2, 3])
@pytest.mark.parametrize("case", [
    dict(dtype=torch.float32, d=32, M=24, width=5),
    dict(dtype=torch.float32, d=80, M=17, width=3),               # a second slot tile of one slot
    dict(dtype=torch.float32, d=64, M=16, width=3, conv_in=1),    # values in the rows of the keys
    dict(dtype=torch.bfloat16, d=64, M=20, width=9),
    dict(dtype=torch.bfloat16, d=40, M=20, width=5, heads=3, protect=True),
], ids=str)
def test_small_scans_hand_over_their_rows(case, steps):
    g = torch.Generator(device=DEV).manual_seed(14)
    h, M, d, dtype, conv_in = case.get("heads", 2), case["M"], case["d"], case["dtype"], case.get("conv_in", 0)
    B = M - 3
    rnd = lambda *s: torch.empty(s, dtype=dtype, device=DEV).normal_(0, 0.3, generator=g)
    q, k, v = (rnd(2, h, B * steps - 1, d) for _ in range(3))
    w, ck, cv = rnd(M, d * (1 + conv_in), case["width"]) * 0.2, rnd(2, h, M, d), rnd(2, h, M, d)
    cfg = lb.make_config(dtype=dtype, batch=2, n_q_heads=h, n_kv_heads=h, head_dim=d, M=M, conv_width=case["width"], conv_in=conv_in, impl=1)
    got = []
    for history in (1, 2, 0):
        cache = lb.Cache(cfg, DEV)
        cache.load(ck, cv, M)
        if case.get("protect"):
            cache.set_protect((torch.arange(M) % 5 == 0).view(1, 1, -1).expand(2, h, -1).numpy())
        o = torch.full_like(q, float("nan"))
        lb.lococo_sequence_forward(cfg, q, k, v, o, w, None, cache, B, lb.workspace(cfg, q.shape[2], B, history, DEV))
        torch.cuda.synchronize()
        got.append((o, cache.k.clone(), cache.v.clone(), cache.len, cache.cur))
    for other in got[1:]:
        assert got[0][3:] == other[3:]
        for x, y in zip(got[0][:3], other[:3]):
            assert torch.isfinite(x.float()).all() and torch.equal(x, y)
