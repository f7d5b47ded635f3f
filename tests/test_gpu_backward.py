"""GPU parity of the backward pass of one block step against the CPU oracle's backward (itself
pinned by finite differences of the forward oracle), single steps in every branch and variant and
a scan of several steps walked in reverse."""
import numpy as np
import pytest
import torch

from oracle import lococo_oracle as orc
from paper_2406_05317_amd import binding as lb
from paper_2406_05317_amd import inputs
from parity_util import oracle_scan_backward

pytestmark = pytest.mark.gpu


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


def _gpu_step_backward(w, cfg, q, k, v, cw, cb, ck, cv, m, d_o, gk, gv, dW, dB, protect=None):
    dev = "cuda"
    cache = lb.Cache(cfg, dev)
    cache.load(torch.as_tensor(ck).to(dev, w.torch_dtype), torch.as_tensor(cv).to(dev, w.torch_dtype), m)
    cache.set_protect(protect)
    f32 = lambda x: torch.as_tensor(np.asarray(x), dtype=torch.float32).to(dev).contiguous()
    out = dict(dq=torch.full(q.shape, float("nan"), device=dev), dk=torch.full(k.shape, float("nan"), device=dev),
               dv=torch.full(v.shape, float("nan"), device=dev),
               d_cache_k=torch.full(ck.shape, float("nan"), device=dev),
               d_cache_v=torch.full(cv.shape, float("nan"), device=dev))
    ws = torch.empty(max(lb.lococo_backward_workspace_bytes(cfg, q.shape[2], m), 256), dtype=torch.uint8, device=dev)
    lb.lococo_segment_step_backward(cfg, q.to(dev), k.to(dev), v.to(dev), None if cw is None else cw.to(dev),
                                    None if cb is None else cb.to(dev), cache, f32(d_o), f32(gk), f32(gv),
                                    out["dq"], out["dk"], out["dv"], out["d_cache_k"], out["d_cache_v"], dW, dB, ws)
    torch.cuda.synchronize()
    return {n: t.cpu().numpy() for n, t in out.items()}


CASES = [
    dict(name="f32 compress", dtype="f32", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=32, B=16, M=24, m=24,
         conv_width=5),
    dict(name="f32 partial cache", dtype="f32", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=16, B=12, M=20, m=14,
         conv_width=3),
    dict(name="f32 fill", dtype="f32", batch=1, n_q_heads=2, n_kv_heads=1, head_dim=16, B=6, M=20, m=5,
         conv_width=3),
    dict(name="bf16 relu-sum", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=64, B=32, M=48, m=48,
         conv_width=7, norm=1, bias_sigma=0.5),
    dict(name="f32 kv channels per-head", dtype="f32", batch=2, n_q_heads=2, n_kv_heads=2, head_dim=8, B=10, M=12,
         m=12, conv_width=3, conv_in=1, per_head_filters=True, bias_sigma=0.3),
    dict(name="bf16 protected", dtype="bf16", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, B=40, M=64, m=64,
         conv_width=15, protect=True),
    # the Eq. 5 contractions on the matrix cores (bf16, head_dim 128, keys-only filters; impl = AUTO)
    dict(name="mfma protected", dtype="bf16", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, B=40, M=64, m=64,
         conv_width=15, protect=True, impl=0),
    dict(name="mfma ragged per-head", dtype="bf16", batch=2, n_q_heads=2, n_kv_heads=2, head_dim=128, B=100, M=160,
         m=160, conv_width=15, per_head_filters=True, bias_sigma=0.4, impl=0),     # T = 260, slots padded to 192
    dict(name="mfma partial cache relu-sum width 21", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128,
         B=70, M=128, m=90, conv_width=21, norm=1, bias_sigma=0.5, impl=0),
    dict(name="mfma several tiles grouped heads", dtype="bf16", batch=3, n_q_heads=2, n_kv_heads=1, head_dim=128,
         B=256, M=256, m=256, conv_width=15, impl=0),                              # 4 position x 2 slot tiles
    dict(name="mfma fill step", dtype="bf16", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=128, B=24, M=96, m=40,
         conv_width=15, impl=0),
    dict(name="mfma head_dim 64 (plain contractions only)", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2,
         head_dim=64, B=40, M=64, m=64, conv_width=7, bias_sigma=0.3, impl=0),
    dict(name="mfma [K|V] filters width 21 relu-sum per-head", dtype="bf16", batch=2, n_q_heads=4, n_kv_heads=2,
         head_dim=128, B=72, M=160, m=160, conv_width=21, conv_in=1, norm=1, per_head_filters=True, bias_sigma=0.4,
         impl=0),                                                                  # the compressor as the paper prints it
    dict(name="mfma [K|V] filters partial cache", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=1, head_dim=128,
         B=100, M=128, m=60, conv_width=15, conv_in=1, impl=0),
    dict(name="mfma width 3", dtype="bf16", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, B=33, M=32, m=20,
         conv_width=3, impl=0),
]


@pytest.mark.parametrize("case", CASES, ids=[c["name"] for c in CASES])
def test_step_backward_matches_the_oracle(case):
    c = dict(case)
    c.pop("name")
    m, use_protect, impl = c.pop("m"), c.pop("protect", False), c.pop("impl", 1)
    w = inputs.Workload(name="bwd", L=c["B"], seed=11, conv_gain=3.0, **c)
    rng = np.random.default_rng(3)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    ck[:, :, m:], cv[:, :, m:] = 0, 0
    d_o = rng.standard_normal(q.shape)
    gk, gv = rng.standard_normal(chains), rng.standard_normal(chains)
    ln = min(w.M, m + w.B)
    gk[:, :, ln:], gv[:, :, ln:] = 0.0, 0.0
    protect = (rng.random((w.batch, w.n_kv_heads, w.M)) < 0.2) if use_protect else None
    want = orc.step_backward(q, k, v, ck, cv, m, cw, cb, d_o, gk, gv, M=w.M, conv_in=w.conv_in, norm=w.norm,
                             protect=protect)
    cfg = lb.config_for(w, impl=impl)
    dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
    dB = None if cb is None else torch.zeros(cb.shape, dtype=torch.float32, device="cuda")
    got = _gpu_step_backward(w, cfg, q, k, v, cw, cb, ck, cv, m, d_o, gk, gv, dW, dB, protect)
    got["d_conv_w"], got["d_conv_b"] = dW.cpu().numpy(), None if dB is None else dB.cpu().numpy()
    errs = {}
    for n in ("dq", "dk", "dv", "d_cache_k", "d_cache_v", "d_conv_w", "d_conv_b"):
        if want[n] is None:
            continue
        if m + w.B <= w.M and n in ("d_conv_w", "d_conv_b"):
            assert not got[n].any()
            continue
        if n == "d_conv_b" and w.norm == 0:
            # a softmax row does not change when its bias does: the gradient is zero up to rounding
            assert np.abs(want[n]).max() < 1e-12
            assert np.abs(got[n]).max() < 1e-5 * np.abs(want["d_conv_w"]).max()
            continue
        errs[n] = _rel(got[n], want[n])
        assert errs[n] < 2e-4, (n, errs[n])          # fp32 sums of up to ~1e3 terms against double
    assert not got["d_cache_k"][:, :, m:].any() and not got["d_cache_v"][:, :, m:].any()
    print(case["name"], {n: f"{e:.1e}" for n, e in errs.items()})


def _draw_step(i):
    rng = np.random.default_rng(17000 + i)
    ch = lambda xs: xs[int(rng.integers(len(xs)))]
    dtype = ch(["bf16", "bf16", "f32"])
    d = ch([64, 128, 128, 128]) if dtype == "bf16" else ch([8, 16, 32, 64])
    M = ch([12, 20, 32, 48, 64, 96, 128, 160, 192, 256])
    Hkv = ch([1, 2, 3])
    case = dict(dtype=dtype, head_dim=d, M=M, B=ch([1, 6, 24, 33, 40, 64, 100, 128, 200]),
                conv_width=ch([1, 3, 5, 7, 15, 21]), norm=ch([0, 0, 1]), conv_in=ch([0, 0, 1]),
                per_head_filters=ch([False, False, True]), bias_sigma=ch([0.0, 0.4]), n_kv_heads=Hkv,
                n_q_heads=Hkv * ch([1, 2, 4]), batch=ch([1, 2]), conv_gain=ch([1.0, 3.0]))
    return case, ch([M, M, int(rng.integers(0, M + 1))]), ch([0, 1]), ch([False, False, True]), rng


@pytest.mark.parametrize("i", range(40))
def test_step_backward_on_a_drawn_case(i):
    """A seeded sweep over storage type, sizes, occupancy, filter width, normalisation, convolution input, filter
    sharing, grouped heads, protected slots and kernel family: every gradient against the oracle's."""
    case, m, impl, use_protect, rng = _draw_step(i)
    w = inputs.Workload(name=f"bwd{i}", L=case["B"], seed=17000 + i, **case)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    ck[:, :, m:], cv[:, :, m:] = 0, 0
    d_o = rng.standard_normal(q.shape)
    gk, gv = rng.standard_normal(chains), rng.standard_normal(chains)
    ln = min(w.M, m + w.B)
    gk[:, :, ln:], gv[:, :, ln:] = 0.0, 0.0
    protect = (rng.random((w.batch, w.n_kv_heads, w.M)) < 0.2) if use_protect else None
    want = orc.step_backward(q, k, v, ck, cv, m, cw, cb, d_o, gk, gv, M=w.M, conv_in=w.conv_in, norm=w.norm,
                             protect=protect)
    cfg = lb.config_for(w, impl=impl)
    dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
    dB = None if cb is None else torch.zeros(cb.shape, dtype=torch.float32, device="cuda")
    got = _gpu_step_backward(w, cfg, q, k, v, cw, cb, ck, cv, m, d_o, gk, gv, dW, dB, protect)
    got["d_conv_w"], got["d_conv_b"] = dW.cpu().numpy(), None if dB is None else dB.cpu().numpy()
    what = f"{w} m={m} impl={impl} protect={use_protect}"
    for n in ("dq", "dk", "dv", "d_cache_k", "d_cache_v", "d_conv_w", "d_conv_b"):
        if want[n] is None:
            continue
        if m + w.B <= w.M and n in ("d_conv_w", "d_conv_b"):
            assert not got[n].any(), (n, what)
        elif n == "d_conv_b" and w.norm == 0:
            assert np.abs(got[n]).max() < 1e-5 * max(np.abs(want["d_conv_w"]).max(), 1e-30), (n, what)
        else:
            assert np.all(np.isfinite(got[n])), (n, what)
            assert _rel(got[n], want[n]) < 2e-4, (n, _rel(got[n], want[n]), what)
    assert not got["d_cache_k"][:, :, m:].any() and not got["d_cache_v"][:, :, m:].any()


def test_scan_backward_in_reverse_matches_the_oracle_and_a_directional_difference():
    """Three block steps (fill, compress, compress): forward on the GPU keeping the cache states,
    backward step by step in reverse, filter gradients collected in one buffer.  Checked against
    the oracle's backward walked the same way, and the filter gradient against a finite
    difference of the ORACLE forward along a random direction."""
    w = inputs.Workload(name="bwdscan", dtype="f32", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=16, L=36, B=12,
                        M=16, conv_width=5, seed=4, conv_gain=3.0)
    rng = np.random.default_rng(8)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    r_o = rng.standard_normal(q.shape)
    r_k, r_v = rng.standard_normal((1, 2, w.M, 16)), rng.standard_normal((1, 2, w.M, 16))

    def loss(cw_):
        o, ck, cv, _ = orc.sequence_forward(q, k, v, cw_, cb, B=w.B, M=w.M)
        return (o * r_o).sum() + (ck * r_k).sum() + (cv * r_v).sum()

    # forward states from the oracle (the GPU forward agrees to 1e-5, tested elsewhere)
    states = [(np.zeros((1, 2, w.M, 16)), np.zeros((1, 2, w.M, 16)), 0)]
    for s0 in range(0, w.L, w.B):
        ck, cv, m = states[-1]
        _, nk, nv, ln = orc.sequence_forward(q[:, :, s0:s0 + w.B], k[:, :, s0:s0 + w.B], v[:, :, s0:s0 + w.B], cw, cb,
                                             B=w.B, M=w.M, cache_k=ck, cache_v=cv, cache_len=m)
        states.append((nk, nv, ln))
    cfg = lb.config_for(w, impl=1)
    dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
    want_dW = np.zeros(cw.shape)
    gk, gv = r_k.copy(), r_v.copy()
    wk, wv = r_k.copy(), r_v.copy()
    for n in reversed(range(w.L // w.B)):
        sl = slice(n * w.B, (n + 1) * w.B)
        ck, cv, m = states[n]
        got = _gpu_step_backward(w, cfg, q[:, :, sl].contiguous(), k[:, :, sl].contiguous(), v[:, :, sl].contiguous(),
                                 cw, None, torch.as_tensor(ck), torch.as_tensor(cv), m, r_o[:, :, sl], gk, gv, dW, None)
        ref = orc.step_backward(q[:, :, sl], k[:, :, sl], v[:, :, sl], ck, cv, m, cw, None, r_o[:, :, sl], wk, wv, M=w.M)
        if ref["d_conv_w"] is not None:
            want_dW += ref["d_conv_w"]
        gk, gv = got["d_cache_k"], got["d_cache_v"]
        wk, wv = ref["d_cache_k"], ref["d_cache_v"]
        assert _rel(got["dq"], ref["dq"]) < 2e-4 and _rel(got["dk"], ref["dk"]) < 2e-4
    assert _rel(dW.cpu().numpy(), want_dW) < 2e-4
    direction = rng.standard_normal(cw.shape)
    eps = 1e-5
    cw64 = cw.double().numpy()
    fd = (loss(cw64 + eps * direction) - loss(cw64 - eps * direction)) / (2 * eps)
    assert abs((dW.cpu().numpy() * direction).sum() - fd) < 2e-4 * max(1.0, abs(fd))


# ---- the whole scan in one call ---------------------------------------------------------------

def _gpu_scan_backward(w, cfg, q, k, v, cw, cb, ck0, cv0, len0, r_o, r_k, r_v, protect):
    dev = "cuda"
    cache = lb.Cache(cfg, dev)
    cache.load(torch.as_tensor(ck0).to(dev, w.torch_dtype), torch.as_tensor(cv0).to(dev, w.torch_dtype), len0)
    cache.set_protect(protect)
    before = (cache.k.clone(), cache.v.clone(), cache.len, cache.cur)
    f32 = lambda x: None if x is None else torch.as_tensor(np.asarray(x), dtype=torch.float32).to(dev).contiguous()
    nan = lambda shape: torch.full(tuple(shape), float("nan"), device=dev)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    out = dict(dq=nan(q.shape), dk=nan(k.shape), dv=nan(v.shape), d_cache0_k=nan(chains), d_cache0_v=nan(chains))
    dW = torch.zeros(cw.shape, dtype=torch.float32, device=dev)
    dB = None if cb is None else torch.zeros(cb.shape, dtype=torch.float32, device=dev)
    L = q.shape[2]
    ws = torch.empty(lb.lococo_sequence_backward_workspace_bytes(cfg, L, w.B), dtype=torch.uint8, device=dev)
    lb.lococo_sequence_backward(cfg, q.to(dev), k.to(dev), v.to(dev), w.B, cw.to(dev), None if cb is None else cb.to(dev),
                                cache, f32(r_o), f32(r_k), f32(r_v), out["dq"], out["dk"], out["dv"],
                                out["d_cache0_k"], out["d_cache0_v"], dW, dB, ws)
    torch.cuda.synchronize()
    assert torch.equal(cache.k, before[0]) and torch.equal(cache.v, before[1])      # the starting state is left alone
    assert (cache.len, cache.cur) == before[2:]
    got = {n: t.cpu().numpy() for n, t in out.items()}
    got["d_conv_w"], got["d_conv_b"] = dW.cpu().numpy(), None if dB is None else dB.cpu().numpy()
    return got


SCAN_CASES = [
    # fill, fill + compress boundary, compress...; a ragged last block; grouped heads
    dict(name="f32 from an empty cache, ragged tail", dtype="f32", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=16,
         L=77, B=12, M=30, conv_width=5, len0=0, tol=3e-4),
    dict(name="f32 from a half-full cache, relu-sum, bias, per-head", dtype="f32", batch=1, n_q_heads=2, n_kv_heads=2,
         head_dim=8, L=60, B=10, M=24, conv_width=3, norm=1, bias_sigma=0.4, per_head_filters=True, len0=13,
         tol=3e-4),
    dict(name="f32 [K|V] filters, protected slots, no final gradient", dtype="f32", batch=1, n_q_heads=2,
         n_kv_heads=1, head_dim=16, L=64, B=16, M=16, conv_width=5, conv_in=1, len0=16, protect=True, final=False,
         tol=3e-4),
    dict(name="f32 one block", dtype="f32", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=16, L=9, B=16, M=12,
         conv_width=3, len0=8, tol=3e-4),
    dict(name="f32 fills only", dtype="f32", batch=2, n_q_heads=2, n_kv_heads=1, head_dim=16, L=20, B=8, M=32,
         conv_width=3, len0=4, tol=3e-4),
    # bf16 storage, the fused compression kernel in the forward, the matrix-core contractions in the
    # backward.  The forward states are rounded to bf16 on both sides (the oracle rounds the exact value,
    # the kernel an fp32 one), so a few state entries differ by one bf16 step: the tolerance is that of
    # the storage type, not of the arithmetic.
    dict(name="bf16 head_dim 128 fused forward", dtype="bf16", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=128,
         L=5 * 64 + 20, B=64, M=64, conv_width=15, len0=0, impl=0, tol=2e-3, state_round="bf16"),
    dict(name="bf16 head_dim 128 [K|V] width 21", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2,
         head_dim=128, L=4 * 96, B=96, M=128, conv_width=21, conv_in=1, bias_sigma=0.4, len0=40, impl=0,
         tol=2e-3, state_round="bf16"),
    # relu + sum has a kink at every zero of a logit: where the two sides' states differ by a bf16 step and
    # a logit sits within that of zero, one side's rectifier passes it and the other's does not, and the
    # gradient jumps by that entry's whole share: the bound is a few such entries, not a rounding level
    dict(name="bf16 head_dim 128 [K|V] width 21 relu-sum", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2,
         head_dim=128, L=4 * 96, B=96, M=128, conv_width=21, conv_in=1, norm=1, bias_sigma=0.4, len0=40, impl=0,
         tol=5e-2, state_round="bf16"),
]


@pytest.mark.parametrize("case", SCAN_CASES, ids=[c["name"] for c in SCAN_CASES])
def test_sequence_backward_matches_the_oracle_walked_in_reverse(case):
    c = dict(case)
    c.pop("name")
    len0, tol, impl = c.pop("len0"), c.pop("tol"), c.pop("impl", 1)
    use_protect, final, state_round = c.pop("protect", False), c.pop("final", True), c.pop("state_round", "none")
    w = inputs.Workload(name="bwdseq", seed=23, conv_gain=3.0, **c)
    rng = np.random.default_rng(17)
    q, k, v = inputs.qkv(w)
    cw, cb = inputs.conv_filters(w)
    if w.bias_sigma == 0.0:
        cb = None
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck0 = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv0 = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    ck0[:, :, len0:], cv0[:, :, len0:] = 0, 0
    r_o = rng.standard_normal(q.shape)
    ln = min(w.M, len0 + w.L)
    r_k, r_v = rng.standard_normal(chains), rng.standard_normal(chains)
    r_k[:, :, ln:], r_v[:, :, ln:] = 0.0, 0.0
    protect = (rng.random(chains[:3]) < 0.2) if use_protect else None
    zero = np.zeros(chains)
    want = oracle_scan_backward(w, q, k, v, cw, cb, ck0.double().numpy(), cv0.double().numpy(), len0, r_o,
                                 r_k if final else zero, r_v if final else zero, protect, state_round)
    cfg = lb.config_for(w, impl=impl)
    got = _gpu_scan_backward(w, cfg, q, k, v, cw, cb, ck0, cv0, len0, r_o, r_k if final else None,
                             r_v if final else None, protect)
    errs = {}
    for n in ("dq", "dk", "dv", "d_cache0_k", "d_cache0_v", "d_conv_w", "d_conv_b"):
        if want[n] is None:
            continue
        if n == "d_conv_b" and w.norm == 0:
            continue
        if not np.abs(want[n]).max() > 0:
            assert not got[n].any(), n
            continue
        errs[n] = _rel(got[n], want[n])
        assert errs[n] < tol, (n, errs[n])
    assert not got["d_cache0_k"][:, :, len0:].any() and not got["d_cache0_v"][:, :, len0:].any()
    print(case["name"], {n: f"{e:.1e}" for n, e in errs.items()})


def test_sequence_backward_equals_the_steps_composed_by_hand_on_the_matrix_cores():
    """bf16, head_dim 128: the one-call scan backward against lococo_segment_step (forward, keeping the
    states) and lococo_segment_step_backward (reverse) called block by block: the same products, a window of
    blocks to a launch or one, so equal up to the order of sums.  Also: the filter gradient against a central
    difference of the ORACLE forward (bf16 inputs, exact arithmetic) along a random direction."""
    w = inputs.Workload(name="bwdseq_mfma", dtype="bf16", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, L=4 * 48 + 16,
                        B=48, M=64, conv_width=15, seed=5, conv_gain=3.0)
    rng = np.random.default_rng(2)
    q, k, v = inputs.qkv(w)
    cw, _ = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    r_o, r_k, r_v = rng.standard_normal(q.shape), rng.standard_normal(chains), rng.standard_normal(chains)
    cfg = lb.config_for(w, impl=0)
    zeros = torch.zeros(chains, dtype=w.torch_dtype)
    got = _gpu_scan_backward(w, cfg, q, k, v, cw, None, zeros, zeros, 0, r_o, r_k, r_v, None)

    dev = "cuda"
    cache = lb.Cache(cfg, dev)
    qd, kd, vd, cwd = q.to(dev), k.to(dev), v.to(dev), cw.to(dev)
    ws = torch.empty(max(lb.lococo_workspace_bytes(cfg, w.B, w.B, 0), 256), dtype=torch.uint8, device=dev)
    starts = list(range(0, w.L, w.B))
    states = []
    for s0 in starts:
        states.append((cache.k.clone(), cache.v.clone(), cache.len))
        if s0 == starts[-1]:
            break                                # the state after the last block is not needed
        sl = slice(s0, s0 + w.B)
        o = torch.empty((w.batch, w.n_q_heads, w.B, w.head_dim), dtype=w.torch_dtype, device=dev)
        lb.lococo_segment_step(cfg, qd[:, :, sl], kd[:, :, sl], vd[:, :, sl], o, cwd, None, cache, ws)
    dW = torch.zeros(cw.shape, dtype=torch.float32, device=dev)
    gk, gv = r_k, r_v
    hand = dict(dq=np.zeros(q.shape, np.float32), dk=np.zeros(k.shape, np.float32), dv=np.zeros(k.shape, np.float32))
    for n in reversed(range(len(starts))):
        sl = slice(starts[n], starts[n] + w.B)
        ck, cv, m = states[n]
        step = _gpu_step_backward(w, cfg, q[:, :, sl].contiguous(), k[:, :, sl].contiguous(), v[:, :, sl].contiguous(),
                                  cw, None, ck.cpu(), cv.cpu(), m,
                                  r_o[:, :, sl], gk, gv, dW, None)
        hand["dq"][:, :, sl], hand["dk"][:, :, sl], hand["dv"][:, :, sl] = step["dq"], step["dk"], step["dv"]
        gk, gv = step["d_cache_k"], step["d_cache_v"]
    for n in ("dq", "dk", "dv"):
        assert _rel(got[n], hand[n]) < 1e-5, (n, _rel(got[n], hand[n]))
    assert _rel(got["d_conv_w"], dW.cpu().numpy()) < 1e-5
    assert not got["d_cache0_k"].any() and not got["d_cache0_v"].any()      # nothing was live at the start

    def loss(cw_):
        o, ck, cv, _ = orc.sequence_forward(q, k, v, cw_, None, B=w.B, M=w.M)
        return (o * r_o).sum() + (ck * r_k).sum() + (cv * r_v).sum()

    direction = rng.standard_normal(cw.shape)
    cw64, eps = cw.double().numpy(), 1e-5
    fd = (loss(cw64 + eps * direction) - loss(cw64 - eps * direction)) / (2 * eps)
    mine = float((got["d_conv_w"].astype(np.float64) * direction).sum())
    # the kernel's states are bf16, the oracle's loss is exact: agreement to the storage type's step
    assert abs(mine - fd) < 2e-2 * max(1.0, abs(fd)), (mine, fd)


def test_step_backward_on_a_full_size_block():
    """One compress step at the headline block and cache size (B = M = 512, head_dim 128, width 15) on two
    chains, every gradient against the oracle."""
    w = inputs.Workload(name="bwd512", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, L=512, B=512,
                        M=512, conv_width=15, seed=31, conv_gain=3.0)
    rng = np.random.default_rng(6)
    q, k, v = inputs.qkv(w)
    cw, _ = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    d_o, gk, gv = rng.standard_normal(q.shape), rng.standard_normal(chains), rng.standard_normal(chains)
    want = orc.step_backward(q, k, v, ck, cv, w.M, cw, None, d_o, gk, gv, M=w.M)
    cfg = lb.config_for(w, impl=0)
    dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
    got = _gpu_step_backward(w, cfg, q, k, v, cw, None, ck, cv, w.M, d_o, gk, gv, dW, None)
    got["d_conv_w"] = dW.cpu().numpy()
    for n in ("dq", "dk", "dv", "d_cache_k", "d_cache_v", "d_conv_w"):
        assert _rel(got[n], want[n]) < 2e-4, (n, _rel(got[n], want[n]))


def test_sequence_backward_refusals():
    w = inputs.Workload(name="bwdseq_bad", dtype="f32", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=16, L=32, B=8, M=8,
                        conv_width=3)
    cfg = lb.config_for(w, impl=1)
    q, k, v = (t.cuda() for t in inputs.qkv(w))
    cw, _ = inputs.conv_filters(w)
    cache = lb.Cache(cfg, "cuda")
    z = lambda *s: torch.zeros(s, device="cuda")
    g = dict(d_o=z(*q.shape), dq=z(*q.shape), dk=z(*k.shape), dv=z(*k.shape), ck=z(1, 1, 8, 16), cv=z(1, 1, 8, 16),
             dW=z(*cw.shape))
    need = lb.lococo_sequence_backward_workspace_bytes(cfg, w.L, w.B)
    small = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
    with pytest.raises(lb.LococoError) as e:
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, cw.cuda(), None, cache, g["d_o"], None, None, g["dq"], g["dk"],
                                    g["dv"], g["ck"], g["cv"], g["dW"], None, small)
    assert e.value.status == lb.LOCOCO_EWORKSPACE
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    with pytest.raises(lb.LococoError) as e:                 # the scan compresses: filters are needed
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, None, None, cache, g["d_o"], None, None, g["dq"], g["dk"],
                                    g["dv"], g["ck"], g["cv"], g["dW"], None, ws)
    assert e.value.status == lb.LOCOCO_EINVAL
    cfg2 = lb.config_for(w.replace(norm=2), impl=1)
    with pytest.raises(lb.LococoError) as e:
        lb.lococo_sequence_backward(cfg2, q, k, v, w.B, cw.cuda(), None, cache, g["d_o"], None, None, g["dq"], g["dk"],
                                    g["dv"], g["ck"], g["cv"], g["dW"], None, ws)
    assert e.value.status == lb.LOCOCO_EUNSUPPORTED


@pytest.mark.parametrize("case", [
    dict(L=1, B=1, M=32, len0=32),                                               # one row, one tile
    dict(L=33, B=33, M=64, len0=0, n_q_heads=6, n_kv_heads=2),                   # no cache rows
    dict(L=129, B=129, M=96, len0=1),                                            # a row past the query tile, one cache row
    dict(L=190, B=65, M=63, len0=63, n_q_heads=4, n_kv_heads=1),                 # a cache tile one row short, ragged tail
    dict(L=40 * 64 - 7, B=64, M=512, len0=0, batch=2, n_q_heads=64, n_kv_heads=64),   # more blocks than one window of the walk holds
], ids=str)
def test_scan_backward_on_the_matrix_cores_against_fp32_arithmetic(case):
    """impl = AUTO against the fp32 vector kernels (impl = GENERIC) from the same bf16 inputs.  The operands that enter a
    matrix product as two bf16 halves keep 16 bits, and the two paths' recomputed states may differ by a bf16 step in an
    entry: 2e-3 per tensor, as in the scans against the oracle above."""
    c = dict(case)
    len0 = c.pop("len0")
    w = inputs.Workload(**{**dict(name="bwdvs", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, conv_width=15,
                                  seed=9, conv_gain=2.0), **c})
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(4)
    rnd = lambda *s, dt=torch.float32, sd=1.0: torch.empty(s, dtype=dt, device=dev).normal_(0, sd, generator=g)
    bf = torch.bfloat16
    q = rnd(w.batch, w.n_q_heads, w.L, 128, dt=bf, sd=0.3)
    k, v = (rnd(w.batch, w.n_kv_heads, w.L, 128, dt=bf, sd=0.3) for _ in range(2))
    cw = rnd(w.M, 128, w.conv_width, dt=bf, sd=0.05)
    state = (w.batch, w.n_kv_heads, w.M, 128)
    ck, cv = rnd(*state, dt=bf, sd=0.3), rnd(*state, dt=bf, sd=0.3)
    d_o, d_fk, d_fv = rnd(*q.shape), rnd(*state), rnd(*state)
    out = []
    for impl in (0, 1):
        cfg = lb.config_for(w, impl=impl)
        cache = lb.Cache(cfg, dev)
        cache.load(ck, cv, len0)
        r = [torch.full(s, float("nan"), device=dev) for s in (q.shape, k.shape, k.shape, state, state)]
        dW = torch.zeros(cw.shape, device=dev)
        ws = torch.empty(lb.lococo_sequence_backward_workspace_bytes(cfg, w.L, w.B), dtype=torch.uint8, device=dev)
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, cw, None, cache, d_o, d_fk, d_fv, *r, dW, None, ws)
        torch.cuda.synchronize()
        out.append(r + [dW])
    for name, x, y in zip(("dq", "dk", "dv", "d_cache0_k", "d_cache0_v", "d_conv_w"), *out):
        assert torch.isfinite(x).all(), name
        err = float((x.double() - y.double()).norm() / y.double().norm().clamp_min(1e-30))
        print(name, f"{err:.1e}")
        assert err < 2e-3, (name, err)


@pytest.mark.parametrize("case", [
    dict(B=128, M=128, conv_width=31),                                           # T = 256: one tile of positions a wave
    dict(B=129, M=128, conv_width=1, norm=1),                                    # 257: two
    dict(B=256, M=256, conv_width=5, conv_in=1),                                 # 512
    dict(B=257, M=256, conv_width=15, n_kv_heads=1),                             # 513: four
    dict(B=512, M=513, conv_width=3),                                            # 1025: the positions are walked twice
    dict(B=1030, M=1020, conv_width=3, norm=1),                                  # 2050, slots that are no multiple of 32
], ids=str)
def test_step_backward_at_the_edges_of_the_row_kernel(case):
    """One compress step, the matrix cores (impl = AUTO) against the fp32 vector kernels (impl = GENERIC) on the same
    inputs, at the numbers of positions where the kernel that holds a row in registers changes its form.  Both sides see
    the same operands; what enters a product as two bf16 halves keeps 16 bits: the 2e-4 of the sweep above."""
    w = inputs.Workload(**{**dict(name="bwdrows", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, L=case["B"],
                                  seed=41, conv_gain=3.0), **case})
    rng = np.random.default_rng(12)
    q, k, v = inputs.qkv(w)
    cw, _ = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    d_o, gk, gv = rng.standard_normal(q.shape), rng.standard_normal(chains), rng.standard_normal(chains)
    out = []
    for impl in (0, 1):
        dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
        r = _gpu_step_backward(w, lb.config_for(w, impl=impl), q, k, v, cw, None, ck, cv, w.M, d_o, gk, gv, dW, None)
        out.append({**r, "d_conv_w": dW.cpu().numpy()})
    for n in out[0]:
        assert np.isfinite(out[0][n]).all(), n
        assert _rel(out[0][n], out[1][n]) < 2e-4, (n, _rel(out[0][n], out[1][n]))


@pytest.mark.parametrize("case", [
    dict(B=512, M=1024, protected=512),                    # the first 512 of 1536 positions: the first of three chunks
    dict(B=130, M=1024, protected=1023),                   # 1154 positions, three parts: one entry left in the first two chunks
    dict(B=128, M=1024, protected=1000, norm=1),           # a rectified sum has no reference
], ids=str)
def test_step_backward_with_a_chunk_of_protected_slots(case):
    """More positions than the row kernel holds at once are walked in chunks of 512; one whose positions are all protected
    has no logit to refer the others to.  Against the fp32 vector kernels, with the bound of the test above."""
    c = dict(case)
    n = c.pop("protected")
    w = inputs.Workload(name="bwdprot", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=1, head_dim=128, L=c["B"], seed=43,
                        conv_gain=3.0, conv_width=3, **c)
    rng = np.random.default_rng(13)
    q, k, v = inputs.qkv(w)
    cw, _ = inputs.conv_filters(w)
    chains = (w.batch, w.n_kv_heads, w.M, w.head_dim)
    ck = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    cv = torch.as_tensor(rng.standard_normal(chains) * 0.5).to(w.torch_dtype)
    d_o, gk, gv = rng.standard_normal(q.shape), rng.standard_normal(chains), rng.standard_normal(chains)
    protect = np.broadcast_to(np.arange(w.M) < n, chains[:3]).copy()
    out = []
    for impl in (0, 1):
        dW = torch.zeros(cw.shape, dtype=torch.float32, device="cuda")
        r = _gpu_step_backward(w, lb.config_for(w, impl=impl), q, k, v, cw, None, ck, cv, w.M, d_o, gk, gv, dW, None, protect)
        out.append({**r, "d_conv_w": dW.cpu().numpy()})
    for name in out[0]:
        assert np.isfinite(out[0][name]).all(), name
        if not out[1][name].any():                         # (filters of slots that are all protected)
            assert not out[0][name].any(), name
        else:
            assert _rel(out[0][name], out[1][name]) < 2e-4, (name, _rel(out[0][name], out[1][name]))


def _off_by_one_float(x):
    """A copy of x that starts one float past a 16-byte boundary, and the buffer around it (NaN outside)."""
    room = torch.full((x.numel() + 8,), float("nan"), device=x.device)
    view = room[1:1 + x.numel()].view(x.shape)
    view.copy_(x)
    assert view.data_ptr() % 16 == 4
    return view, room


def _backward_of(w, entry, impl, off, len0=None):
    """All gradients of one step (entry = "step") or scan with seeded inputs; `off`: every gradient array off by a float."""
    dev, bf = "cuda", w.torch_dtype
    g = torch.Generator(device=dev).manual_seed(6)
    rnd = lambda *s, dt=torch.float32, sd=1.0: torch.empty(s, dtype=dt, device=dev).normal_(0, sd, generator=g)
    d = w.head_dim
    q = rnd(w.batch, w.n_q_heads, w.L, d, dt=bf, sd=0.3)
    k, v = (rnd(w.batch, w.n_kv_heads, w.L, d, dt=bf, sd=0.3) for _ in range(2))
    cw = rnd(w.M, d, w.conv_width, dt=bf, sd=0.05)
    state = (w.batch, w.n_kv_heads, w.M, d)
    cfg = lb.config_for(w, impl=impl)
    cache = lb.Cache(cfg, dev)
    cache.load(rnd(*state, dt=bf, sd=0.3), rnd(*state, dt=bf, sd=0.3), w.M if len0 is None else len0)
    rooms = []
    def place(x):
        if not off:
            return x
        view, room = _off_by_one_float(x)
        rooms.append((room, x.numel()))
        return view
    up = [place(rnd(*s)) for s in (q.shape, state, state)]
    out = [place(torch.full(s, float("nan"), device=dev)) for s in (q.shape, k.shape, k.shape, state, state)]
    dW = place(torch.zeros(cw.shape, device=dev))
    if entry == "step":
        ws = torch.empty(lb.lococo_backward_workspace_bytes(cfg, w.L, cache.len), dtype=torch.uint8, device=dev)
        lb.lococo_segment_step_backward(cfg, q, k, v, cw, None, cache, *up, *out, dW, None, ws)
    else:
        ws = torch.empty(lb.lococo_sequence_backward_workspace_bytes(cfg, w.L, w.B), dtype=torch.uint8, device=dev)
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, cw, None, cache, *up, *out, dW, None, ws)
    torch.cuda.synchronize()
    for room, n in rooms:                                  # nothing was written around the arrays
        assert torch.isnan(room[0]) and torch.isnan(room[n + 1:]).all()
    return dict(zip(("dq", "dk", "dv", "d_cache_k", "d_cache_v", "d_conv_w"), out + [dW]))


def _norm_err(x, y):
    return float((x.double() - y.double()).norm() / y.double().norm().clamp_min(1e-30))


@pytest.mark.parametrize("case", [
    dict(entry="step", B=72, M=64, L=72),
    dict(entry="step", B=70, M=160, L=70, n_q_heads=4),
    dict(entry="scan", B=64, M=64, L=200),
    dict(entry="step", B=72, M=64, L=72, head_dim=64),     # the plain contractions and the vector kernels
    dict(entry="scan", B=64, M=64, L=200, head_dim=64),
], ids=str)
def test_gradients_at_any_float_address(case):
    """Gradient arrays are asked to be contiguous floats, no more: views that start in the middle of sixteen bytes, against
    the fp32 vector kernels with aligned ones."""
    c = dict(case)
    entry = c.pop("entry")
    w = inputs.Workload(**{**dict(name="bwdoff", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, conv_width=15,
                                  seed=1), **c})
    got, want = _backward_of(w, entry, 0, True), _backward_of(w, entry, 1, False)
    for n in want:
        assert _norm_err(got[n], want[n]) < (2e-4 if entry == "step" else 2e-3), (n, _norm_err(got[n], want[n]))


@pytest.mark.parametrize("case", [
    dict(B=70, M=64),                                      # a number of positions that is no multiple of 4
    dict(B=511, M=512),
    dict(B=255, M=1024, conv_width=5, norm=1),             # walked in chunks by the row kernel
    dict(B=72, M=64, off=True),                            # gradients that are not 16-byte aligned
    dict(B=512, M=512, off=True, n_kv_heads=1),
    dict(B=256, M=1024, off=True, conv_width=5),
], ids=str)
def test_steps_whose_operands_enter_in_three_parts(case):
    """Steps the fp32 vector kernels used to take keep all 24 bits of what enters a matrix product: against those kernels on
    the same inputs, 2-norms.  dq and dv carry sums of up to 1e3 fp32 products only (measured: at most 8e-7; 3.5e-6 with 16 bits
    kept, 1.8e-6 without the third parts' products alone).  dk and the filter gradient also carry the gradient of the logits,
    which has always entered in two halves: a rounding of 2^-17, uniform, is 2.2e-6 in the 2-norm (measured: 2.2e-6 and 2.6e-6;
    2.8e-6 and 3.1e-6 at least with a third part of anything else left out)."""
    c = dict(case)
    off = c.pop("off", False)
    w = inputs.Workload(**{**dict(name="bwd24", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, conv_width=15,
                                  L=c["B"], seed=1), **c})
    got, want = _backward_of(w, "step", 0, off), _backward_of(w, "step", 1, False)
    bound = dict(dq=1.5e-6, dv=1.5e-6, d_cache_v=1.5e-6, dk=2.8e-6, d_cache_k=2.8e-6, d_conv_w=3.0e-6)
    errs = {n: _norm_err(got[n], want[n]) for n in want}
    print({n: f"{e:.1e}" for n, e in errs.items()})
    for n in want:
        assert errs[n] < bound[n], (n, errs[n])


@pytest.mark.parametrize("case", [
    dict(dtype="f32", head_dim=32, L=77, B=12, M=30, conv_width=5, len0=0),
    dict(dtype="f32", head_dim=32, L=12, B=12, M=16, conv_width=5, len0=16),       # one block: it is the last and the first
    dict(dtype="bf16", head_dim=64, L=96, B=32, M=48, conv_width=5, len0=40),      # the plain contractions
    dict(dtype="bf16", head_dim=128, L=200, B=64, M=64, conv_width=15, len0=64),
    dict(dtype="bf16", head_dim=128, L=64, B=64, M=64, conv_width=15, len0=64),
], ids=str)
def test_scan_backward_in_place(case):
    """d_q may be the array d_o came in, and d_cache0_k / v those of d_final_k / v: same results as with arrays apart."""
    c = dict(case)
    len0 = c.pop("len0")
    w = inputs.Workload(**{**dict(name="inplace", batch=2, n_q_heads=2, n_kv_heads=2, seed=3), **c})
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(2)
    rnd = lambda *s, dt=w.torch_dtype: torch.empty(s, dtype=dt, device=dev).normal_(0, 0.3, generator=g)
    d, state = w.head_dim, (w.batch, w.n_kv_heads, w.M, w.head_dim)
    q, k, v = rnd(w.batch, w.n_q_heads, w.L, d), rnd(w.batch, w.n_kv_heads, w.L, d), rnd(w.batch, w.n_kv_heads, w.L, d)
    cw, ck, cv = rnd(w.M, d, w.conv_width), rnd(*state), rnd(*state)
    d_o, d_fk, d_fv = (rnd(*s, dt=torch.float32) for s in (q.shape, state, state))
    cfg = lb.config_for(w)
    cache = lb.Cache(cfg, dev)
    cache.load(ck, cv, len0)
    ws = torch.empty(lb.lococo_sequence_backward_workspace_bytes(cfg, w.L, w.B), dtype=torch.uint8, device=dev)
    out = []
    for same in (False, True):
        up = [t.clone() for t in (d_o, d_fk, d_fv)]
        dq, dck, dcv = up if same else [torch.full_like(t, float("nan")) for t in up]
        dk, dv = torch.full(k.shape, float("nan"), device=dev), torch.full(k.shape, float("nan"), device=dev)
        dW = torch.zeros(cw.shape, device=dev)
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, cw, None, cache, *up, dq, dk, dv, dck, dcv, dW, None, ws)
        torch.cuda.synchronize()
        out.append(dict(dq=dq, dk=dk, dv=dv, d_cache0_k=dck, d_cache0_v=dcv, d_conv_w=dW))
    for n in out[0]:
        if n == "d_conv_w":                      # (atomic sums)
            assert _norm_err(out[1][n], out[0][n]) < 1e-5, n
        else:
            assert torch.equal(out[1][n], out[0][n]), (n, _norm_err(out[1][n], out[0][n]))


@pytest.mark.parametrize("case", [
    dict(L=10 * 64 + 30, B=64, M=64, len0=0),                                # a fill block, compress blocks, a ragged one
    dict(L=600, B=24, M=96, len0=50, batch=2, n_q_heads=4, conv_width=21, conv_in=1, norm=1),
], ids=str)
def test_scan_backward_takes_a_smaller_workspace(case):
    """As many blocks to a window as the workspace holds, down to one: the same gradients up to the order of the sums over
    blocks; less than that is refused."""
    c = dict(case)
    len0 = c.pop("len0")
    w = inputs.Workload(**{**dict(name="smaller", dtype="bf16", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, conv_width=15,
                                  seed=8), **c})
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(5)
    rnd = lambda *s, dt=torch.bfloat16, sd=0.3: torch.empty(s, dtype=dt, device=dev).normal_(0, sd, generator=g)
    state = (w.batch, w.n_kv_heads, w.M, 128)
    q, k, v = rnd(w.batch, w.n_q_heads, w.L, 128), rnd(w.batch, w.n_kv_heads, w.L, 128), rnd(w.batch, w.n_kv_heads, w.L, 128)
    cw, ck, cv = rnd(w.M, 256 if w.conv_in else 128, w.conv_width, sd=0.05), rnd(*state), rnd(*state)
    up = [rnd(*s, dt=torch.float32) for s in (q.shape, state, state)]
    cfg = lb.config_for(w)
    cache = lb.Cache(cfg, dev)
    cache.load(ck, cv, len0)

    def run(n_bytes):
        out = [torch.full(s, float("nan"), device=dev) for s in (q.shape, k.shape, k.shape, state, state)]
        dW = torch.zeros(cw.shape, device=dev)
        room = torch.full((n_bytes + 4096,), 77, dtype=torch.uint8, device=dev)
        lb.lococo_sequence_backward(cfg, q, k, v, w.B, cw, None, cache, *up, *out, dW, None, room[:n_bytes])
        torch.cuda.synchronize()
        assert (room[n_bytes:] == 77).all()                # nothing past the workspace
        return out + [dW]

    full = lb.lococo_sequence_backward_workspace_bytes(cfg, w.L, w.B)
    with pytest.raises(lb.LococoError, match="workspace needs") as e:
        run(256)
    assert e.value.status == lb.LOCOCO_EWORKSPACE
    least = int(str(e.value).split("workspace needs ")[1].split()[0])
    assert least < full / 3
    with pytest.raises(lb.LococoError):
        run(least - 256)
    want = run(full)
    for n_bytes in (full - 256, (full + 2 * least) // 3 // 256 * 256, least):
        for name, x, y in zip(("dq", "dk", "dv", "d_cache0_k", "d_cache0_v", "d_conv_w"), run(n_bytes), want):
            assert _norm_err(x, y) < 1e-5, (n_bytes, name, _norm_err(x, y))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("B", [100, 200])
def test_a_bad_token_stays_out_of_what_does_not_see_it(B, bad):
    """A fill step (no compression, which mixes everything) with one entry of a query, or of a value row, that is no number:
    the gradients of keys and values behind the query's token, and of queries before the value's, do not depend on it."""
    w = inputs.Workload(name="bad", dtype="bf16", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, L=B, B=B, M=256, conv_width=15)
    dev, r0, col, m = "cuda", 41, 7, 37
    g = torch.Generator(device=dev).manual_seed(9)
    rnd = lambda *s, dt=torch.float32: torch.empty(s, dtype=dt, device=dev).normal_(0, 0.5, generator=g)
    state = (1, 2, w.M, 128)
    cw, ck, cv = (rnd(*s, dt=torch.bfloat16) for s in ((w.M, 128, 15), state, state))
    up = [rnd(*s) for s in ((1, 4, B, 128), state, state)]
    for which in ("q", "v"):
        for impl in (0, 1):
            q, k, v = (rnd(1, h, B, 128, dt=torch.bfloat16) for h in (4, 2, 2))
            (q if which == "q" else v)[0, 1, r0, col] = bad
            cfg = lb.config_for(w, impl=impl)
            cache = lb.Cache(cfg, dev)
            cache.load(ck, cv, m)
            dq, dk, dv = (torch.full(t.shape, float("nan"), device=dev) for t in (q, k, v))
            dck, dcv = torch.empty(state, device=dev), torch.empty(state, device=dev)
            ws = torch.empty(lb.lococo_backward_workspace_bytes(cfg, B, m), dtype=torch.uint8, device=dev)
            lb.lococo_segment_step_backward(cfg, q, k, v, cw, None, cache, *up, dq, dk, dv, dck, dcv,
                                            torch.zeros(cw.shape, device=dev), None, ws)
            torch.cuda.synchronize()
            if which == "q":                     # head 1 reads the keys of kv head 0; 0 x bad in its own column
                others = torch.arange(128, device=dev) != col
                assert torch.isfinite(dk[0, 0, r0 + 1:][:, others]).all() and torch.isfinite(dk[0, 1]).all(), impl
                assert torch.isfinite(dv[0, :, r0 + 1:]).all() and torch.isfinite(dv[0, 1]).all(), impl
                assert torch.isfinite(dq[0, [0, 2, 3]]).all() and torch.isfinite(dq[0, 1, torch.arange(B) != r0]).all(), impl
            else:                                # the values of kv head 1 are those of heads 2 and 3
                assert torch.isfinite(dq[0, :2]).all() and torch.isfinite(dq[0, 2:, :r0]).all(), impl
                assert torch.isfinite(dv).all(), impl
