"""The backward kernels of Eq. 4 - 6 at the edges of their tiles, and the logits a recomputed scan leaves behind."""
import pytest
import torch

from paper_2406_05317_amd import binding as lb
from paper_2406_05317_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rnd(g, *shape, sd=0.3, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0, sd, generator=g)


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm().clamp_min(1e-30))


@pytest.mark.parametrize("case", [
    # (chains x row tiles decide the tile: 128, 64, 32 rows, and 32 rows in halves)
    dict(batch=2, n_kv_heads=32, M=256, B=256),                                    # 128 rows, whole
    dict(batch=2, n_kv_heads=32, M=253, B=254),                                    # 128 rows in three parts (507 positions)
    dict(batch=2, n_kv_heads=32, M=100, B=100, conv_width=5),                      # 64 rows, slots past a chunk, KW % 3 = 2
    dict(batch=2, n_kv_heads=32, M=97, B=101, conv_width=31),                      # the same in three parts, KW % 3 = 1
    dict(batch=2, n_kv_heads=32, M=64, B=36, conv_width=21),                       # 32 rows
    dict(batch=2, n_kv_heads=32, M=33, B=66, conv_width=3),                        # 32 rows in three parts, one slot past a tile
    dict(batch=1, n_kv_heads=2, M=129, B=1),                                       # halves, a token
    dict(batch=1, n_kv_heads=3, M=160, B=77, conv_width=7, per_head=True),         # halves in three parts, banks of their own
    dict(batch=1, n_kv_heads=2, M=130, B=62, conv_in=1, conv_width=21),            # [K | V] filters: taps on both halves
    dict(batch=2, n_kv_heads=32, M=128, B=384, conv_in=1),                         # the same with 128 rows
    dict(batch=1, n_kv_heads=2, M=16, B=8, conv_width=1),                          # the smallest: sixteen slots, one tap
    # (32 rows in halves: the slots in four parts up to 64 of them, in eight above with so few workgroups; whole: always in four)
    dict(batch=1, n_kv_heads=2, M=64, B=1, conv_width=5),                          # halves in three parts, four parts of slots
    dict(batch=1, n_kv_heads=3, M=64, B=60, conv_in=1, conv_width=31),             # halves
    dict(batch=2, n_kv_heads=32, M=49, B=63, conv_width=15),                       # whole, a slot past 48
    dict(batch=1, n_kv_heads=2, M=65, B=7, conv_width=21),                         # halves, the first with eight parts
], ids=str)
def test_input_and_filter_gradients_at_tile_edges(case):
    """Against the shape-agnostic fp32 kernels, which agree with the oracle to 3e-7.  g, n and dl keep 16 bits where they enter
    a product: at most three such roundings of 2^-17 each on any path, 2.3e-5."""
    c = dict(dict(conv_width=15, conv_in=0, per_head=False), **case)
    g = torch.Generator(device=DEV).manual_seed(5)
    b, h, M, B, kw = c["batch"], c["n_kv_heads"], c["M"], c["B"], c["conv_width"]
    C = 256 if c["conv_in"] else 128
    q, k, v = (_rnd(g, b, h, B, 128) for _ in range(3))
    ck, cv = _rnd(g, b, h, M, 128), _rnd(g, b, h, M, 128)
    cw = _rnd(g, *([h] if c["per_head"] else []), M, C, kw, sd=0.05)
    d_o, gk, gv = (_rnd(g, *s, sd=1.0, dtype=torch.float32) for s in (q.shape, ck.shape, ck.shape))
    got = []
    for impl in (lb.LOCOCO_IMPL_AUTO, lb.LOCOCO_IMPL_GENERIC):
        cfg = lb.make_config(dtype=torch.bfloat16, batch=b, n_q_heads=h, n_kv_heads=h, head_dim=128, M=M, conv_width=kw,
                             conv_in=c["conv_in"], impl=impl, **({"w_head_stride": M * C * kw} if c["per_head"] else {}))
        cache = lb.Cache(cfg, DEV)
        cache.load(ck, cv, M)
        out = [torch.full_like(t, float("nan"), dtype=torch.float32) for t in (q, k, v, ck, cv)]
        d_w = torch.zeros_like(cw, dtype=torch.float32)
        ws = torch.full((lb.lococo_backward_workspace_bytes(cfg, B, M),), 0xff, dtype=torch.uint8, device=DEV)
        lb.lococo_segment_step_backward(cfg, q, k, v, cw, None, cache, d_o, gk, gv, *out, d_w, None, ws)
        got.append(out + [d_w])
    for name, a, want in zip(("d_q", "d_k", "d_v", "d_cache_k", "d_cache_v", "d_w"), *got):
        assert _rel(a, want) < 2.3e-5, (name, _rel(a, want))


@pytest.mark.parametrize("case", [
    dict(batch=4, n_kv_heads=32, M=64, B=128),                                     # 64 rows: a quarter of two 128-row tiles is padding
    dict(batch=4, n_kv_heads=32, M=65, B=122, conv_width=31),                      # the same in three parts, a row past a tile less
    dict(batch=4, n_kv_heads=32, M=64, B=65, conv_in=1, conv_width=21),            # 129 rows, taps on both halves
    dict(batch=2, n_kv_heads=32, M=160, B=32),                                     # 32 rows whole, four parts of more than 64 slots
    dict(batch=2, n_kv_heads=32, M=129, B=30, conv_width=7),                       # the same in three parts, one slot past a chunk
    dict(batch=1, n_kv_heads=3, M=192, B=64, conv_width=31),                       # halves, eight parts of two chunks
    dict(batch=1, n_kv_heads=2, M=190, B=3, conv_in=1),                            # the same in three parts
    dict(batch=8, n_kv_heads=32, M=32, B=32),                                      # up to 64 rows of 256 chains: one 64-row tile each
    dict(batch=8, n_kv_heads=32, M=33, B=22, conv_width=5),                        # the same in three parts
], ids=str)
def test_gradients_on_the_tiles_that_pad_least(case):
    test_input_and_filter_gradients_at_tile_edges(case)


@pytest.mark.parametrize("case", [
    dict(M=64, B=48, conv_width=15),                                               # 16 chains, 20 blocks
    dict(M=63, B=42, conv_width=7),                                                # the same in three parts
], ids=str)
def test_rows_of_many_short_blocks_at_once(case):
    """The rows of all blocks of a window in one launch, 64-row tiles from 256 chains and blocks on, against windows of one block,
    32-row tiles: the same products, fp32 sums of up to 2e3 terms in another order (3e-7 each at most, uncorrelated)."""
    M, B, kw = case["M"], case["B"], case["conv_width"]
    L, h = M + 20 * B, 16
    g = torch.Generator(device=DEV).manual_seed(17)
    q, k, v = (_rnd(g, 1, h, L, 128) for _ in range(3))
    cw = _rnd(g, M, 128, kw, sd=0.05)
    d_o, gk, gv = (_rnd(g, 1, h, n, 128, sd=1.0, dtype=torch.float32) for n in (L, M, M))
    cfg = lb.make_config(dtype=torch.bfloat16, batch=1, n_q_heads=h, n_kv_heads=h, head_dim=128, M=M, conv_width=kw)
    full = lb.lococo_sequence_backward_workspace_bytes(cfg, L, B)

    def run(n_bytes):
        out = [torch.full_like(t, float("nan"), dtype=torch.float32) for t in (q, k, v, gk, gv)]
        d_w = torch.zeros_like(cw, dtype=torch.float32)
        lb.lococo_sequence_backward(cfg, q, k, v, B, cw, None, lb.Cache(cfg, DEV), d_o, gk, gv, *out, d_w, None,
                                    torch.full((n_bytes,), 0xff, dtype=torch.uint8, device=DEV))
        return out + [d_w]

    with pytest.raises(lb.LococoError, match="workspace needs") as e:
        run(256)
    least = int(str(e.value).split("workspace needs ")[1].split()[0])
    for name, a, want in zip(("d_q", "d_k", "d_v", "d_cache0_k", "d_cache0_v", "d_w"), run(full), run(least)):
        assert _rel(a, want) < 1e-5, (name, _rel(a, want))


@pytest.mark.parametrize("case", [
    # (32 rows in halves; four parts where slots and workgroups are enough)
    dict(batch=1, n_kv_heads=3, M=200, B=40, per_head=True, conv_width=7),         # eight parts, two chunks of slots
    dict(batch=1, n_kv_heads=2, M=253, B=33, conv_in=1, conv_width=21),            # the same in three parts, taps on both halves
    dict(batch=1, n_kv_heads=4, M=320, B=32, conv_width=3),                        # three chunks: too few workgroups for four parts
    dict(batch=1, n_kv_heads=8, M=192, B=64),                                      # four parts
    dict(batch=1, n_kv_heads=8, M=190, B=3, conv_in=1, conv_width=7),              # the same in three parts
    dict(batch=2, n_kv_heads=8, M=320, B=33, conv_width=3),                        # four parts, five chunks, three parts of n and g
    dict(batch=2, n_kv_heads=8, M=448, B=32, conv_width=3),                        # the same in two parts, seven chunks
], ids=str)
def test_gradients_of_launches_in_halves(case):
    test_input_and_filter_gradients_at_tile_edges(case)


@pytest.mark.parametrize("case", [
    # (tiles of 32 rows of all heads of a group; two waves per 32 keys from four of them on where the launch fills no more than the chip)
    dict(kv=2, group=4, M=128, B=16),                      # four heads of a tile each
    dict(kv=1, group=5, M=60, B=20),                       # five: one wave of the two ends a tile earlier
    dict(kv=2, group=1, M=128, B=128),                     # keys of the block see four tiles, three, two, one
    dict(kv=1, group=1, M=128, B=100),                     # a last tile of four rows
    dict(kv=2, group=3, M=32, B=96),                       # nine tiles, all keys in one workgroup
    dict(kv=1, group=2, M=500, B=260),                     # a last workgroup of keys that is mostly empty
    dict(kv=1, group=3, M=96, B=32),                       # three tiles: one wave per 32 keys
    dict(kv=2, group=1, M=128, B=1),                       # three parts, nothing for the second wave
    dict(kv=1, group=5, M=61, B=20),                       # three parts, five tiles
    dict(kv=1, group=3, M=33, B=65),                       # three parts, nine tiles
    dict(kv=96, group=2, M=190, B=129),                    # three parts, more workgroups than compute units: one wave again
    dict(kv=96, group=1, M=191, B=129),                    # the same in two parts
], ids=str)
def test_key_and_value_gradients_by_size_of_the_launch(case):
    """Against the shape-agnostic fp32 kernels.  Two parts: 16 bits kept of dO, P and dS, at most two such roundings of 2^-17 in a
    product: 1.6e-5; three parts: nothing lost, fp32 sums of up to 1300 terms in another order."""
    h, gr, M, B = (case[n] for n in ("kv", "group", "M", "B"))
    g = torch.Generator(device=DEV).manual_seed(13)
    q = _rnd(g, 1, h * gr, B, 128, sd=1.0)
    k, v, ck, cv = (_rnd(g, 1, h, n, 128, sd=1.0) for n in (B, B, M, M))
    cw = _rnd(g, M, 128, 3, sd=0.05)
    d_o = _rnd(g, *q.shape, sd=1.0, dtype=torch.float32)
    no_grad = torch.zeros(ck.shape, device=DEV)            # of the new state: only the attention's part is left
    got = []
    for impl in (lb.LOCOCO_IMPL_AUTO, lb.LOCOCO_IMPL_GENERIC):
        cfg = lb.make_config(dtype=torch.bfloat16, batch=1, n_q_heads=h * gr, n_kv_heads=h, head_dim=128, M=M, conv_width=3, impl=impl)
        cache = lb.Cache(cfg, DEV)
        cache.load(ck, cv, M)
        out = [torch.full_like(t, float("nan"), dtype=torch.float32) for t in (q, k, v, ck, cv)]
        ws = torch.full((lb.lococo_backward_workspace_bytes(cfg, B, M),), 0xff, dtype=torch.uint8, device=DEV)
        lb.lococo_segment_step_backward(cfg, q, k, v, cw, None, cache, d_o, no_grad, no_grad, *out, torch.zeros_like(cw, dtype=torch.float32),
                                        None, ws)
        got.append(out)
    bound = 1.6e-5 if (M + B) % 4 == 0 else 1e-6
    for name, a, want in zip(("d_q", "d_k", "d_v", "d_cache_k", "d_cache_v"), *got):
        assert _rel(a, want) < bound, (name, _rel(a, want))


@pytest.mark.parametrize("case", [
    dict(batch=1, n_kv_heads=2, M=64, B=48, L=300),                                # pairs of workgroups; a fill, a ragged block
    dict(batch=1, n_kv_heads=2, M=96, B=96, L=481, conv_width=21, norm=1, bias=True),   # last block of one token
    dict(batch=2, n_kv_heads=32, M=96, B=64, L=320),                               # a workgroup per chain and 32 slots
    dict(batch=4, n_kv_heads=32, M=96, B=64, L=256, norm=1, bias=True),            # several chains per workgroup
    dict(batch=4, n_kv_heads=32, M=128, B=70, L=333),                              # 64 slots
    dict(batch=8, n_kv_heads=32, M=128, B=128, L=512, norm=1),                     # 64 slots, several chains per workgroup
    dict(batch=1, n_kv_heads=2, M=64, B=64, L=256, protect=True),                  # computed window by window in either case
    dict(batch=1, n_kv_heads=2, M=64, B=64, L=256, conv_in=1),
], ids=str)
def test_logits_left_by_the_scan_are_those_computed_again(case):
    """With one byte less than the full workspace the logits are computed in a kernel of their own: the same products in
    another order (1e-6 of a logit, which moves a softmax weight by as much; under the rectified sum one logit in 1e6 may
    also change sides of zero, which takes its entry in or out)."""
    c = dict(dict(conv_width=15, norm=0, conv_in=0, bias=False, protect=False), **case)
    g = torch.Generator(device=DEV).manual_seed(9)
    b, h, M, B, L, kw = (c[n] for n in ("batch", "n_kv_heads", "M", "B", "L", "conv_width"))
    C = 256 if c["conv_in"] else 128
    cfg = lb.make_config(dtype=torch.bfloat16, batch=b, n_q_heads=h, n_kv_heads=h, head_dim=128, M=M, conv_width=kw,
                         conv_in=c["conv_in"], norm=c["norm"])
    q, k, v = (_rnd(g, b, h, L, 128) for _ in range(3))
    cw = _rnd(g, M, C, kw, sd=0.05)
    cb = _rnd(g, M, sd=0.5) if c["bias"] else None
    d_o = _rnd(g, *q.shape, sd=1.0, dtype=torch.float32)
    gk, gv = (_rnd(g, b, h, M, 128, sd=1.0, dtype=torch.float32) for _ in range(2))
    full = lb.lococo_sequence_backward_workspace_bytes(cfg, L, B)
    got = []
    for n_bytes in (full, full - 1):
        cache = lb.Cache(cfg, DEV)
        if c["protect"]:
            cache.set_protect((torch.arange(M) < 3).view(1, 1, -1).expand(b, h, -1).numpy())
        out = [torch.full_like(t, float("nan"), dtype=torch.float32) for t in (q, k, v, gk, gv)]
        d_w, d_b = torch.zeros_like(cw, dtype=torch.float32), torch.zeros(M, device=DEV) if c["bias"] else None
        ws = torch.full((full,), 0xff, dtype=torch.uint8, device=DEV)[:n_bytes]
        lb.lococo_sequence_backward(cfg, q, k, v, B, cw, cb, cache, d_o, gk, gv, *out, d_w, d_b, ws)
        got.append(out + [d_w] + ([d_b] if c["bias"] else []))
    for a, want in zip(*got):
        assert torch.isfinite(a).all()
        assert _rel(a, want) < (1e-3 if c["norm"] else 1e-5), _rel(a, want)
    # logits that were kept show in the last bits of the gradients (no atomics in these); computed both times, they are the same
    kept = not (c["protect"] or c["conv_in"])
    assert all(torch.equal(a, want) for a, want in zip(got[0][:5], got[1][:5])) != kept


@pytest.mark.parametrize("entry", ["step", "scan"])
@pytest.mark.parametrize("case", [
    dict(M=128, B=128),
    dict(M=96, B=33, conv_width=21, conv_in=1),            # three parts, filters over [K | V]
    dict(M=64, B=64, n_kv_heads=4, per_head=True),
], ids=str)
def test_least_workspace_has_one_place_for_the_filters(entry, case):
    """What a step and a scan of one block did with before the filters were packed in two orders still does: one place for both, a
    launch more, the same gradients.  Nothing is written behind it, and less is refused."""
    c = dict(dict(conv_width=15, conv_in=0, n_kv_heads=2, per_head=False), **case)
    g = torch.Generator(device=DEV).manual_seed(11)
    h, M, B, kw = c["n_kv_heads"], c["M"], c["B"], c["conv_width"]
    C = 256 if c["conv_in"] else 128
    banks = h if c["per_head"] else 1
    q, k, v = (_rnd(g, 1, h, B, 128) for _ in range(3))
    ck, cv = _rnd(g, 1, h, M, 128), _rnd(g, 1, h, M, 128)
    cw = _rnd(g, *([h] if c["per_head"] else []), M, C, kw, sd=0.05)
    d_o, gk, gv = (_rnd(g, *s, sd=1.0, dtype=torch.float32) for s in (q.shape, ck.shape, ck.shape))
    cfg = lb.make_config(dtype=torch.bfloat16, batch=1, n_q_heads=h, n_kv_heads=h, head_dim=128, M=M, conv_width=kw,
                         conv_in=c["conv_in"], **({"w_head_stride": M * C * kw} if c["per_head"] else {}))
    cache = lb.Cache(cfg, DEV)
    cache.load(ck, cv, M)

    def run(n_bytes):
        out = [torch.full_like(t, float("nan"), dtype=torch.float32) for t in (q, k, v, ck, cv)]
        d_w = torch.zeros_like(cw, dtype=torch.float32)
        room = torch.full((n_bytes + 4096,), 0xff, dtype=torch.uint8, device=DEV)
        if entry == "step":
            lb.lococo_segment_step_backward(cfg, q, k, v, cw, None, cache, d_o, gk, gv, *out, d_w, None, room[:n_bytes])
        else:
            lb.lococo_sequence_backward(cfg, q, k, v, B, cw, None, cache, d_o, gk, gv, *out, d_w, None, room[:n_bytes])
        assert (room[n_bytes:] == 0xff).all()
        return out + [d_w]

    up = lambda n: (n + 255) // 256 * 256
    packed = up(banks * kw * M * C * 2)
    full = lb.lococo_backward_workspace_bytes(cfg, B, M) if entry == "step" else lb.lococo_sequence_backward_workspace_bytes(cfg, B, B)
    want, got = run(full), run(full - packed)
    for name, a, b in zip(("d_q", "d_k", "d_v", "d_cache_k", "d_cache_v"), got, want):
        assert torch.equal(a, b), name
    assert _rel(got[5], want[5]) < 1e-6                    # (atomic sums)
    with pytest.raises(lb.LococoError, match=f"workspace needs {full - packed} bytes") as e:
        run(full - packed - 256)
    assert e.value.status == lb.LOCOCO_EWORKSPACE
