"""The backward walk over the blocks of a window in one launch, against the same walk with two launches a block (the two differ in
the order of their sums alone): slot tiles of every number it takes, odd ones whose last pair of row tiles is half empty, blocks
in two and in three parts, first blocks with fewer live slots, its meetings, and what it does where it cannot have the device.
How many walks a call launched is read from its timing rows, and asserted."""
import itertools

import pytest
import torch

from paper_2406_05317_amd import binding as lb

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture
def options():
    yield lb.lococo_debug_option
    lb.lococo_debug_option(lb.LOCOCO_OPT_RESET, 0)


def rnd(g, *shape, sd=0.3, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0, sd, generator=g)


class Scan:
    def __init__(self, M, B, L, batch=1, heads=2, kv=2, width=15, len0=0, per_head=False, seed=3):
        g = torch.Generator(device=DEV).manual_seed(seed)
        self.cfg = lb.make_config(dtype=torch.bfloat16, batch=batch, n_q_heads=heads, n_kv_heads=kv, head_dim=128, M=M, conv_width=width,
                                  **({"w_head_stride": M * 128 * width} if per_head else {}))
        self.B, self.L = B, L
        self.q, self.k, self.v = rnd(g, batch, heads, L, 128), rnd(g, batch, kv, L, 128), rnd(g, batch, kv, L, 128)
        self.w = rnd(g, *([kv] if per_head else []), M, 128, width, sd=0.05)
        self.cache = lb.Cache(self.cfg, DEV)
        if len0:
            self.cache.load(rnd(g, batch, kv, M, 128), rnd(g, batch, kv, M, 128), len0)
        f32 = dict(dtype=torch.float32)
        self.d_o = rnd(g, *self.q.shape, sd=1.0, **f32)
        self.state = (batch, kv, M, 128)
        self.d_f = [rnd(g, *self.state, sd=1.0, **f32) for _ in range(2)]
        self.ws = torch.full((lb.lococo_sequence_backward_workspace_bytes(self.cfg, L, B),), 0xff, dtype=torch.uint8, device=DEV)
        self.out = [torch.empty(s, device=DEV, **f32) for s in (self.q.shape, self.k.shape, self.k.shape, self.state, self.state)]
        self.d_w = torch.zeros(self.w.shape, device=DEV, **f32)

    def enqueue(self):
        self.d_w.zero_()
        lb.lococo_sequence_backward(self.cfg, self.q, self.k, self.v, self.B, self.w, None, self.cache, self.d_o, *self.d_f, *self.out,
                                    self.d_w, None, self.ws)

    def run(self):
        for t in self.out:
            t.fill_(float("nan"))
        lb.lococo_timing_begin()
        self.enqueue()
        self.walks = lb.lococo_timing_end().get("bwd_walk", (0, 0.0))[0]
        torch.cuda.synchronize()
        return [t.clone() for t in (*self.out, self.d_w)]

    def runs(self):
        """Walks the call takes: runs of compressing blocks of one form (three parts: positions no multiple of 4), of at least 6, or of
        4 in three parts or on 64 slots and fewer."""
        forms = [(before + n) % 4 != 0 for _, n, branch, before, _, _ in lb.lococo_plan(self.L, self.B, self.cfg.M, self.cache.len) if branch]
        return sum(len(list(run)) >= (4 if three or self.cfg.M <= 64 else 6) for three, run in itertools.groupby(forms))

    def status(self):
        return lb.lococo_scan_status(self.cfg, self.ws)


def close(got, want):
    """g and dl keep 16 bits where they enter a product: where the fp32 sums differ in their last bit, two values rounded to either
    side differ by 2^-16 at most."""
    for name, a, b in zip(("d_q", "d_k", "d_v", "d_cache_k", "d_cache_v", "d_w"), got, want):
        assert torch.isfinite(a).all(), name
        err = float((a.double() - b.double()).norm() / b.double().norm().clamp_min(1e-30))
        assert err < 2.0 ** -16, (name, err)


CASES = [
    dict(M=32, B=32, L=170),                                                  # one slot tile: half a pair of row tiles
    dict(M=64, B=33, L=300, kv=3, heads=6),                                   # three parts, chains not all on one XCD
    dict(M=96, B=96, L=692, width=21),                                        # an odd number of tiles
    dict(M=128, B=128, L=956, kv=32, heads=32),                               # every compute unit
    dict(M=128, B=128, L=906, len0=70),                                       # a first block that finds 70 live slots
    dict(M=128, B=101, L=500, len0=128, width=21, per_head=True),             # three parts, banks of their own
    dict(M=160, B=97, L=600, kv=8, heads=8),                                  # 257 positions: two tiles a wave, one round of five
    dict(M=192, B=191, L=1091, batch=2),                                       # three parts, two rounds of three
    dict(M=224, B=224, L=1448, kv=4, heads=8),                                # one round of seven, a half-empty pair
    dict(M=256, B=256, L=1913, kv=8, heads=8, batch=2),                       # the largest; the last block in parts of its own
    dict(M=256, B=255, L=1300, len0=3, width=21),                             # three parts, three live slots
    dict(M=96, B=20, L=330, kv=4, heads=4),                                   # four fill blocks in the filters' launch
    dict(M=64, B=200, L=900),                                                 # blocks longer than the cache, an empty first state
    dict(M=128, B=100, L=700, len0=128),                                      # six blocks and a seventh
    dict(M=64, B=33, L=132, len0=64),                                         # four in three parts: the fewest
    dict(M=96, B=96, L=576, len0=96),                                         # six in two
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_one_launch_against_two_a_block(case, options):
    s = Scan(**case)
    got = s.run()
    assert s.status() == 0 and s.walks == s.runs() > 0
    options(lb.LOCOCO_OPT_SCAN_PER_STEP, 1)
    close(got, s.run())
    assert s.walks == 0


@pytest.mark.parametrize("case", [dict(M=96, B=96, L=480, len0=96), dict(M=64, B=33, L=99, len0=64), dict(M=128, B=128, L=256, len0=128)], ids=str)
def test_few_blocks_are_walked_one_by_one(case):
    s = Scan(**case)
    s.run()
    assert s.walks == s.runs() == 0 and s.status() == 0


def test_windows_of_a_smaller_workspace(options):
    """Counters cleared again for every window; windows too short for the walk."""
    s = Scan(M=64, B=64, L=64 * 31)
    want, whole = s.run(), s.ws
    walks = []
    for part in (0.6, 0.4, 0.25):
        s.ws = torch.full((int(part * whole.numel()),), 0xff, dtype=torch.uint8, device=DEV)
        close(s.run(), want)
        assert s.status() == 0
        walks.append(s.walks)
    assert walks[0] > 1 and walks[-1] != walks[0], walks


def test_meetings_with_device_scope(options):
    s = Scan(M=96, B=80, L=660, kv=8, heads=8)
    got = s.run()
    assert s.walks == s.runs() > 0
    options(lb.LOCOCO_OPT_CHAIN_SYNC_DEVICE, 1)
    again = s.run()
    assert s.status() == 0 and s.walks == s.runs()
    for a, b in zip(got[:5], again[:5]):
        assert torch.equal(a, b)


def test_a_wait_that_gives_up_is_reported(options):
    s = Scan(M=128, B=128, L=956)
    want = s.run()
    options(lb.LOCOCO_OPT_SPIN_LIMIT, -1)
    s.run()
    assert s.status() == 1
    options(lb.LOCOCO_OPT_SPIN_LIMIT, 0)
    close(s.run(), want)
    assert s.status() == 0


def test_the_walk_reports_a_wait_of_its_own(options):
    """The recomputed scan in launches per step, which wait for nobody: what is in the status word is the walk's."""
    s = Scan(M=128, B=128, L=956)
    options(lb.LOCOCO_OPT_SCAN_PER_STEP, 2)
    want = s.run()
    assert s.walks == s.runs() > 0 and s.status() == 0
    options(lb.LOCOCO_OPT_SPIN_LIMIT, -1)
    s.run()
    assert s.walks > 0 and s.status() == 1
    options(lb.LOCOCO_OPT_SCAN_PER_STEP, 1)                                   # (nobody waits: the word is cleared and stays so)
    close(s.run(), want)
    assert s.walks == 0 and s.status() == 0


def test_gradients_of_the_last_state_that_are_4_byte_aligned_only():
    s = Scan(M=96, B=80, L=660, kv=8, heads=8)
    want = s.run()
    s.d_f = [torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape) for t in s.d_f]
    assert all(t.data_ptr() % 16 for t in s.d_f)
    got = s.run()
    assert s.walks == s.runs() > 0
    for a, b in zip(got[:5], want[:5]):
        assert torch.equal(a, b)


def test_two_launches_a_block_where_the_grid_would_not_be_resident(options):
    s = Scan(M=128, B=128, L=956, kv=4, heads=4)
    want = s.run()
    assert s.walks == s.runs() > 0
    options(lb.LOCOCO_OPT_MAX_RESIDENT, 15)                                   # four workgroups a chain and pair of tiles: 32
    close(s.run(), want)
    assert s.status() == 0 and s.walks == 0


def test_two_streams_and_a_captured_graph():
    s, t = Scan(M=128, B=100, L=800, kv=8, heads=8), Scan(M=128, B=100, L=800, kv=8, heads=8, seed=9)
    want = [x.run() for x in (s, t)]
    assert s.walks == t.walks == s.runs() > 0
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(3):
        for x, st in zip((s, t), streams):
            st.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(st):
                x.enqueue()
        torch.cuda.synchronize()
        for x, w in zip((s, t), want):
            close([*x.out, x.d_w], w)
            assert x.status() == 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s.enqueue()
    for i in range(4):
        for o in s.out:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        close([*s.out, s.d_w], want[0])
        t.run()                                                               # work of its own between the replays
