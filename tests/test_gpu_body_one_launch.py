"""The draft body's step as one launch (up to 16 rows, heads of 64 or 128): the sizes where its items, pieces and buffers have
edges, against the oracle to the bars of test_gpu_body.py; and that what it keeps between launches (counters, two sets of buffers
in the workspace) survives other uses of the workspace, graph replays, and streams that compete for the compute units."""
import ctypes

import numpy as np
import pytest

from paper_2601_20357_amd import synth
from test_gpu_body import BodyPair, _gpu, _route, _to_dev

pytestmark = pytest.mark.gpu

B = synth.BodyConfig
# rows 1, 2, 3, 5, 8, 9, 16 (lanes, halves and sums of a block of 16 rows); positions around a chunk of 32 keys and a step of 256 (128);
# pieces of 256 keys, up to 8 of shorter ones and 16 of others; the widest of each number of units a wave, and one past it;
# d_ff below a unit of 32, or that ends inside a tile of 16, inside a unit of 32, and in neither; d of one and of several units a wave, above 768 too
SHAPES = [
    ("rows1_hd64", B(layers=2, d=64, heads=1, d_ff=8, V=30, max_ctx=300), [257]),
    ("rows2_hd128", B(layers=2, d=128, heads=1, d_ff=264, V=30, max_ctx=200), [128, 129]),
    ("rows2_d_ff_16", B(layers=2, d=64, heads=1, d_ff=16, V=30, max_ctx=40), [20, 31]),
    ("rows7_d_ff_24", B(layers=1, d=128, heads=2, d_ff=24, V=30, max_ctx=40), list(range(7))),
    ("rows3_hd64", B(layers=1, d=192, heads=3, d_ff=520, V=30, max_ctx=700), [0, 31, 600]),
    ("rows5_hd64", B(layers=2, d=768, heads=12, d_ff=3072, V=30, max_ctx=90), [32, 33, 63, 64, 65]),
    ("rows8_hd128", B(layers=1, d=1024, heads=8, d_ff=4096, V=30, max_ctx=70), [0, 1, 2, 30, 31, 32, 33, 60]),
    ("rows9_hd64", B(layers=1, d=832, heads=13, d_ff=2216, V=30, max_ctx=130), [0, 0, 5, 31, 32, 95, 96, 97, 120]),
    ("rows16_hd64", B(layers=1, d=1024, heads=16, d_ff=2728, V=30, max_ctx=70), list(range(0, 64, 4))),
    ("rows16_hd128", B(layers=1, d=256, heads=2, d_ff=1000, V=30, max_ctx=600), [17 * i for i in range(16)]),
    ("rows4_quarter", B(layers=2, d=256, heads=4, d_ff=1024, V=30, max_ctx=90), [32, 33, 63, 64]),
    ("rows2_past_the_quarter", B(layers=1, d=256, heads=2, d_ff=1032, V=30, max_ctx=90), [0, 64]),
    ("rows3_half", B(layers=1, d=512, heads=8, d_ff=2048, V=30, max_ctx=90), [1, 40, 85]),
    ("rows6_half_hd128", B(layers=2, d=384, heads=3, d_ff=1360, V=30, max_ctx=300), [5, 64, 100, 127, 128, 297]),
    ("rows2_past_the_half_hd128", B(layers=1, d=768, heads=6, d_ff=2056, V=30, max_ctx=90), [31, 60]),
    ("rows1_eight_pieces", B(layers=1, d=64, heads=1, d_ff=64, V=30, max_ctx=2100), [2046]),
    ("rows2_nine_to_sixteen_pieces", B(layers=1, d=128, heads=1, d_ff=64, V=30, max_ctx=4200), [2048, 4094]),
    ("rows1_eight_thousand", B(layers=1, d=64, heads=1, d_ff=64, V=30, max_ctx=8192), [8189]),
]


@pytest.mark.parametrize("name,bc,ctx", SHAPES, ids=[s[0] for s in SHAPES])
def test_one_launch_step_matches_the_oracle(oracle, name, bc, ctx):
    assert _route(_gpu()[1], bc, len(ctx)) == 0
    pair = BodyPair(oracle, bc, len(ctx), seed=len(name), fill=lambda g: ctx)
    g = np.random.default_rng(7)
    for _ in range(2):
        pair.step(g.integers(0, bc.V, size=len(ctx)))


def test_positions_that_change_how_the_attention_is_cut(oracle):
    """Most workgroups have no projection to do here, and with every 32 positions a row's keys are cut into one more piece: a
    workgroup that took the positions of the step after would wait for pieces that nobody computes.  Steps across two such edges."""
    bc = B(layers=1, d=64, heads=1, d_ff=8, V=30, max_ctx=200)
    pair = BodyPair(oracle, bc, 3, seed=4, fill=lambda g: [30, 62, 95])
    g = np.random.default_rng(8)
    for _ in range(36):
        pair.step(g.integers(0, bc.V, size=3))


class _Device:
    """One body on the GPU: weights, caches, a step from the same start whenever asked."""

    def __init__(self, torch, binding, bc, rows, seed):
        w = synth.make_body_weights(bc, seed)
        dev = dict(embed=_to_dev(torch, w["embed"]), g_final=torch.from_numpy(w["g_final"]).cuda())
        for key in ("wqkv", "wo", "wgu", "wdown"):
            dev[key] = [_to_dev(torch, a) for a in w[key]]
        for key in ("g_attn", "g_mlp"):
            dev[key] = [torch.from_numpy(a).cuda() for a in w[key]]
        self.torch, self.binding, self.rows = torch, binding, rows
        self.cfg = binding.make_body_cfg(layers=bc.layers, d=bc.d, heads=bc.heads, d_ff=bc.d_ff, V=bc.V, max_ctx=bc.max_ctx)
        self.body = binding.BodyBuffers(self.cfg, rows, dev)
        g = torch.Generator().manual_seed(seed)
        self.k0 = torch.randn(self.body.kcache.shape, generator=g).to(torch.bfloat16).cuda()
        self.v0 = torch.randn(self.body.vcache.shape, generator=g).to(torch.bfloat16).cuda()
        self.base = torch.randint(0, bc.max_ctx - 2, (rows,), generator=g, dtype=torch.int32).cuda()
        self.tokens = torch.randint(0, bc.V, (rows,), generator=g, dtype=torch.int32).cuda()

    def reset(self):
        self.body.kcache.copy_(self.k0)
        self.body.vcache.copy_(self.v0)
        self.body.ctx_len.copy_(self.base)

    def step(self, ws=None):
        b = self.body
        self.binding.tabed_draft_body_step(self.cfg, b.table, b.ws if ws is None else ws, self.rows, self.tokens, 1, 1, b.ctx_len, b.kcache,
                                           b.vcache, b.H)

    def step_with(self, ws, late_from=0, absent=0):
        """A step whose workgroups from `late_from` on come late, or whose workgroup `absent` does nothing; how many took part."""
        torch, b, c = self.torch, self.body, ctypes
        ptr = lambda t: c.c_void_p(t.data_ptr())  # noqa: E731
        rc = self.binding.load().tabed_testing_body_step(
            c.byref(self.cfg), c.byref(b.table), ptr(ws), c.c_int32(self.rows), ptr(self.tokens), c.c_int32(1), c.c_int32(1), ptr(b.ctx_len),
            ptr(b.kcache), ptr(b.vcache), ptr(b.H), c.c_void_p(torch.cuda.current_stream().cuda_stream), c.c_int32(late_from), c.c_int32(absent))
        assert rc == 0
        return int(ws[25 * 128 + 24:25 * 128 + 28].view(torch.int32))

    def result(self):
        b = self.body
        return [t.clone() for t in (b.H.view(b.H.dtype), b.kcache, b.vcache, b.ctx_len)]

    def once(self, ws=None):
        self.reset()
        self.step(ws)
        return self.result()


def _same(torch, a, b):
    return all(torch.equal(x.view(torch.int16) if x.dtype == torch.bfloat16 else x, y.view(torch.int16) if y.dtype == torch.bfloat16 else y)
               for x, y in zip(a, b))


def test_a_workspace_shared_with_other_sizes_gives_the_same_results():
    """One workspace, prepared once, used in turn for two sizes of one-launch steps, fewer rows of one of them and a step that
    takes the launches per phase, whose scratch lies over the other steps' buffers."""
    torch, binding = _gpu()
    devs = [_Device(torch, binding, B(layers=2, d=256, heads=4, d_ff=520, V=50, max_ctx=80), 12, 1),
            _Device(torch, binding, B(layers=1, d=512, heads=4, d_ff=1024, V=50, max_ctx=80), 5, 2),
            _Device(torch, binding, B(layers=2, d=256, heads=4, d_ff=520, V=50, max_ctx=80), 3, 3),
            _Device(torch, binding, B(layers=1, d=256, heads=16, d_ff=512, V=50, max_ctx=80), 40, 4)]
    alone = [d.once() for d in devs]
    need = max(binding.tabed_body_workspace_bytes(d.cfg, d.rows) for d in devs)
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    binding.tabed_body_workspace_init(devs[0].cfg, devs[0].rows, ws)
    for i in (0, 0, 1, 0, 3, 0, 2, 2, 3, 1, 1, 0):
        assert _same(torch, devs[i].once(ws), alone[i]), i


@pytest.mark.parametrize("ctx_a,ctx_b", [(80, 256), (256, 1024), (1024, 80)])
def test_a_workspace_shared_by_bodies_that_differ_in_the_cache_length(ctx_a, ctx_b):
    """The launches per phase would cut such bodies' attention into other numbers of ranges; the one-launch step's buffers are the same."""
    torch, binding = _gpu()
    devs = [_Device(torch, binding, B(layers=3, d=768, heads=12, d_ff=520, V=50, max_ctx=m), 4, 5 + i) for i, m in enumerate((ctx_a, ctx_b))]
    alone = [d.once() for d in devs]
    ws = torch.full((max(binding.tabed_body_workspace_bytes(d.cfg, d.rows) for d in devs),), 0x5A, dtype=torch.uint8, device="cuda")
    binding.tabed_body_workspace_init(devs[0].cfg, devs[0].rows, ws)
    for i in (0, 1, 0, 1, 1, 0, 0, 1):
        assert _same(torch, devs[i].once(ws), alone[i]), i


def test_a_workspace_of_many_rows_serves_few_and_many_in_turn():
    """Prepared for rows that take whole matrix products for the projections, then one-launch steps of 16 and 3 rows, whose buffers
    need more room than those, and the many rows again."""
    torch, binding = _gpu()
    bc = B(layers=10, d=1024, heads=8, d_ff=8, V=50, max_ctx=6)
    devs = [_Device(torch, binding, bc, rows, 5) for rows in (301, 16, 3)]
    alone = [d.once() for d in devs]
    ws = torch.full((binding.tabed_body_workspace_bytes(devs[0].cfg, 301) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    binding.tabed_body_workspace_init(devs[0].cfg, 301, ws)
    for i in (0, 1, 0, 2, 1, 2, 0):
        assert _same(torch, devs[i].once(ws), alone[i]), i
    assert bool((ws[-4096:] == 0x5A).all())


@pytest.mark.parametrize("fill", [0x00, 0x5A, 0xFF], ids=hex)
def test_a_workspace_that_nobody_prepared(fill):
    """Not asked for by the interface, but no reason for a step that does nothing and says nothing: the results are the same bits, and a
    workspace written over after the preparation is as good as new once it is prepared again."""
    torch, binding = _gpu()
    d = _Device(torch, binding, B(layers=2, d=256, heads=4, d_ff=520, V=50, max_ctx=80), 5, 1)
    alone = d.once()
    ws = torch.full((binding.tabed_body_workspace_bytes(d.cfg, d.rows),), fill, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        assert _same(torch, d.once(ws), alone)
    binding.tabed_body_workspace_init(d.cfg, d.rows, ws)
    for _ in range(3):
        assert _same(torch, d.once(ws), alone)
    ws.fill_(fill)
    assert _same(torch, d.once(ws), alone)


def test_graph_replays_of_one_launch_steps():
    """Three steps in a graph, replayed with eager steps and synchronisation in between: each replay gives what eager steps give."""
    torch, binding = _gpu()
    d = _Device(torch, binding, B(layers=2, d=256, heads=4, d_ff=520, V=50, max_ctx=80), 4, 5)
    d.reset()
    d.base.clamp_(max=60)
    d.reset()
    for _ in range(3):
        d.step()
    want = d.result()
    d.reset()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(3):
            d.step()
    for _ in range(5):
        d.reset()
        graph.replay()
        torch.cuda.synchronize()
        assert _same(torch, d.result(), want)
        d.once()


def test_one_launch_steps_on_streams_that_compete():
    """Two bodies on two streams, each with its workspace, and large matrix products on a third: whoever gets compute units late
    takes no part, and the results are the same bits."""
    torch, binding = _gpu()
    a = _Device(torch, binding, B(layers=3, d=256, heads=4, d_ff=1024, V=50, max_ctx=120), 6, 6)
    b = _Device(torch, binding, B(layers=2, d=512, heads=4, d_ff=520, V=50, max_ctx=120), 16, 7)
    want_a, want_b = a.once(), b.once()
    streams = [torch.cuda.Stream() for _ in range(3)]
    x = torch.randn(2048, 2048, device="cuda")
    torch.cuda.synchronize()
    for _ in range(10):
        a.reset()
        b.reset()
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[2]):
            y = x @ x
        with torch.cuda.stream(streams[0]):
            a.step()
        with torch.cuda.stream(streams[1]):
            b.step()
        with torch.cuda.stream(streams[2]):
            y = y @ x
        torch.cuda.synchronize()
        assert _same(torch, a.result(), want_a) and _same(torch, b.result(), want_b)
    assert y.shape == x.shape


@pytest.mark.parametrize("late_from", [255, 200, 64, 63, 9, 1])
@pytest.mark.parametrize("rows,bc", [(5, B(layers=2, d=768, heads=12, d_ff=3072, V=50, max_ctx=600)), (16, B(layers=2, d=256, heads=2, d_ff=1000, V=50, max_ctx=300))],
                         ids=["rows5_hd64", "rows16_hd128"])
def test_workgroups_that_come_late_take_no_part(rows, bc, late_from):
    """The others close the registration (after 20 us, or 1 ms where fewer than 64 are in) and deal all items to themselves: same bits,
    on a workspace that has to be filled first, on one that is filled, and with all workgroups again afterwards."""
    torch, binding = _gpu()
    d = _Device(torch, binding, bc, rows, 9)
    want = d.once()
    ws = torch.full((binding.tabed_body_workspace_bytes(d.cfg, rows),), 0x5A, dtype=torch.uint8, device="cuda")
    binding.tabed_body_workspace_init(d.cfg, rows, ws)
    for _ in range(3):
        d.reset()
        assert 1 <= d.step_with(ws, late_from=late_from) <= late_from      # (all of them, unless one is 20 us behind the rest)
        assert _same(torch, d.result(), want)
    d.reset()
    assert 64 <= d.step_with(ws) <= 256
    assert _same(torch, d.result(), want)


@pytest.mark.parametrize("absent", [7, 40, 192])
def test_a_wait_that_ends_unanswered_is_seen(absent):
    """A workgroup that registers and computes nothing (q/k/v and gate / up, gate / up alone, output and down projections): no result
    that looks like one, positions where they were, and the next step as ever."""
    torch, binding = _gpu()
    d = _Device(torch, binding, B(layers=2, d=256, heads=4, d_ff=1024, V=50, max_ctx=120), 6, 10)
    want = d.once()
    ws = torch.full((binding.tabed_body_workspace_bytes(d.cfg, d.rows),), 0x5A, dtype=torch.uint8, device="cuda")
    binding.tabed_body_workspace_init(d.cfg, d.rows, ws)
    for filled in (False, True, True):
        if filled:
            assert _same(torch, d.once(ws), want)
        d.reset()
        d.body.H.zero_()
        d.step_with(ws, absent=absent)
        assert torch.equal(d.body.ctx_len, d.base)
        assert bool(torch.isnan(d.body.H.float()).all())
    assert _same(torch, d.once(ws), want)
