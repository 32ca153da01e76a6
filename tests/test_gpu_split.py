"""Few windows spread over several workgroups per tile (the split step and
forward) against the one-workgroup-per-tile kernels, which the other tests
hold to the oracle: the same products summed in the same order, so every
output, cycle and counter is identical.  With fewer slots than sub-traces a
run takes the one-workgroup step; with a slot for each it is split (2, 66 and
128 tiles: column slices, one unit per group or several groups per unit).
Batches above 2,048 windows take the one-workgroup forward.  RB7's residual
blocks run on tiles of another size per row count."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

D, L = 50, 111
COLS = synth.dynamic_columns(D)
KEYS = ("fetch", "drain", "final", "warm_tick", "total", "n_clamped", "n_nonfinite")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def sn():
    import paper_2105_05821_amd as m
    m.lib()
    return m


NETS = {"c3": (synth.net_c3, synth.OUT_BIAS), "dep": (synth.net_c3, synth.OUT_BIAS),
        "hyb": (synth.net_c3_hybrid_infer, synth.HYB_BIAS),
        "st": (synth.net_c3_store, synth.OUT_BIAS_STORE),
        "rb7": (synth.net_rb7, synth.HYB_BIAS)}


def streams(n_sub, seed):
    length = synth.loguniform_lengths(seed, n_sub, 1, 24)
    start = np.concatenate([[0], np.cumsum(length)[:-1]]).astype(np.int64)
    return start, length, np.minimum(start, length % 7).astype(np.int32)


def simulator(sn, torch, net, prec, start, length, warm, codes=False):
    n = int(start[-1] + length[-1])
    feat = (synth.trace_codes(1, n).view(np.int32) if codes
            else synth.trace_features(1, n, D))
    mem = (torch.from_numpy(synth.trace_mem(1, n).view(np.int32)).cuda() if net == "dep"
           else None)
    s = sn.Simulator(torch.from_numpy(feat).cuda(), L, COLS, start, length, warm, prec=prec,
                     n_feat=D, n_out=3 if net == "st" else 2, store_col=synth.STORE_COL,
                     mem=mem, col_dep=synth.DEP_COLS if net == "dep" else -1)
    layers, bias = NETS[net][0](), NETS[net][1]
    s.load_weights(layers, sn.flat_params(*synth.init_weights(2, layers, out_bias=bias)))
    if prec == sn.SIM_FP8E4M3:
        s.calibrate(4)
    return s


def same(a, b):
    for k in KEYS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("net,prec,n_sub,codes", [
    ("c3", 1, 17, False), ("c3", 1, 1041, True), ("c3", 1, 2048, False), ("c3", 0, 17, True),
    ("c3", 0, 600, False), ("c3", 2, 300, False), ("dep", 1, 40, False), ("dep", 0, 40, True),
    ("hyb", 1, 530, True), ("hyb", 0, 33, False), ("st", 1, 290, False), ("st", 0, 290, True),
    ("rb7", 1, 33, False), ("rb7", 0, 17, True)])
def test_split_step_equals_one_workgroup(torch, sn, net, prec, n_sub, codes):
    start, length, warm = streams(n_sub, 3)
    s = simulator(sn, torch, net, prec, start, length, warm, codes)
    n_out = NETS[net][0]()[-1].c_out
    got = torch.zeros((s.n_pred, n_out), device="cuda")
    want = torch.full_like(got, np.nan)
    s.record_logits(got)
    a = s.run()                     # split
    s.reset()
    got2 = torch.zeros_like(got)
    s.record_logits(got2)
    for n in (1, 5, 2):             # in pieces
        s.step(n)
    b = s.run()
    s.set_tuning(0, (n_sub + 15) // 16 - 1)
    s.record_logits(want)
    c = s.run()                     # one workgroup per tile, slots refilled
    same(a, c)
    same(b, c)
    assert torch.equal(got, want) and torch.equal(got2, want)
    s.close()


@pytest.mark.parametrize("net,prec", [("c3", 1), ("st", 1), ("st", 0), ("hyb", 0)])
def test_split_and_injected_steps_alternate(torch, sn, net, prec):
    """Steps of both kinds share one state: injected latencies run on the
    one-workgroup step, shadow steps with the same latencies are split; long
    fetch-free runs fill the processor queue past its 110 entries."""
    n_sub, n = 18, 400
    start = np.arange(n_sub, dtype=np.int64) * n
    length = np.full(n_sub, n, np.int64)
    length[3], length[7] = 150, 9
    s = simulator(sn, torch, net, prec, start, length, np.zeros(n_sub, np.int32))
    t = synth.latency_table(4, s.n_pred, 3 if net == "st" else 2, e_max=300, heavy=0.05)
    t[::1, 0] *= np.random.default_rng(1).random(len(t)) < 0.3
    table = torch.from_numpy(t).cuda()
    want = s.run(sn.SIM_LAT_INJECT, table)
    s.reset()
    for i, m in enumerate((3, 130, 1, 7, 25, 60, 2)):
        s.step(m, sn.SIM_LAT_INJECT if i % 2 == 0 else sn.SIM_LAT_SHADOW, table)
    got = s.run(sn.SIM_LAT_SHADOW, table)
    for k in ("fetch", "drain", "final", "warm_tick", "total"):
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)
    s.close()


@pytest.mark.parametrize("net,prec", [("c3", 0), ("c3", 1), ("c3", 2), ("hyb", 0), ("hyb", 1),
                                      ("st", 0), ("st", 1), ("rb7", 0), ("rb7", 1)])
def test_split_forward_equals_one_workgroup(torch, sn, net, prec):
    s = simulator(sn, torch, net, prec, np.array([0]), np.array([8]), np.array([0], np.int32))
    x = torch.randn((2049, L, D), generator=torch.Generator().manual_seed(3)).cuda()
    want = s.forward(x)
    for B in (1, 16, 17, 600, 1000, 1030, 1500, 2048):
        assert torch.equal(s.forward(x[:B].contiguous()), want[:B]), B
    s.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_split_training_forward_equals_one_workgroup(torch, sn, prec):
    layers = synth.net_c3_hybrid()
    ws, bs = synth.init_weights(2, layers, out_bias=None, out_gain=1.0)
    pred = sn.Predictor(layers, prec)
    pred.load_weights(layers, sn.flat_params(ws, bs))
    x = torch.randn((2049, L, D), generator=torch.Generator().manual_seed(3)).cuda()
    sizes = (52 * 64, 26 * 128, 13 * 256, 512)

    def parts(save, B):
        v = save[:pred.save_bytes(B)].view(torch.float32 if prec == 0 else torch.int16)
        at = np.cumsum([0] + [B * n for n in sizes])
        return [v[at[i]:at[i + 1]].view(B, n) for i, n in enumerate(sizes)]

    z, save = pred.forward(x)
    want = parts(save, 2049)
    for B in (1, 17, 1030, 2048):
        zb, sb = pred.forward(x[:B].contiguous())
        assert torch.equal(zb, z[:B]), B
        for g, w in zip(parts(sb, B), want):
            assert torch.equal(g, w[:B]), B
    pred.close()


@pytest.mark.parametrize("net", ["c3", "hyb"])
def test_forward_over_rounds_equals_single_tiles(torch, sn, net):
    """More windows than 16 per CU: whole rounds through the convolutions'
    outputs in memory, a short rest split; on 256 CUs two, three and four row
    tiles per workgroup, two passes, a rest of one window and of 513."""
    s = simulator(sn, torch, net, 1, np.array([0]), np.array([8]), np.array([0], np.int32))
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    rnd = 16 * n_cu
    x = torch.randn((4 * rnd + rnd // 8 + 1, L, D), device="cuda",
                    generator=torch.Generator("cuda").manual_seed(3))
    want = torch.cat([s.forward(x[i:i + rnd].contiguous()) for i in range(0, len(x), rnd)])
    for B in (rnd + 1, 2 * rnd - 15, 2 * rnd + rnd // 8, 2 * rnd + rnd // 2, 3 * rnd + rnd // 2,
              4 * rnd, len(x)):
        assert torch.equal(s.forward(x[:B].contiguous()), want[:B]), B
    s.close()


def test_captured_forwards_replay(torch, sn):
    """A captured forward of few windows (split) and of more than a round
    (through memory), replayed between eager calls of other sizes, gives the
    eager result every time."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = simulator(sn, torch, "c3", 1, np.array([0]), np.array([8]), np.array([0], np.int32))
        rnd = 16 * torch.cuda.get_device_properties(0).multi_processor_count
        x = torch.randn((2 * rnd, L, D), device="cuda",
                        generator=torch.Generator("cuda").manual_seed(5))
        want = s.forward(x)
        side.synchronize()
        for B in (5, rnd + rnd // 2):
            xb = x[:B].contiguous()
            out = torch.empty_like(want[:B])
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                out.copy_(s.forward(xb))
            for i in range(3):
                out.zero_()
                graph.replay()
                side.synchronize()
                assert torch.equal(out, want[:B]), (B, i)
                assert torch.equal(s.forward(x[:B - 1 - i].contiguous()), want[:B - 1 - i])
        s.close()


@pytest.mark.parametrize("net,prec,n_sub,other", [
    ("c3", 1, 512, 2400), ("c3", 0, 512, 2400), ("c3", 2, 300, 2400), ("dep", 1, 512, 2400),
    ("hyb", 1, 777, 2400), ("st", 1, 512, 2400), ("st", 0, 290, 2400), ("rb7", 1, 200, 2400),
    ("c3", 1, 512, 2048), ("hyb", 0, 2048, 512)])
def test_split_run_beside_another_context(torch, sn, net, prec, n_sub, other):
    """A split run on one stream beside another context's steps on a second.
    The other context's workgroups hold CUs (2,400 sub-traces: 150 of them for
    its whole launch; fewer: a split run too), so a launch's workgroups start at
    different times, some after others of their tile have ended: every output
    equals that of the same run alone, one workgroup per tile."""
    start, length, warm = streams(n_sub, 3)
    n_out = NETS[net][0]()[-1].c_out
    n = 100
    o_start = np.arange(other, dtype=np.int64) * n
    o_len = np.full(other, n, np.int64)
    with torch.cuda.stream(torch.cuda.Stream()):
        s = simulator(sn, torch, net, prec, start, length, warm)
    with torch.cuda.stream(torch.cuda.Stream()):
        o = simulator(sn, torch, "c3", 1, o_start, o_len, np.zeros(other, np.int32), codes=True)
    o_want = o.run()
    s.set_tuning(0, (n_sub + 15) // 16 - 1)
    want_z = torch.full((s.n_pred, n_out), np.nan, device="cuda")
    got_z = torch.zeros_like(want_z)
    torch.cuda.synchronize()
    s.record_logits(want_z)
    want = s.run()
    s.set_tuning(0, (n_sub + 15) // 16)
    s.record_logits(got_z)
    for i in range(3):
        o.reset()
        s.reset()
        torch.cuda.synchronize()
        got_z.zero_()
        torch.cuda.synchronize()
        o.step(n)
        same(s.run(), want)
        assert torch.equal(got_z, want_z), i
        same(o.run(), o_want)
    s.close()
    o.close()


def test_large_forward_returns_an_error(torch, sn):
    """A batch of several passes whose first pass fails (here an error that an
    earlier call of this thread left behind and the launch picks up) returns
    the error, and the next call is right."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so.7")
    s = simulator(sn, torch, "hyb", 1, np.array([0]), np.array([8]), np.array([0], np.int32))
    rnd = 16 * torch.cuda.get_device_properties(0).multi_processor_count
    x = torch.randn((4 * rnd + rnd // 2, L, D), device="cuda",
                    generator=torch.Generator("cuda").manual_seed(3))
    want = s.forward(x)
    out = torch.empty_like(want)
    torch.cuda.synchronize()
    assert hip.hipSetDevice(-1) != 0
    with pytest.raises(sn.SimError):
        s.forward(x, out)
    torch.cuda.synchronize()
    assert torch.equal(s.forward(x, out), want)
    s.close()


@pytest.mark.parametrize("net", ["c3", "rb7"])
def test_captured_reset_replayed_after_steps(torch, sn, net):
    """A reset that was captured and is replayed after eager steps: the run
    that follows is a whole run (the host does not see the replay)."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        start, length, warm = streams(50, 3)
        s = simulator(sn, torch, net, 1, start, length, warm)
        want = s.run()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            s.reset()
        for n in (3, 9, 40):
            graph.replay()
            s.step(n)
            side.synchronize()
        graph.replay()
        same(s.run(), want)
        s.reset()
        s.step(5)
        same(s.run(), want)
        s.close()


@pytest.mark.parametrize("net,prec,B", [("c3", 1, 5), ("c3", 0, 40), ("hyb", 1, 600), ("st", 1, 33),
                                        ("c3", 1, 4600)])
def test_captured_forwards_replay_at_once(torch, sn, net, prec, B):
    """Two captured forwards of one context replayed on two streams, beside
    the context's own steps: none shares memory with another."""
    side, a, b = (torch.cuda.Stream() for _ in range(3))
    with torch.cuda.stream(side):
        start, length, warm = streams(300, 3)
        s = simulator(sn, torch, net, prec, start, length, warm)
        want_run = s.run()
        x = torch.randn((2, B, L, D), device="cuda",
                        generator=torch.Generator("cuda").manual_seed(7))
        want = [s.forward(x[i]) for i in range(2)]
        out = [torch.zeros_like(w) for w in want]
        graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
        for g, xi, o in zip(graphs, x, out):
            with torch.cuda.graph(g, stream=side):
                s.forward(xi, o)
    torch.cuda.synchronize()
    for i in range(4):
        for o in out:
            o.zero_()
        s.reset()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            s.step(10)
        for g, st in zip(graphs, (a, b)):
            with torch.cuda.stream(st):
                for _ in range(3):
                    g.replay()
        same(s.run(), want_run)
        torch.cuda.synchronize()
        for o, w in zip(out, want):
            assert torch.equal(o, w), i
    s.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_captured_training_forwards_replay_at_once(torch, sn, prec):
    side, a, b = (torch.cuda.Stream() for _ in range(3))
    layers = synth.net_c3_hybrid()
    params = sn.flat_params(*synth.init_weights(2, layers, out_bias=None, out_gain=1.0))
    with torch.cuda.stream(side):
        pred = sn.Predictor(layers, prec)
        pred.load_weights(layers, params)
        x = torch.randn((2, 40, L, D), device="cuda",
                        generator=torch.Generator("cuda").manual_seed(7))
        want = [pred.forward(xi) for xi in x]
        graphs, got = [], []
        for xi in x:
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1], stream=side):
                got.append(pred.forward(xi))
    torch.cuda.synchronize()
    for i in range(4):
        for z, save in got:
            z.zero_()
            save.zero_()
        torch.cuda.synchronize()
        for g, st in zip(graphs, (a, b)):
            with torch.cuda.stream(st):
                g.replay()
        torch.cuda.synchronize()
        for (z, save), (wz, ws) in zip(got, want):
            assert torch.equal(z, wz) and torch.equal(save, ws), i
    pred.close()


@pytest.mark.parametrize("net,prec,n_sub", [("c3", 1, 600), ("c3", 0, 40), ("c3", 1, 9), ("hyb", 1, 40)])
def test_autotune_times_a_split_shape_once(torch, sn, net, prec, n_sub):
    """The split step is one kernel whatever the variant: one trial of the
    full shape, with the choice's results and every variant's own (below the
    full shape, where its kernel runs) those of the default."""
    start, length, warm = streams(n_sub, 3)
    s = simulator(sn, torch, net, prec, start, length, warm, codes=True)
    want = s.run()
    full = (n_sub + 15) // 16
    t = s.autotune(6)
    shapes = {full} | {max(1, full * q // 4) for q in (2, 3)}
    assert [n for _, n, _ in t["trials"]].count(full) == 1 and t["trials"][-1][1] == full
    assert {n for _, n, _ in t["trials"]} == shapes
    assert (t["variant"], t["n_wg"]) in [(v, n) for v, n, _ in t["trials"]]
    if net == "c3" and len(shapes) > 1:
        free = {v for v in range(4) if s.variant_scratch(v) == 0} or set(range(4))
        assert {v for v, n, _ in t["trials"] if n != full} == free
    same(s.run(), want)
    for v in range(4):
        for n in shapes:
            s.set_tuning(v, n)
            same(s.run(), want)
    s.close()


@pytest.mark.parametrize("net", ["c3", "st"])
def test_short_calls_on_many_tiles(torch, sn, net):
    """Calls of one and two steps on 86 to 128 tiles (one workgroup per tile)
    between longer ones (split), and a run with two steps left."""
    start, length, warm = streams(1400, 3)
    s = simulator(sn, torch, net, 1, start, length, warm)
    want = s.run()
    for calls in ((1, 3, 2, 1, 4, 2), (2, 1), (int((length + warm).max()) - 2,)):
        s.reset()
        for n in calls:
            s.step(n)
        same(s.run(), want)
    s.close()
