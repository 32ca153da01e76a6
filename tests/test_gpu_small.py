"""The small network's step kernels that hold each processor queue in a row
of 16 lanes: the 16-slot tile (variant 0, every form) and four wavefronts per
slot (variant 2, FP32).  The tile makes the products of the forward kernel in
the same order, so its recorded outputs equal, bit for bit, the forward of
windows built here from the same latencies; state is carried over launches,
modes and refilled slots without a change to any result."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

D, L = 32, 16
COLS = synth.dynamic_columns(D)  # residence, execution latency, (none)
KEYS = ("fetch", "drain", "final", "warm_tick", "total")


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


def simulator(sn, torch, prec, codes, length, W):
    start = np.concatenate([[0], np.cumsum(length)[:-1]]).astype(np.int64)
    n = int(length.sum())
    feat = (synth.trace_codes(1, n).view(np.int32) if codes
            else synth.trace_features(1, n, D))
    s = sn.Simulator(torch.from_numpy(feat).cuda(), L, COLS, start, length,
                     np.zeros(len(length), np.int32), retire_width=W, prec=prec,
                     n_feat=D)
    layers = synth.net_small()
    s.load_weights(layers, sn.flat_params(*synth.init_weights(2, layers,
                                                              out_bias=synth.OUT_BIAS)))
    if prec == sn.SIM_FP8E4M3:
        s.calibrate(4)
    return s


def windows(length, table, W):
    """Every prediction's window under the latencies `table` (clock and queue
    written out plainly; the small network has no store column)."""
    feat = synth.trace_features(1, int(length.sum()), D)
    out = np.zeros((len(feat), L, D), np.float32)
    i = 0
    for n in length:
        cur, r_prev, q, rs = 0, 0, [], []  # q: (row, T, E, r), oldest first
        for _ in range(n):
            out[i, 0] = feat[i]
            out[i, 0, COLS[:2]] = 0
            for w, (row, t, e, _) in enumerate(reversed(q), 1):
                out[i, w] = feat[row]
                out[i, w, COLS[:2]] = cur - t, e
            f, e = int(table[i, 0]), int(table[i, 1])
            cur += f
            q = [x for x in q if x[3] > cur]
            r = max(cur + e + 1, r_prev, rs[-W] + 1 if len(rs) >= W else 0)
            rs.append(r)
            q = (q + [(i, cur, e, r)])[-(L - 1):]
            r_prev = r
            i += 1
    return out


def case(seed):
    rng = np.random.default_rng(seed)
    length = rng.integers(1, 60, 37)
    length[:3] = 1, 59, 2
    n = int(length.sum())
    table = np.stack([rng.integers(0, 4, n), rng.integers(0, 30, n)], 1).astype(np.int32)
    table[rng.random(n) < 0.4, 0] = 0  # long queues
    table[rng.random(n) < 0.05, 0] = 90  # and empty ones
    return length, table


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("codes,W", [(False, 8), (True, 1), (False, 16)])
def test_tile_outputs_equal_forward_of_its_windows(torch, sn, prec, codes, W):
    length, table = case(3)
    s = simulator(sn, torch, prec, codes, length, W)
    s.set_tuning(0, 3)
    z = torch.full((s.n_pred, 2), np.nan, device="cuda")
    s.record_logits(z)
    s.run(sn.SIM_LAT_SHADOW, torch.from_numpy(table).cuda())
    want = s.forward(torch.from_numpy(windows(length, table, W)).cuda())
    assert torch.equal(z, want)
    s.close()


@pytest.mark.parametrize("prec,variant", [(0, 0), (1, 0), (2, 0), (0, 2)])
def test_pieces_modes_and_refills_carry_the_state(torch, sn, prec, variant):
    length, table = case(5)
    s = simulator(sn, torch, prec, False, length, 5)
    dev = torch.from_numpy(table).cuda()
    s.set_tuning(variant, 3)
    want = s.run(sn.SIM_LAT_SHADOW, dev)
    s.reset()
    free = s.run()
    for n_wg in (1, 2):  # 16 and 32 slots for 37 sub-traces
        s.set_tuning(variant, n_wg)
        for i, m in enumerate((3, 20, 1, 7, 30, 2)):
            s.step(m, sn.SIM_LAT_INJECT if i % 2 else sn.SIM_LAT_SHADOW, dev)
        got = s.run(sn.SIM_LAT_SHADOW, dev)
        for k in KEYS:
            np.testing.assert_array_equal(got[k], want[k], err_msg=k)
        s.reset()
        for m in (1, 16, 5):
            s.step(m)
        got = s.run()
        for k in KEYS:
            np.testing.assert_array_equal(got[k], free[k], err_msg=k)
    s.close()


@pytest.mark.parametrize("n_sub", [5, 65536, 65537])
def test_results_however_they_are_copied(torch, sn, n_sub):
    """Few sub-traces' results come in one copy, many straight to the caller's
    arrays, and only the arrays asked for: the same numbers, and those of the
    sub-traces in two halves."""
    import ctypes as C
    rng = np.random.default_rng(7)
    length = rng.integers(1, 4, n_sub)
    at = np.concatenate([[0], np.cumsum(length)])
    table = np.stack([rng.integers(0, 4, at[-1]), rng.integers(0, 30, at[-1])], 1).astype(np.int32)

    def run(lo, hi):
        s = simulator(sn, torch, 1, True, length[lo:hi], 8)
        dev = torch.from_numpy(table[at[lo]:at[hi]]).cuda()
        return s, dev, s.run(sn.SIM_LAT_INJECT, dev)

    s, dev, got = run(0, n_sub)
    halves = [run(0, n_sub // 2)[2], run(n_sub // 2, n_sub)[2]]
    for k in ("fetch", "drain", "final", "warm_tick"):
        np.testing.assert_array_equal(got[k], np.concatenate([h[k] for h in halves]), err_msg=k)
    assert got["total"] == int((got["final"] - got["warm_tick"]).sum())
    fields = {"fetch": "fetch_cycles", "drain": "drain_cycles", "final": "final_tick",
              "warm_tick": "warm_tick"}
    for asked in ((), ("drain",), ("fetch", "warm_tick"), ("final",)):
        s.reset()
        res, out = sn.sim_result(), {k: np.full(n_sub, -1, np.int64) for k in asked}
        for k in asked:
            setattr(res, fields[k], out[k].ctypes.data_as(C.POINTER(C.c_int64)))
        assert sn.lib().sim_run(s.ctx, sn.SIM_LAT_INJECT, dev.data_ptr(), C.byref(res)) == 0
        assert res.total_cycles == got["total"] and res.measured_instr == at[-1]
        for k in asked:
            np.testing.assert_array_equal(out[k], got[k], err_msg=k)
    s.close()


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("codes", [False, True])
def test_short_sub_traces_refill_the_slots(torch, sn, prec, codes):
    """More sub-traces than slots, 1 to 9 instructions each (slots of a
    workgroup end together and apart, the last ones find nothing left): run at
    once, in pieces that stop between and at ends, and in 32 slots."""
    length = np.random.default_rng(11).integers(1, 10, 17_000)
    s = simulator(sn, torch, prec, codes, length, 4)
    s.set_tuning(0, 1024)
    z = [torch.full((s.n_pred, 2), np.nan, device="cuda") for _ in range(3)]
    s.record_logits(z[0])
    want = s.run()
    for out, n_wg in ((z[1], 1024), (z[2], 2)):
        s.set_tuning(0, n_wg)
        s.record_logits(out)
        for m in (1, 2, 5, 3):
            s.step(m)
        got = s.run()
        for k in KEYS + ("n_clamped", "n_nonfinite"):
            np.testing.assert_array_equal(got[k], want[k], err_msg=k)
        assert torch.equal(out, z[0])
    s.close()
