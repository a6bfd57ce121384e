"""The stop test and restart pick with a group of threads per rollout (one wave, one workgroup of
256, or one of 1,024 / 512 threads, by the average rollout), against the oracle: rollouts at the
edges of a group's chunk, empty rollouts, a K0 at the end, both units, and offsets that do not
cover the units."""
import numpy as np
import pytest

from tests import harness as H

pytestmark = pytest.mark.gpu

SIZES = {  # lengths at the edges of a chunk of 128, 1,024 and 8,192 (restart: 128, 2,048, 4,096) units
    "wave": [1, 0, 127, 128, 129, 0, 2, 300, 63, 64, 65, 1, 255, 256, 257, 3, 0],
    "block": [1023, 1024, 1025, 1, 0, 2047, 2048, 2049, 255, 257, 700, 5],
    "wide": [8191, 8192, 8193, 1, 0, 4095, 4096, 4097, 16385, 12289, 2],
    "skewed": [40000] + [3] * 1500,
    # longer than a wave takes (1,024 units) among short ones: alone, one after the other, the first and the
    # last; and more rollouts than the workgroups that take these look at in one round (127 x 256)
    "far": [1023, 1024, 1025, 2049, 1, 0, 5000, 1536, 1537] + [2] * 200 + [9000] + [1] * 150 + [1100],
    "far in a second round": [1500] + [3] * 32600 + [1100, 2, 1300] + [1] * 30,
    "block and far": [8193, 20000, 8192, 16500] + [300] * 100,   # past eight chunks of a workgroup
    "tiles": [140000, 1, 0, 2048],   # past the average a group takes: the tile scan
}


@pytest.mark.parametrize("unit", ["turn", "token"])
@pytest.mark.parametrize("name", list(SIZES))
def test_groups_against_the_oracle(name, unit):
    import torch
    import paper_2609_14636_amd as P
    g = np.random.default_rng(len(name) + (unit == "turn"))
    sizes = np.array(SIZES[name])
    R = sizes.size
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    U = int(off[-1])
    if unit == "token":
        rto, tto = np.arange(R + 1, dtype=np.int32), off
    else:
        rto, tto = off.astype(np.int32), np.concatenate([[0], np.cumsum(g.integers(0, 4, U))]).astype(np.int64)
    N = int(tto[-1])
    vals = -np.abs(g.normal(0.5, 0.5, size=U))
    vals[g.random(U) < 0.002] = -np.inf if unit == "token" else -30.0
    vals = vals.astype(np.float32 if unit == "token" else np.float64)
    lam, alpha = [-0.3 * sizes.max(), -40.0, -np.inf], [-1.9, -np.inf, -4.0]
    dom = g.integers(0, 3, size=R).astype(np.int32)
    start = (g.random(R) * sizes * 0.4).astype(np.int32)
    start[::5] = sizes[::5] + 7   # past the end: clamped to the rollout's length
    start[1::7] = -3
    mask = (g.random(U) < 0.999).astype(np.uint8)
    k0 = np.clip(start, 0, sizes).astype(np.int32)
    rows = tto if unit == "turn" else np.arange(U + 1, dtype=np.int64)
    cum_o, stop_o, ret_o = H.OP.O.stop(off, vals.astype(np.float64), np.array(lam)[dom], k0, rows)
    rec = np.where(stop_o >= 0, stop_o + 1, sizes).astype(np.int32)
    ks_o, k0_o, km_o = H.OP.O.restart(off, vals.astype(np.float64), rec, np.array(alpha)[dom], mask)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    lay = P.Layout(dev(rto), dev(tto), N, dev(dom))
    code = P.STRIDE_UNIT_TOKEN if unit == "token" else P.STRIDE_UNIT_TURN
    path = P.Path(lay, code, with_student=False)
    for t in (path.cum, path.stop_unit, path.retained, path.k_star, path.k0, path.k_max):
        t.fill_(77)
    P.stride_stop(lay, code, dev(vals), lam, dev(start), path.cum, path.stop_unit, path.retained,
                  path.flags, path.ws)
    P.stride_restart_turn(lay, code, dev(vals), path.stop_unit, alpha, dev(mask), path.k_star,
                          path.k0, path.k_max, path.flags)
    got = path.host()
    assert got["flags"] == 0
    fin = np.isfinite(cum_o)
    assert np.array_equal(got["cum"][~fin], cum_o[~fin])
    # sums of at most 16,385 doubles in another order: far below 1e-9 of their size
    assert np.all(np.abs(got["cum"][fin] - cum_o[fin]) <= 1e-9 * np.maximum(np.abs(cum_o[fin]), 1))
    for k, o in (("stop_unit", stop_o), ("retained", ret_o), ("k_star", ks_o), ("k0", k0_o), ("k_max", km_o)):
        assert np.array_equal(got[k], o), k


def test_units_in_no_rollout():
    """Offsets that start late or end early are flagged; the units in no rollout are NaN and
    nothing past the arrays is written."""
    import torch
    import paper_2609_14636_amd as P
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    lay = P.Layout(dev(np.array([3, 5, 9], np.int32)), dev(np.arange(13, dtype=np.int64)), 12)
    cum = torch.full((20,), 5.0, dtype=torch.float64, device="cuda")
    stop = torch.full((2,), 5, dtype=torch.int32, device="cuda")
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.stride_workspace_size(lay, P.STRIDE_UNIT_TURN), dtype=torch.uint8, device="cuda")
    vals = -torch.ones(12, dtype=torch.float64, device="cuda")
    P.stride_stop(lay, P.STRIDE_UNIT_TURN, vals, [-2.5], None, cum, stop, None, flags, ws)
    assert int(flags.item()) == P.STRIDE_FLAG_BAD_OFFSETS
    c = cum.cpu().numpy()
    assert np.isnan(c[:3]).all() and np.isnan(c[9:12]).all() and (c[12:] == 5.0).all()
    assert c[3:9].tolist() == [-1, -2, -1, -2, -3, -4] and stop.tolist() == [-1, 2]


@pytest.mark.parametrize("late,early", [(3, 0), (0, 5), (5000, 7000), (2047, 2049)])
def test_units_in_no_rollout_as_tiles(late, early):
    """The same with more rollouts than the groups take: the tile scan.  The units before the first
    rollout and past the last one are NaN, whole tiles of them too; the others are summed as without them."""
    import torch
    import paper_2609_14636_amd as P
    R = (1 << 15) + 1
    g = np.random.default_rng(late + early)
    off = late + np.concatenate([[0], np.cumsum(g.integers(0, 3, R))]).astype(np.int64)
    U = int(off[-1]) + early
    vals = -np.abs(g.normal(0.5, 0.5, U))
    rows = np.arange(U + 1, dtype=np.int64)
    inner = slice(late, U - early)
    cum_o, stop_o, ret_o = H.OP.O.stop(off - late, vals[inner].copy(), np.full(R, -1.2), np.zeros(R, np.int32),
                                       np.arange(U - late - early + 1, dtype=np.int64))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    lay = P.Layout(dev(off.astype(np.int32)), dev(rows), U)
    cum = torch.full((U + 5,), 5.0, dtype=torch.float64, device="cuda")
    stop = torch.full((R,), 77, dtype=torch.int32, device="cuda")
    ret = torch.full((R,), 77, dtype=torch.int64, device="cuda")
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.stride_workspace_size(lay, P.STRIDE_UNIT_TURN), dtype=torch.uint8, device="cuda")
    P.stride_stop(lay, P.STRIDE_UNIT_TURN, dev(vals), [-1.2], None, cum, stop, ret, flags, ws)
    assert int(flags.item()) == P.STRIDE_FLAG_BAD_OFFSETS
    c = cum.cpu().numpy()
    assert np.isnan(c[:late]).all() and np.isnan(c[U - early:U]).all() and (c[U:] == 5.0).all()
    assert np.max(np.abs(c[inner] - cum_o)) <= 1e-12
    assert np.array_equal(stop.cpu().numpy(), stop_o) and np.array_equal(ret.cpu().numpy(), ret_o)


def test_many_short_rollouts_as_tiles():
    """One rollout more than the groups take: the tile scan, against float64 sums."""
    import torch
    import paper_2609_14636_amd as P
    R = (1 << 15) + 1
    g = np.random.default_rng(4)
    off = np.concatenate([[0], np.cumsum(g.integers(0, 5, R))]).astype(np.int64)
    U = int(off[-1])
    vals = -np.abs(g.normal(0.5, 0.5, U))
    lam = [-1.2]
    cum_o, stop_o, ret_o = H.OP.O.stop(off, vals, np.full(R, lam[0]), np.zeros(R, np.int32),
                                       np.arange(U + 1, dtype=np.int64))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    lay = P.Layout(dev(off.astype(np.int32)), dev(np.arange(U + 1, dtype=np.int64)), U)
    path = P.Path(lay, P.STRIDE_UNIT_TURN, with_student=False)
    P.stride_stop(lay, P.STRIDE_UNIT_TURN, dev(vals), lam, None, path.cum, path.stop_unit, path.retained,
                  path.flags, path.ws)
    assert int(path.flags.item()) == 0
    assert np.max(np.abs(path.cum.cpu().numpy() - cum_o)) <= 1e-12
    assert np.array_equal(path.stop_unit.cpu().numpy(), stop_o)
    assert np.array_equal(path.retained.cpu().numpy(), ret_o)


@pytest.mark.parametrize("call", ["stop", "restart"])
def test_one_long_rollout_among_short_ones_takes_its_own_time(call):
    """40,000 units before 1,500 rollouts of 3: the stop test and the restart pick take at most 2.5 times
    what the long rollout takes alone (a wave of its own takes 6 and 8 times as long)."""
    import torch
    import paper_2609_14636_amd as P
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731

    def time(sizes):
        off = np.concatenate([[0], np.cumsum(sizes)])
        U = int(off[-1])
        lay = P.Layout(dev(off.astype(np.int32)), dev(np.arange(U + 1, dtype=np.int64)), U)
        path = P.Path(lay, P.STRIDE_UNIT_TURN, with_student=False)
        vals = -torch.rand(U, dtype=torch.float64, device="cuda")

        def run():
            if call == "stop":
                P.stride_stop(lay, P.STRIDE_UNIT_TURN, vals, [-1e9], None, path.cum, path.stop_unit,
                              path.retained, path.flags, path.ws)
            else:
                P.stride_restart_turn(lay, P.STRIDE_UNIT_TURN, vals, None, [-1e9], None, path.k_star,
                                      path.k0, path.k_max, path.flags)
        run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                run()
        graph.replay()
        best = float("inf")
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    alone, among = time([40000]), time([40000] + [3] * 1500)
    print(f"{call}, ms for 20 calls: alone {alone:.3f}, among short ones {among:.3f}", flush=True)
    assert among <= 2.5 * alone


def test_a_record_that_does_not_fill_its_chunk():
    """Restart pick of 64 records of 4,095 units with a mask, one less than a chunk: the time of 4,096."""
    import torch
    import paper_2609_14636_amd as P
    graphs = []
    for n in (4095, 4096):
        U = 64 * n
        lay = P.Layout(torch.arange(65, dtype=torch.int32, device="cuda"),
                       torch.arange(0, U + 1, n, dtype=torch.int64, device="cuda"), U)
        path = P.Path(lay, P.STRIDE_UNIT_TOKEN, with_student=False)
        vals, mask = -torch.rand(U, device="cuda"), torch.ones(U, dtype=torch.uint8, device="cuda")

        def run(lay=lay, vals=vals, mask=mask, path=path):
            P.stride_restart_turn(lay, P.STRIDE_UNIT_TOKEN, vals, None, [-2.0], mask, path.k_star, path.k0,
                                  path.k_max, path.flags)
        run()
        torch.cuda.synchronize()
        assert path.k_max.tolist() == [n] * 64
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(50):
                run()
        graphs.append((graph, run))
    best = [float("inf")] * 2
    for _ in range(15):
        for i in (0, 1):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            graphs[i][0].replay()
            a.record()
            graphs[i][0].replay()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 20)
    print(f"us: 4,095 units {best[0]:.2f}, 4,096 units {best[1]:.2f}", flush=True)
    assert best[0] <= 1.04 * best[1]   # a branch for each load: 1.06 and more
