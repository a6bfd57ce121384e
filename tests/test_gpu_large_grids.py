"""Calls with more rows, turns or rollouts than fit one dimension of a launch at the threads that each
gets (2^32 threads): every one of them is done, the last ones too."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free():
    import torch
    assert torch.cuda.is_available()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _one_turn(n):
    import torch
    import paper_2609_14636_amd as P
    return P.Layout(torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                    torch.tensor([0, n], dtype=torch.int64, device="cuda"), n)


def test_rows():
    """The student is the teacher, so that the rows fit the card."""
    import torch
    import paper_2609_14636_amd as P
    n, vocab = (1 << 23) + 3, 8192          # twice that many rows, four wavefronts each
    x = torch.zeros((n, vocab), dtype=torch.bfloat16, device="cuda")
    x[:, 5] = 1.0
    x[n - 1, 5] = 2.0
    ids = torch.full((n,), 5, dtype=torch.int32, device="cuda")
    ids[::2] = 6
    path = P.Path(_one_turn(n), P.STRIDE_UNIT_TURN)
    path.score(vocab, [x], x, ids)
    assert int(path.flags.item()) == 0
    for got in (path.logp_t, path.logp_s):
        for y, at in ((0.0, slice(0, n - 1, 2)), (1.0, slice(1, n - 1, 2))):
            want = y - math.log(vocab - 1 + math.e)
            assert float((got[at] - want).abs().max()) <= 2e-5
        assert abs(float(got[n - 1]) - (0.0 - math.log(vocab - 1 + math.exp(2.0)))) <= 2e-5


def test_gradient():
    import torch
    import paper_2609_14636_amd as P
    n, vocab = (1 << 24) + 3, 2056          # four wavefronts each
    s = torch.zeros((n, vocab), dtype=torch.bfloat16, device="cuda")
    grad = torch.full_like(s, 7.0)
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    lay = _one_turn(n)
    lp = torch.full((n,), -math.log(vocab), device="cuda")
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(P.stride_workspace_size(lay, P.STRIDE_UNIT_TURN), dtype=torch.uint8, device="cuda")
    P.stride_opd_grad(lay, P.STRIDE_UNIT_TURN, vocab, s, ids, lp + 1.0, lp, None, None, 1.0, grad, None, flags, ws)
    assert int(flags.item()) == 0
    want = torch.tensor([1.0 / vocab - 1.0, 1.0 / vocab], device="cuda")
    for col in (0, 1, vocab - 1):
        g = grad[:, col].float()
        assert float((g - want[min(col, 1)]).abs().max()) <= 2.0 ** -8 * float(want[min(col, 1)].abs())


def test_turn_means():
    import torch
    import paper_2609_14636_amd as P
    T = (1 << 24) + 3                       # 256 threads each
    x = torch.zeros((T, 8), dtype=torch.bfloat16, device="cuda")
    x[:, 0] = torch.arange(T, device="cuda") % 7
    lay = P.Layout(torch.tensor([0, T], dtype=torch.int32, device="cuda"),
                   torch.arange(T + 1, dtype=torch.int64, device="cuda"), T)
    path = P.Path(lay, P.STRIDE_UNIT_TURN, with_student=False)
    path.turn_mean.fill_(9.0)
    path.score(8, [x], None, torch.zeros(T, dtype=torch.int32, device="cuda"))
    assert int(path.flags.item()) == 0
    assert torch.equal(path.turn_mean, path.logp_t.double())


def _restart(sizes, vals, lay, per, alpha):
    import torch
    import paper_2609_14636_amd as P
    out = [torch.full((sizes,), 77, dtype=torch.int32, device="cuda") for _ in range(3)]
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    P.stride_restart_turn(lay, P.STRIDE_UNIT_TOKEN, vals, None, [alpha], None, *out, flags)
    assert int(flags.item()) == 0
    return out


@pytest.mark.parametrize("R,per", [((1 << 23) + 3, 1025), ((1 << 24) + 3, 130)])
def test_restart_pick(R, per):
    """512 and 256 threads each."""
    import torch
    import paper_2609_14636_amd as P
    vals = torch.full((R, per), -1.0, device="cuda")
    vals[:, 7] = -1.5
    vals[R - 1, 3] = -3.0
    off = torch.arange(R + 1, dtype=torch.int64, device="cuda") * per
    lay = P.Layout(torch.arange(R + 1, dtype=torch.int32, device="cuda"), off, R * per)
    out = _restart(R, vals, lay, per, -2.0)
    for got, most, last in zip(out, (7, 7, per), (0, 0, 3)):
        assert int(got[R - 1]) == last and (got[:R - 1] == most).all()


def test_short_rollouts():
    """64 threads each: the restart pick and the online stop test."""
    import torch
    import paper_2609_14636_amd as P
    R = (1 << 26) + 5
    vals = torch.full((R,), -1.0, device="cuda")
    vals[R - 2] = -3.0
    off = torch.arange(R + 1, dtype=torch.int64, device="cuda")
    lay = P.Layout(torch.arange(R + 1, dtype=torch.int32, device="cuda"), off, R)
    ks, k0, km = _restart(R, vals, lay, 1, -2.0)
    assert int(km.sum()) == R - 1 and int(km[R - 2]) == 0 and int(ks.sum()) == -1 and not k0.any()
    cum = torch.zeros(R, dtype=torch.float64, device="cuda")
    units = torch.zeros(R, dtype=torch.int32, device="cuda")
    stop = torch.full((R,), -1, dtype=torch.int32, device="cuda")
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    P.stride_stop_step(torch.arange(R, dtype=torch.int32, device="cuda"), off, P.STRIDE_UNIT_TOKEN, vals, None,
                       [-2.0], cum, units, stop, flags)
    assert int(flags.item()) == 0
    assert torch.equal(cum, vals.double()) and (units == 1).all()
    assert int(stop[R - 2]) == 0 and int(stop.sum()) == -(R - 1)


def test_fused_tiles():
    import torch
    import paper_2609_14636_amd as P
    n, vocab, d = (1 << 23) + 300, 65536, 64    # 32,770 x 256 tiles of 512 threads
    g = torch.Generator(device="cuda").manual_seed(3)
    h = torch.empty((n, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    w = torch.empty((vocab, d), dtype=torch.bfloat16, device="cuda").normal_(0, 0.3, generator=g)
    ids = torch.randint(0, vocab, (n,), dtype=torch.int32, device="cuda", generator=g)
    path = P.Path(_one_turn(n), P.STRIDE_UNIT_TURN, with_student=False, fused_vocab=vocab)
    path.fused_ws.fill_(0xFF)
    path.score_fused(vocab, h, w, None, ids)
    assert int(path.flags.item()) == 0
    assert torch.isfinite(path.logp_t).all()
    at = torch.cat([torch.arange(0, n, n // 50, device="cuda"), torch.arange(n - 300, n, 7, device="cuda")])
    z = h[at].double() @ w.double().t()
    want = z.gather(1, ids[at].long().unsqueeze(1)).squeeze(1) - torch.logsumexp(z, 1)
    assert float((path.logp_t[at].double() - want).abs().max()) <= 2e-3
