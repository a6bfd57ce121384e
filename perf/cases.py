"""The work that users of this package have it do on one GPU, as cases that a timing program can
prepare, run and check.

A case is a dict of plain values.  Its ``kind`` says which calls a pass makes:

  step    ``Path.run``: score every row with the teacher(s) and the student, per-turn means, the
          early stop and the restart pick, for a batch of whole rollouts;
  train   the same calls followed by the OPD loss and gradient of the retained rows;
  fused   the step with the teacher's logits formed inside the kernel from its hidden states;
  online  the rows that active rollouts have just produced are scored and the online stop test
          takes the new units, as a generation loop does after each turn;
  sweep   stop and restart alone on values scored earlier, as for another threshold.

Logits are normal draws with a boost at the sampled token, hidden states and lm_head weights are
normal draws: the shapes and distributions of ``synth/workloads.py``, drawn here by torch.
"""
import math
import random

import numpy as np
import torch

import paper_2609_14636_amd as P

V_FULL = 151936
BASE = dict(kind="step", rollouts=8, turns=1, tok_lo=8, tok_hi=8, vocab=V_FULL, pad=0,
            dtype="bf16", unit="turn", teachers=1, student=True, exact_kl=False, masked=False,
            prefix=False, d=0, graph=False)


def listed():
    return [dict(BASE, **c) for c in (
        # A generation loop's call: 8 active rollouts have just produced a turn of 8 tokens; the
        # teacher scores them and the stop test advances.  The smallest call there is.
        dict(name="online_turn_64", kind="online", student=False),
        # The smallest whole step, 64 rows, as a program replays it: captured once in a HIP graph.
        dict(name="step_graph_64", graph=True),
        # A small batch of short ragged turns issued call by call.
        dict(name="step_ragged_2k", rollouts=5, turns=9, tok_lo=9, tok_hi=89, masked=True),
        # The agentic workload in full: 16 rollouts of 12 turns of 128 to 768 tokens.
        dict(name="step_agentic", rollouts=16, turns=12, tok_lo=128, tok_hi=768, masked=True),
        # Long single-turn rollouts with token units, as in the reasoning workload.
        dict(name="step_reasoning", rollouts=4, tok_lo=16384, tok_hi=16384, unit="token"),
        # Two teachers, each rollout's rows routed to its domain's teacher; part of each rollout
        # is a reused prefix.
        dict(name="step_multi", rollouts=8, turns=8, tok_lo=256, tok_hi=256, teachers=2,
             masked=True, prefix=True),
        # The exact reverse KL beside the sampled one.
        dict(name="step_exact_kl", rollouts=4, turns=8, tok_lo=31, tok_hi=193, exact_kl=True),
        # float32 logits over a smaller, odd vocabulary with padded rows.
        dict(name="step_f32_32k", rollouts=16, turns=8, tok_lo=8, tok_hi=64, vocab=32003, pad=13,
             dtype="f32", masked=True),
        # One training step: scores, stop, restart, loss and the gradient of the retained rows.
        dict(name="train_bf16", kind="train", rollouts=8, turns=8, tok_lo=64, tok_hi=384),
        # The fused projection on a training batch, with the student's logits given.
        dict(name="fused_16k", kind="fused", rollouts=16, turns=8, tok_lo=128, tok_hi=128, d=2048),
        # The fused projection in a generation loop: a few hundred new rows, teacher only.
        dict(name="online_fused_200", kind="online", rollouts=25, tok_lo=2, tok_hi=14, d=2048,
             student=False),
        # Thresholds tried again on 64 scored rollouts of up to 8,192 tokens, token units.
        dict(name="sweep_tokens_256k", kind="sweep", rollouts=64, tok_lo=33, tok_hi=8192,
             unit="token", prefix=True),
    )]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; none moves more bytes or does more arithmetic than the
    largest listed one of its kind."""
    kind = rng.choice(("step", "step", "step", "train", "fused", "online", "online", "sweep"))
    c = dict(BASE, kind=kind)
    vocab = rng.choice((V_FULL, V_FULL, _log(rng, 1000, V_FULL), _log(rng, 30000, V_FULL)))
    c.update(vocab=vocab, prefix=rng.random() < 0.3, masked=rng.random() < 0.5)
    if kind == "sweep":
        unit = rng.choice(("turn", "token"))
        units, rollouts = _log(rng, 500, 300000), _log(rng, 4, 1000)
        per = max(1, units // rollouts)
        if unit == "token":
            c.update(unit=unit, rollouts=rollouts, tok_lo=max(1, per // 8), tok_hi=2 * per)
        else:
            c.update(unit=unit, rollouts=rollouts, turns=min(per, 64), tok_lo=1, tok_hi=9)
        return c
    if kind == "online":
        rows, rollouts = _log(rng, 16, 1500), _log(rng, 2, 200)
        per = max(1, rows // rollouts)
        c.update(rollouts=rollouts, tok_lo=max(1, per // 2), tok_hi=max(1, per + per // 2),
                 student=False, prefix=False, masked=False, unit=rng.choice(("turn", "token")),
                 d=rng.choice((0, 0, 1024, 2048)))
        if c["d"]:
            c.update(vocab=rng.choice((V_FULL, _log(rng, 30000, V_FULL))))
        return c
    if kind == "fused":
        d = rng.choice((1024, 2048, 4096))
        rows = _log(rng, 200, 16384 * 2048 // max(d, 2048))
        c.update(d=d, student=rng.random() < 0.5, vocab=rng.choice((V_FULL, _log(rng, 30000, V_FULL))))
        most = rows
    else:
        c.update(dtype="f32" if rng.random() < 0.25 else "bf16")
        es = 4 if c["dtype"] == "f32" else 2
        most = min(30000, int(12e9 / (vocab * es * 2)))
        if kind == "step":
            c.update(exact_kl=rng.random() < 0.25, teachers=rng.choice((1, 1, 1, 2, 3)))
            c.update(student=c["exact_kl"] or rng.random() < 0.85)
        else:
            most = min(most, 12000)
        rows = _log(rng, 48, most)
    c.update(unit=rng.choice(("turn", "turn", "token")))
    rollouts = max(1, min(rows // 4, _log(rng, 1, 48)))
    turns = 1 if c["unit"] == "token" and rng.random() < 0.5 else _log(rng, 1, 16)
    turns = max(1, min(turns, rows // rollouts))
    per = max(1, rows // (rollouts * turns))
    c.update(rollouts=rollouts, turns=turns, tok_lo=max(1, per // 3), tok_hi=max(1, 2 * per - max(1, per // 3)))
    ratio = 8 if c["dtype"] == "bf16" else 4
    c.update(pad=(-c["vocab"]) % ratio + rng.choice((0, 0, ratio)))
    c.update(graph=kind == "step" and rows < 1024 and rng.random() < 0.3)
    return c


def _layout(case):
    """Turn offsets [R+1] and row offsets [T+1]: lengths spread over the case's range, the same
    for every seed so that the work of a pass is the case's own."""
    g = random.Random(case["rollouts"] * 7919 + case["turns"])
    n = case["rollouts"] * case["turns"]
    lens = [g.randint(case["tok_lo"], case["tok_hi"]) for _ in range(n)]
    rto = np.arange(0, n + 1, case["turns"], dtype=np.int32)
    return rto, np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


def _esize(case):
    return 4 if case["dtype"] == "f32" else 2


def _ld(case):
    per = 16 // _esize(case)
    ld = case["vocab"] + case["pad"]
    return ld + (-ld) % per


def _mean_logp(case):
    """About the mean teacher log-probability of a row, which the thresholds hang on."""
    if case["d"]:
        return -math.log(case["vocab"]) - 0.5 * case["d"] * 0.02 ** 2
    return 4.0 - math.log(case["vocab"]) - 4.5


def _thresholds(case):
    """(lambda, alpha) per domain: rollouts stop around two thirds of their length; units well
    below the mean are not correct."""
    m = _mean_logp(case)
    units = 12 if case["kind"] == "online" else case["turns"]
    if case["unit"] == "token":
        units *= (case["tok_lo"] + case["tok_hi"]) / 2
    n = case["teachers"]
    lam = [m * units * (0.65 + 0.05 * i) for i in range(n)]
    alpha = -math.inf if case["unit"] == "token" else m - 4.0
    return lam, [alpha] * n


def _logits(g, n, case, ids, boost):
    x = torch.empty((n, _ld(case)), device="cuda",
                    dtype=torch.float32 if case["dtype"] == "f32" else torch.bfloat16)
    x.normal_(0.0, 3.0, generator=g)
    at = ids.long().unsqueeze(1)
    x.scatter_add_(1, at, boost.to(x.dtype).unsqueeze(1))
    return x


def _inputs(case, seed):
    """The tensors a user's program has in hand, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rto, tto = _layout(case)
    n, r = int(tto[-1]), case["rollouts"]
    x = dict(n=n, rto=rto, tto=tto)
    normal = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    units = (tto[rto] if case["unit"] == "token" else rto.astype(np.int64))
    per = torch.from_numpy(np.diff(units)).cuda()
    x["domain"] = None
    if case["teachers"] > 1:
        x["domain"] = torch.randint(0, case["teachers"], (r,), dtype=torch.int32, device="cuda", generator=g)
    x["start"] = None
    if case["prefix"]:  # up to a quarter of the rollout is a reused prefix
        u = torch.rand(r, device="cuda", generator=g, dtype=torch.float64)
        x["start"] = (u * 0.25 * per).to(torch.int32)
    x["mask"] = None
    if case["masked"]:  # a unit in fifty is marked wrong
        x["mask"] = (torch.rand(int(units[-1]), device="cuda", generator=g) < 0.98).to(torch.uint8)
    if case["kind"] == "sweep":
        v = _mean_logp(case) + 3.0 * normal(int(units[-1]))
        x["values"] = v.clamp_(max=0.0) if case["unit"] == "token" else v.double()
        return x
    x["ids"] = torch.randint(0, case["vocab"], (n,), dtype=torch.int32, device="cuda", generator=g)
    if case["d"]:
        x["hidden"] = normal(n, case["d"]).to(torch.bfloat16)
        w = torch.empty((case["vocab"], case["d"]), device="cuda", dtype=torch.bfloat16)
        x["w"] = w.normal_(0.0, 0.02, generator=g)
    else:
        boost = 4.0 + 2.0 * normal(n)
        x["teachers"] = [_logits(g, n, case, x["ids"], boost) for _ in range(case["teachers"])]
    x["student"] = None
    if case["student"]:
        x["student"] = _logits(g, n, case, x["ids"], 5.0 + 2.0 * normal(n))
    if case["kind"] == "online":  # sums that the rollouts' earlier turns left, down to lambda
        x["sums"] = _thresholds(case)[0][0] * torch.rand(r, device="cuda", generator=g, dtype=torch.float64)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    unit = P.STRIDE_UNIT_TOKEN if case["unit"] == "token" else P.STRIDE_UNIT_TURN
    layout = P.Layout(torch.from_numpy(x["rto"]).cuda(), torch.from_numpy(x["tto"]).cuda(), x["n"],
                      x["domain"])
    path = P.Path(layout, unit, with_student=case["student"], exact_kl=case["exact_kl"],
                  fused_vocab=case["vocab"] if case["d"] else None)
    s = dict(case=case, x=x, unit=unit, layout=layout, path=path, graph=None)
    s["lam"], s["alpha"] = _thresholds(case)
    if case["kind"] == "train":
        s["grad"] = torch.zeros_like(x["student"])
        s["loss"] = torch.empty(x["n"], device="cuda")
    if case["kind"] == "online":
        r = case["rollouts"]
        s["slot"] = torch.arange(r, dtype=torch.int32, device="cuda")
        offs = x["tto"] if unit == P.STRIDE_UNIT_TOKEN else np.arange(r + 1, dtype=np.int64)
        s["new_off"] = torch.from_numpy(offs).cuda()
        # per-rollout state in one buffer: sums (float64), units seen and stops (int32)
        s["fresh"] = torch.zeros(16 * r, dtype=torch.uint8, device="cuda")
        s["fresh"][:8 * r].view(torch.float64).copy_(x["sums"])
        s["fresh"][8 * r:12 * r].view(torch.int32).fill_(100)
        s["fresh"][12 * r:].view(torch.int32).fill_(-1)
        s["state"] = s["fresh"].clone()
        s["cum"] = s["state"][:8 * r].view(torch.float64)
        s["seen"] = s["state"][8 * r:12 * r].view(torch.int32)
        s["stop"] = s["state"][12 * r:].view(torch.int32)
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _calls(s)  # once before the capture, as torch asks
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _calls(s)
    return s


def _calls(s):
    case, x, path = s["case"], s["x"], s["path"]
    if case["kind"] == "sweep":
        P.stride_stop(s["layout"], s["unit"], x["values"], s["lam"], x["start"], path.cum,
                      path.stop_unit, path.retained, path.flags, path.ws)
        P.stride_restart_turn(s["layout"], s["unit"], x["values"], path.stop_unit, s["alpha"],
                              x["mask"], path.k_star, path.k0, path.k_max, path.flags)
        return
    if case["kind"] == "online":
        if case["d"]:
            path.score_fused(case["vocab"], x["hidden"], x["w"], None, x["ids"])
        else:
            path.score(case["vocab"], x["teachers"], None, x["ids"])
        s["state"].copy_(s["fresh"])  # the slots' state, as a program sets it for its next rollouts
        P.stride_stop_step(s["slot"], s["new_off"], s["unit"], path.values(), None, s["lam"],
                           s["cum"], s["seen"], s["stop"], path.flags)
        return
    if case["kind"] == "fused":
        path.score_fused(case["vocab"], x["hidden"], x["w"], x["student"], x["ids"])
        path.stop(s["lam"], x["start"])
        path.restart(s["alpha"], x["mask"])
        return
    path.run(case["vocab"], x["teachers"], x["student"], x["ids"], s["lam"], s["alpha"], x["start"],
             x["mask"])
    if case["kind"] == "train":
        path.grad(case["vocab"], x["student"], x["ids"], s["grad"], s["loss"], x["start"],
                  scale=1.0 / x["n"])


_STOPS = ("cum", "stop_unit", "retained", "k_star", "k0", "k_max")
_SCORES = ("logp_t", "logp_s", "kl", "kl_full", "turn_mean")


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _calls(state)
    case, path = state["case"], state["path"]
    names = () if case["kind"] == "sweep" else _SCORES
    if case["kind"] != "online":
        names += _STOPS
    out = {k: getattr(path, k) for k in names if getattr(path, k) is not None}
    out["flags"] = path.flags
    if case["kind"] == "online":
        out.update(state_cum=state["cum"], state_units=state["seen"], stop=state["stop"])
    if case["kind"] == "train":
        out.update(grad=state["grad"], loss=state["loss"])
    return out


def work(case):
    rto, tto = _layout(case)
    n, t, r, es = int(tto[-1]), len(tto) - 1, case["rollouts"], _esize(case)
    units = n if case["unit"] == "token" else t
    row = case["vocab"] * es
    flops, total = 0.0, 8.0 * (t + r)
    if case["kind"] == "sweep":
        return dict(bytes=total + units * (4 + 8 + 4 if case["unit"] == "token" else 24) + 24.0 * r, flops=0.0)
    if case["d"]:
        total += 2.0 * case["d"] * (n + case["vocab"])
        flops += 2.0 * n * case["d"] * case["vocab"]
    else:
        total += float(n) * row
    total += 8.0 * n  # token ids and logp_t
    if case["student"]:
        total += float(n) * (row + 8)
    if case["exact_kl"]:
        total += 4.0 * n
    if case["kind"] == "train":
        total += float(n) * (row + 4)
    if case["kind"] != "online":
        total += 8.0 * units
    return dict(bytes=total, flops=flops)


def tolerance(case):
    if case["kind"] == "sweep":
        return {"rel": 1e-12}  # sums in float64
    if case["kind"] == "train" and case["dtype"] == "bf16":
        return {"rel": 6e-3}   # the gradient is written in the logits' type: 1.4e-3 off 64 bits
    return {"rel": 2e-6}       # sums in float32: up to 2.5e-7 off 64 bits


# ---- the same results in 64 bits, in plain torch and numpy ----

def _row_scores(x, ids, vocab):
    """log softmax at ids and the row log-sum-exp, in float64, by blocks of rows."""
    lp, lse = [], []
    step = max(1, int(2e9 / (vocab * 8)))
    for i in range(0, x.shape[0], step):
        z = x[i:i + step, :vocab].double()
        l = torch.logsumexp(z, dim=1)
        lse.append(l)
        lp.append(z.gather(1, ids[i:i + step].long().unsqueeze(1)).squeeze(1) - l)
    return torch.cat(lp), torch.cat(lse)


def _stops(case, x, values):
    """cum, stop, retained, k_star, k0, k_max of Eq. (5) and Sec. 4.2 from float64 values."""
    rto, tto = x["rto"], x["tto"]
    off = tto[rto] if case["unit"] == "token" else rto.astype(np.int64)
    lam, alpha = _thresholds(case)
    v = values.double().cpu().numpy()
    start = None if x["start"] is None else x["start"].cpu().numpy()
    mask = None if x["mask"] is None else x["mask"].cpu().numpy()
    dom = np.zeros(len(rto) - 1, int) if x["domain"] is None else x["domain"].cpu().numpy()
    cum = np.zeros(len(v))
    outs = [[], [], [], [], []]
    for r in range(len(rto) - 1):
        a, b = off[r], off[r + 1]
        k0 = 0 if start is None else int(start[r])
        w = v[a:b]
        c = np.cumsum(w[k0:])
        cum[a + k0:b] = c
        hit = np.nonzero(c < lam[dom[r]])[0]
        stop = int(hit[0]) + k0 if len(hit) else -1
        end = stop + 1 if stop >= 0 else len(w)
        kept = end - k0 if case["unit"] == "token" else int(tto[a + end] - tto[a + k0])
        ok = w[:end] > alpha[dom[r]]
        if mask is not None:
            ok = ok & (mask[a:a + end] != 0)
        wrong = np.nonzero(~ok)[0]
        km = int(wrong[0]) if len(wrong) else end
        ks = int(np.argmin(w[:km])) if km else -1
        for o, y in zip(outs, (stop, kept, ks, max(ks, 0), km)):
            o.append(y)
    names = ("stop_unit", "retained", "k_star", "k0", "k_max")
    return dict(cum=torch.from_numpy(cum), **{k: torch.tensor(o) for k, o in zip(names, outs)})


def exact(case, seed):
    x = _inputs(case, seed)
    out = dict(flags=None)
    if case["kind"] == "sweep":
        out.update(_stops(case, x, x["values"]))
        return out
    rto, tto, ids, n = x["rto"], x["tto"], x["ids"], x["n"]
    lens = torch.from_numpy(np.diff(tto)).cuda()
    row_turn = torch.repeat_interleave(torch.arange(len(lens), device="cuda"), lens)
    if case["d"]:
        lp = []
        wt = x["w"].double().t()
        step = max(1, int(8e9 / (case["vocab"] * 8)))
        for i in range(0, n, step):
            z = x["hidden"][i:i + step].double() @ wt
            lp.append(_row_scores(z, ids[i:i + step], case["vocab"])[0])
        lt = torch.cat(lp)
        del wt
    else:
        lt, lset = _row_scores(x["teachers"][0], ids, case["vocab"])
        if case["teachers"] > 1:
            rd = x["domain"].long()[row_turn // case["turns"]]
            for d in range(1, case["teachers"]):
                l, s = _row_scores(x["teachers"][d], ids, case["vocab"])
                lt, lset = torch.where(rd == d, l, lt), torch.where(rd == d, s, lset)
    out["logp_t"] = lt
    mean = torch.zeros(len(lens), dtype=torch.float64, device="cuda").index_add_(0, row_turn, lt) / lens
    out["turn_mean"] = mean
    if case["student"]:
        ls, lses = _row_scores(x["student"], ids, case["vocab"])
        out.update(logp_s=ls, kl=ls - lt)
    if case["exact_kl"]:
        kl = torch.empty(n, dtype=torch.float64, device="cuda")
        step = max(1, int(1e9 / (case["vocab"] * 8)))
        rd = [0] * n if case["teachers"] == 1 else rd.tolist()
        for d in range(case["teachers"]):
            rows = torch.tensor([i for i in range(n) if rd[i] == d], device="cuda", dtype=torch.long)
            for at in rows.split(step):
                p = x["student"][at][:, :case["vocab"]].double() - lses[at].unsqueeze(1)
                q = x["teachers"][d][at][:, :case["vocab"]].double() - lset[at].unsqueeze(1)
                kl[at] = (p.exp() * (p - q)).sum(1)
        out["kl_full"] = kl
    values = lt if case["unit"] == "token" else mean
    if case["kind"] == "online":
        off = tto[rto] if case["unit"] == "token" else rto.astype(np.int64)
        v, sums, lam = values.cpu().numpy(), x["sums"].cpu().numpy(), _thresholds(case)[0][0]
        cum, stop = [], []
        for r in range(len(rto) - 1):
            c = sums[r] + np.cumsum(v[off[r]:off[r + 1]])
            hit = np.nonzero(c < lam)[0]
            cum.append(c[hit[0]] if len(hit) else c[-1])
            stop.append(100 + int(hit[0]) if len(hit) else -1)
        out.update(state_cum=torch.tensor(cum), state_units=None, stop=torch.tensor(stop))
        return out
    out.update(_stops(case, x, values))
    if case["kind"] == "train":
        off = tto[rto] if case["unit"] == "token" else rto.astype(np.int64)
        keep = torch.zeros(n, dtype=torch.bool, device="cuda")
        start = np.zeros(len(rto) - 1, int) if x["start"] is None else x["start"].cpu().numpy()
        for r, s in enumerate(out["stop_unit"].tolist()):
            a, b = off[r] + start[r], off[r] + s + 1 if s >= 0 else off[r + 1]
            if case["unit"] == "turn":
                a, b = tto[a], tto[b]
            keep[a:b] = True
        c = torch.where(keep, (lt - ls) / n, torch.zeros_like(lt))
        out["loss"] = -c * ls
        grad = torch.zeros(x["student"].shape, dtype=torch.float64, device="cuda")
        step = max(1, int(1e9 / (case["vocab"] * 8)))
        for i in range(0, n, step):
            p = (x["student"][i:i + step, :case["vocab"]].double() - lses[i:i + step].unsqueeze(1)).exp_()
            grad[i:i + step, :case["vocab"]] = p.mul_(c[i:i + step].unsqueeze(1))
        grad[torch.arange(n, device="cuda"), ids.long()] -= c
        out["grad"] = grad
    return out
