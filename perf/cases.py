"""The work a user has the library do, as timed cases: control ticks from the
smallest call to a million candidates, the many-loop service, the learned
proposal's ticks and training, the separable calls, the lifted form and the
model refit.

Sizes are those of the workloads the repository's benchmark and tests run
(balance bot, race car, three-input car, 64 mixed loops, 2,048 proposals,
batch 4,096) and generic ones beside them.  Every input follows from the
seed; the fitted models follow from fixed synthetic data, as a deployed
controller's model does.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1906_02318_amd import mpmi
from paper_1906_02318_amd.proposal import LearnedTicker, ProposalNet

# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
# kind      what one pass is
# tick      one fused control tick: record, and first violations with "fv"
# loops     one tick of many loops, served as a graph replay
# learned   network forward, proposals, tick over them, gated fallback
# train     one training step: gradient, then Adam
# stages    rollout_batch, safe_mask, select_min_intervention
# lifted    one tick with lifted whole-horizon predictions
# refit     the re-lifting model and the lifted operator from transitions


def listed():
    return [
        # The smallest call: 1,024 held inputs of the balance bot, 20 steps ahead.
        _tick("bot_grid_1k", "bot", "grid", 1024, 20, 1, "fp32", fv=True),
        # The balance bot at its real-time size: 10,240 five-segment sequences, in the
        # launch shape its control loop keeps.
        _tick("bot_sequences_10k", "bot", "uniform", 10240, 50, 5, "fp32", fv=False, block=256, lanes=4),
        # The race car at its stated size, decisions those of FP64 rollouts, verdicts read back.
        _tick("car_grid_16k", "car", "grid", 16384, 60, 1, "recheck64", fv=True),
        # The largest tick, the headline: a million race-car candidates, FP64 decisions.
        _tick("car_grid_1m", "car", "grid", 1048576, 60, 1, "recheck64", fv=False),
        # The paper's three-input car on a basis given as data: 22 x 23 x 20 points, 25 steps.
        _tick("car3_grid_10k", "car3", "grid", 10120, 25, 1, "fp32", fv=True),
        # 64 mixed loops of uneven size served by one graph replay per tick.
        {"name": "loops_64", "kind": "loops", "n": 64, "n_lo": 1024, "n_hi": 65536, "h_lo": 20, "h_hi": 60},
        # The learned tick that replaces an exhaustive one: 2,048 proposals, gated 128 x 128 fallback.
        {"name": "learned_2k", "kind": "learned", "n": 2048, "h": 60, "lanes": 8, "block": 256},
        # A training step of the proposal network at its own batch, and at the largest batch.
        {"name": "train_4096", "kind": "train", "n": 4096},
        {"name": "train_65536", "kind": "train", "n": 65536},
        # The separable calls with the cloud kept, at a ragged size.
        {"name": "stages_250k", "kind": "stages", "n": 250047, "h": 60},
        # The million-candidate tick with lifted predictions.
        {"name": "lifted_1m", "kind": "lifted", "n": 1048576, "h": 60},
        # Learning both operators of the race car from 50,000 transitions.
        {"name": "refit_50k", "kind": "refit", "n": 50000},
    ]


def _tick(name, system, gen, n, h, s, precision, fv, block=0, lanes=0):
    return {"name": name, "kind": "tick", "system": system, "gen": gen, "n": n, "h": h, "s": s,
            "precision": precision, "fv": fv, "block": block, "lanes": lanes}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bot", "bot", "car", "car", "car3", "loops", "learned", "train", "train", "stages", "lifted",
                       "refit"])
    c = None
    if kind == "bot":
        gen = rng.choice(["grid", "uniform", "explicit"])
        s = 1 if gen == "grid" else rng.choice([1, 2, 3, 5, 8])
        c = _tick("", "bot", gen, _log_int(rng, 256, 131072), rng.randint(15, 100), s,
                  rng.choice(["fp32", "recheck64"]), rng.random() < 0.5)
    elif kind == "car":
        gen = rng.choice(["grid", "uniform", "explicit"])
        s = 1 if gen == "grid" else rng.choice([1, 2, 4])
        c = _tick("", "car", gen, _log_int(rng, 1024, 900000), rng.randint(20, 60), s,
                  rng.choice(["fp32", "recheck64", "recheck64"]), rng.random() < 0.5)
    elif kind == "car3":
        c = _tick("", "car3", rng.choice(["grid", "uniform"]), _log_int(rng, 1000, 60000), rng.randint(15, 60), 1,
                  rng.choice(["fp32", "recheck64"]), rng.random() < 0.5)
    elif kind == "loops":
        c = {"name": "", "kind": "loops", "n": _log_int(rng, 8, 128), "n_lo": 512, "n_hi": 32768,
             "h_lo": rng.randint(15, 25), "h_hi": rng.randint(40, 60)}
    elif kind == "learned":
        c = {"name": "", "kind": "learned", "n": _log_int(rng, 256, 8192), "h": rng.randint(30, 60),
             "lanes": rng.choice([1, 2, 4, 8]), "block": 256}
    elif kind == "train":
        c = {"name": "", "kind": "train", "n": _log_int(rng, 200, 65536)}
    elif kind == "stages":
        c = {"name": "", "kind": "stages", "n": _log_int(rng, 2000, 400000), "h": rng.randint(20, 60)}
    elif kind == "lifted":
        c = {"name": "", "kind": "lifted", "n": _log_int(rng, 16384, 1000000), "h": rng.randint(20, 60)}
    else:
        c = {"name": "", "kind": "refit", "n": _log_int(rng, 2000, 60000)}
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Plants, track and models (fixed data)
# ---------------------------------------------------------------------------
def _rk4(f, x, u, dt):
    k1 = f(x, u)
    k2 = f(x + 0.5 * dt * k1, u)
    k3 = f(x + 0.5 * dt * k2, u)
    k4 = f(x + dt * k3, u)
    return x + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)


def _cartpole(x, u):
    """Frictionless cart-pole, rows [p, p', theta, theta'], force u."""
    s, c = np.sin(x[:, 2]), np.cos(x[:, 2])
    a = (u[:, 0] + 0.1 * x[:, 3] ** 2 * s) / 1.2
    thdd = (9.81 * s - c * a) / (0.5 * (4.0 / 3.0 - 0.2 * c * c / 1.2))
    return np.stack([x[:, 1], a - 0.1 * thdd * c / 1.2, x[:, 3], thdd], axis=1)


def _bicycle(x, u):
    """Dynamic bicycle with saturated linear tyres, rows [x, y, psi, vx, vy, r], u = [delta, a]."""
    m, iz, lf, lr, cf = 1500.0, 2500.0, 1.2, 1.4, 5.0e4
    psi, vx, vy, r = x[:, 2], x[:, 3], x[:, 4], x[:, 5]
    d, a = u[:, 0], u[:, 1]
    v = np.maximum(vx, 1.0)
    ff, fr = m * 9.81 * lr / (lf + lr), m * 9.81 * lf / (lf + lr)
    fy = np.clip(cf * (d - np.arctan((vy + lf * r) / v)), -ff, ff)
    ry = np.clip(-cf * np.arctan((vy - lr * r) / v), -fr, fr)
    return np.stack([vx * np.cos(psi) - vy * np.sin(psi), vx * np.sin(psi) + vy * np.cos(psi), r,
                     a - fy * np.sin(d) / m + vy * r, (fy * np.cos(d) + ry) / m - vx * r,
                     (lf * fy * np.cos(d) - lr * ry) / iz], axis=1)


@functools.lru_cache(maxsize=None)
def _track():
    phase = np.random.default_rng(3).uniform(0.0, 2.0 * math.pi, size=4).astype(np.float32)
    amp = np.array([2.0, 1.0, 2.0 / 3.0, 0.5], np.float32)
    return dict(r0=30.0, half=3.0, amp=[float(v) for v in amp], freq=[2, 3, 4, 5], phase=[float(v) for v in phase],
                infl=0.0)


def _car_states(rng, n, offset, psi_sd, vx, vy, r):
    """States on the track: radial offset uniform, heading the tangent's plus noise, speeds uniform."""
    t = _track()
    phi = rng.uniform(0.0, 2.0 * math.pi, size=n)
    rc = t["r0"] + sum(a * np.sin(f * phi + p) for a, f, p in zip(t["amp"], t["freq"], t["phase"]))
    drc = sum(a * f * np.cos(f * phi + p) for a, f, p in zip(t["amp"], t["freq"], t["phase"]))
    rho = rc + rng.uniform(-offset, offset, size=n)
    psi = np.arctan2(drc * np.sin(phi) + rc * np.cos(phi), drc * np.cos(phi) - rc * np.sin(phi))
    return np.stack([rho * np.cos(phi), rho * np.sin(phi), psi + psi_sd * rng.standard_normal(n),
                     rng.uniform(*vx, size=n), rng.uniform(*vy, size=n), rng.uniform(*r, size=n)], axis=1)


def _car_transitions(rng, n, inputs=2):
    X = _car_states(rng, n, 3.5, 0.4, (2.0, 18.0), (-1.5, 1.5), (-0.8, 0.8))
    lo, hi = (np.array([-0.4, -3.0]), np.array([0.4, 3.0])) if inputs == 2 else (
        np.array([-1.0, 0.0, -1.0]), np.array([1.0, 1.0, 0.0]))
    U = lo + (hi - lo) * rng.uniform(size=(n, inputs))
    u = U if inputs == 2 else np.stack([0.4 * U[:, 0], 3.0 * (U[:, 1] + U[:, 2])], axis=1)
    Y = _rk4(_bicycle, X, u, 1.0 / 60.0)
    Y[:, 3] = np.maximum(Y[:, 3], 0.0)
    return X, U, Y


def _bot_states(rng, n):
    return rng.uniform([-1.5, -1.0, -0.3, -1.0], [1.5, 1.0, 0.3, 1.0], size=(n, 4))


def _bot_transitions(rng, n):
    X = rng.uniform([-3.0, -3.0, -0.8, -3.0], [3.0, 3.0, 0.8, 3.0], size=(n, 4))
    U = rng.uniform(-5.0, 5.0, size=(n, 1))
    return X, U, _rk4(_cartpole, X, U, 0.01)


def _quad(w):
    return [w[k] * w[l] for k in range(len(w)) for l in range(k, len(w))]


def _psi(system, x, u):
    """Features of rows [x; u], in the library's documented order (torch or numpy columns)."""
    trig = torch if isinstance(x, torch.Tensor) else np
    w = [x[:, j] for j in range(x.shape[1])] + [u[:, j] for j in range(u.shape[1])]
    one = w[0] * 0.0 + 1.0
    if system == "bot":
        f = [one] + w + _quad(w)
    elif system == "car":
        sp, cp, sd, cd = trig.sin(w[2]), trig.cos(w[2]), trig.sin(w[6]), trig.cos(w[6])
        vx, vy, r, a = w[3], w[4], w[5], w[7]
        f = [one] + w + _quad(w) + [sp, cp, sd, cd, sp * vx, sp * vy, sp * r, sp * a, cp * vx, cp * vy, cp * r, cp * a,
                                    sd * vx, sd * vy, sd * r, cd * vx, cd * vy, cd * r, a * sd]
    else:
        val = {"one": lambda v: one, "var": lambda v: w[v], "sin": lambda v: trig.sin(w[v]),
               "cos": lambda v: trig.cos(w[v])}
        at = [val[k](v) for k, v in _car3_basis()[0]]
        f = [at[p] * at[q] for p, q in _car3_basis()[1]]
    return trig.stack(f, 1)


def _car3_basis():
    """64 features of the three-input car as products of atoms of [x, y, psi, vx, vy, r, heading, gas, brake]."""
    atoms = [("one", 0)] + [("var", k) for k in range(9)] + [("sin", 2), ("cos", 2), ("sin", 6), ("cos", 6)]
    w, sp, cp, sh, ch = list(range(1, 10)), 10, 11, 12, 13
    f = [(0, 0)] + [(k, 0) for k in w]
    f += [(w[k], w[l]) for k in range(6) for l in range(k, 6)] + [(w[k], w[l]) for k in range(6, 9) for l in range(k, 9)]
    f += [(w[3], w[6]), (w[4], w[6]), (w[5], w[6]), (w[3], w[7]), (w[3], w[8]), (sp, 0), (cp, 0), (sh, 0), (ch, 0)]
    f += [(t, w[k]) for t in (sp, cp) for k in (3, 4, 5)] + [(t, w[k]) for t in (sp, cp) for k in (7, 8)]
    f += [(t, w[k]) for t in (sh, ch) for k in (3, 4, 5)] + [(w[7], sh), (w[8], sh)]
    return atoms, f


def _lstsq(P, Y):
    s = np.sqrt(np.mean(P * P, axis=0))
    return np.linalg.lstsq(P / s, Y, rcond=None)[0] / s[:, None]


_SHAPE = {"bot": (4, 1), "car": (6, 2), "car3": (6, 3)}


@functools.lru_cache(maxsize=None)
def _fitted(system, lifted=False):
    """FP64 least-squares operator of a plant from fixed transitions (rows = features)."""
    rng = np.random.default_rng({"bot": 100, "car": 200, "car3": 300}[system])
    X, U, Y = _bot_transitions(rng, 5000) if system == "bot" else _car_transitions(rng, 20000, _SHAPE[system][1])
    return _lstsq(_psi(system, X, U), _psi(system, Y, U) if lifted else Y)


@functools.lru_cache(maxsize=None)
def _context():
    return mpmi.Context(0)


def _system(system):
    if system == "bot":
        return mpmi.balance_bot_system()
    if system == "car":
        return mpmi.race_car_system(_track())
    atoms, feats = _car3_basis()
    return mpmi.custom_system(6, 3, atoms, feats, [(4, 2.0, 0.0)], (-1.0, 0.0, -1.0), (1.0, 1.0, 0.0), track=_track(),
                              eps_box=[0.02], eps_track=0.02, eps32_box=[3e-4], eps32_track=2e-3)


def _model(system):
    return mpmi.mpmi_model_pack(_context(), _system(system), torch.tensor(_fitted(system), device="cuda"))


def _situation(system, seed):
    """A held-out state and the user's input at it."""
    rng = np.random.default_rng([seed, 1])
    s = _system(system)
    m = _SHAPE[system][1]
    x = _bot_states(rng, 1)[0] if system == "bot" else _car_states(rng, 1, 2.0, 0.2, (5.0, 15.0), (-0.5, 0.5),
                                                                  (-0.3, 0.3))[0]
    u = np.array([rng.uniform(s.u_lo[j], s.u_hi[j]) for j in range(m)])
    return _f32(x), _f32(u)


def _f32(v):
    return torch.tensor(np.ascontiguousarray(v), dtype=torch.float32, device="cuda")


def _grid(n, m):
    """Points per input whose product is at most n, near equal; the last takes what is left."""
    if n == 10120 and m == 3:
        return [22, 23, 20]
    g, left = [], n
    for j in range(m - 1):
        g.append(max(1, int(round(left ** (1.0 / (m - j))))))
        left //= g[-1]
    return g + [max(1, left)]


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
_GEN = {"grid": mpmi.GEN_GRID, "uniform": mpmi.GEN_UNIFORM, "explicit": mpmi.GEN_EXPLICIT}
_PREC = {"fp32": mpmi.PREC_FP32, "recheck64": mpmi.PREC_FP32_RECHECK64}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


def _prepare_tick(case, seed):
    model = _model(case["system"])
    x, u = _situation(case["system"], seed)
    m = model.m
    n, grid, cand = case["n"], None, None
    if case["gen"] == "grid":
        grid = _grid(n, m)
        n = int(np.prod(grid))
    elif case["gen"] == "explicit":
        lo, hi = _f32(list(model.system.u_lo)[:m]), _f32(list(model.system.u_hi)[:m])
        g = torch.Generator(device="cuda").manual_seed(seed)
        r = torch.rand((case["s"], m, n), device="cuda", generator=g)
        cand = (lo[None, :, None] + (hi - lo)[None, :, None] * r).contiguous()
    d = mpmi.tick_desc(n, case["h"], gen=_GEN[case["gen"]], grid=grid, n_seg=case["s"], seed=seed, tick=0,
                       precision=_PREC[case["precision"]], block=case["block"], lanes_per_cand=case["lanes"])
    return dict(run=_run_tick, model=model, x=x, u=u, cand=cand, desc=d,
                out=torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda"),
                fv=torch.zeros(n + 1, dtype=torch.int16, device="cuda") if case["fv"] else None)


def _run_tick(st):
    mpmi.mpmi_tick(_context(), st["model"], st["desc"], st["x"], st["u"], cand=st["cand"], out=st["out"],
                   first_violation=st["fv"])
    st["desc"].tick += 1
    return st["out"] if st["fv"] is None else (st["out"], st["fv"])


def _prepare_loops(case, seed):
    rng = np.random.default_rng([seed, 2])
    n = case["n"]
    sizes = np.random.default_rng(5)  # the served fleet is fixed; the situations are the seed's
    N = np.rint(np.exp(sizes.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), size=n))).astype(int)
    H = sizes.integers(case["h_lo"], case["h_hi"] + 1, size=n)
    nb = n // 2
    models = {k: _model(k) for k in ("bot", "car")}
    x, u = np.zeros((n, 8)), np.zeros((n, 4))
    x[:nb, :4], u[:nb, 0] = _bot_states(rng, nb), rng.uniform(-5.0, 5.0, size=nb)
    x[nb:, :6] = _car_states(rng, n - nb, 2.0, 0.2, (5.0, 15.0), (-0.5, 0.5), (-0.3, 0.3))
    u[nb:, 0], u[nb:, 1] = rng.uniform(-0.4, 0.4, size=n - nb), rng.uniform(-3.0, 3.0, size=n - nb)
    xd, ud = _f32(x), _f32(u)
    out = torch.zeros((n, mpmi.SELECTION_BYTES), dtype=torch.uint8, device="cuda")
    loops = [dict(model=models["bot" if i < nb else "car"], x_t=xd[i], u_user=ud[i], out=out[i], n_cand=int(N[i]),
                  horizon=int(H[i]), gen=mpmi.GEN_UNIFORM, seed=1000 + i) for i in range(n)]
    multi = mpmi.Multi(_context(), loops, block=512)
    multi.capture_graph()
    return dict(run=_run_loops, multi=multi, out=out, keep=(models, xd, ud))


def _run_loops(st):
    st["multi"].launch_graph()
    return st["out"]


def _prepare_learned(case, seed):
    ctx = _context()
    x, u = _situation("car", seed)
    ticker = LearnedTicker(ctx, _model("car"), ProposalNet.load(ctx), proposals=case["n"], horizon=case["h"],
                           lanes_per_cand=case["lanes"], block=case["block"])
    return dict(run=_run_learned, ticker=ticker, x=x, u=u, k=seed % 1000,
                out=torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda"))


def _run_learned(st):
    st["k"] += 1
    st["ticker"].tick(st["x"], st["u"], st["k"], out=st["out"])
    return {"record": st["out"], "head": st["ticker"].head, "proposals": st["ticker"].cand}


_LAYERS = [(8, 256), (256, 256), (256, 256), (256, 80)]


def _train_inputs(case, seed):
    """A training state part of the way through, and one batch of (state, user input) -> chosen input."""
    rng = np.random.default_rng([seed, 3])
    B = case["n"]
    parts = []
    for k, n in _LAYERS:
        parts += [rng.uniform(-1.0, 1.0, size=k * n) / math.sqrt(k), 0.05 * rng.standard_normal(n)]
    flat = np.concatenate(parts)
    X = _car_states(rng, B, 3.0, 0.3, (3.0, 17.0), (-1.0, 1.0), (-0.5, 0.5))
    un = rng.uniform(-1.0, 1.0, size=(B, 2))
    X = np.concatenate([X, un * [0.4, 3.0]], axis=1).astype(np.float32)
    T = np.clip(un + 0.2 * rng.standard_normal((B, 2)), -1.0, 1.0).astype(np.float32)
    mean, std = X.mean(axis=0), X.std(axis=0)
    mom = 1e-3 * rng.standard_normal(flat.size)
    vel = 1e-6 * rng.uniform(0.5, 2.0, size=flat.size)
    return flat, X, T, mean, std, mom, vel


def _prepare_train(case, seed):
    ctx = _context()
    flat, X, T, mean, std, mom, vel = _train_inputs(case, seed)
    net = ProposalNet(ctx, flat, mean, std, step=1000, m=mom, v=vel)
    return dict(run=_run_train, net=net, X=_f32(X), T=_f32(T), work=mpmi.mlp_workspace(ctx, case["n"]),
                grad=torch.empty(mpmi.MLP_PARAMS, device="cuda"), loss=torch.empty(1, device="cuda"))


def _run_train(st):
    ctx, net = _context(), st["net"]
    mpmi.mlp_grad(ctx, net.w16, net.w32, net.mean, net.std, st["X"], st["T"], work=st["work"], grad=st["grad"],
                  loss=st["loss"])
    net.step += 1
    mpmi.mlp_adam(ctx, net.w32, net.w16, net.m, net.v, st["grad"], net.step, 1e-3)
    return {"grad": st["grad"], "loss": st["loss"], "w32": net.w32, "w16": net.w16, "m": net.m, "v": net.v}


def _stage_inputs(case, seed):
    """State, user input and held candidate inputs (1, 2, Nc), the user's first."""
    x, u = _situation("car", seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    cand = (_f32([0.4, 3.0])[:, None] * (2.0 * torch.rand((2, case["n"]), device="cuda", generator=g) - 1.0))[None]
    cand[0, :, 0] = u
    return x, u, cand.contiguous()


def _prepare_stages(case, seed):
    x, u, cand = _stage_inputs(case, seed)
    return dict(run=_run_stages, model=_model("car"), x=x, u=u, cand=cand, h=case["h"],
                traj=mpmi.new_traj(_context(), case["h"], 6, case["n"]))


def _run_stages(st):
    ctx = _context()
    traj = mpmi.rollout_batch(ctx, st["model"], st["x"], st["cand"], st["h"], traj=st["traj"])
    fv, margin = mpmi.safe_mask(ctx, st["model"], traj)
    rec = mpmi.select_min_intervention(ctx, st["model"], st["cand"], fv, st["h"], st["u"])
    return {"traj": traj, "fv": fv, "margin": margin, "record": rec}


def _prepare_lifted(case, seed):
    ctx, model = _context(), _model("car")
    x, u = _situation("car", seed)
    lift = mpmi.mpmi_lifted_pack(ctx, model, torch.tensor(_fitted("car", True), device="cuda"), case["h"])
    grid = _grid(case["n"], 2)
    d = mpmi.tick_desc(int(np.prod(grid)), case["h"], gen=mpmi.GEN_GRID, grid=grid)
    return dict(run=_run_lifted, lift=lift, x=x, u=u, desc=d,
                out=torch.zeros(mpmi.SELECTION_BYTES, dtype=torch.uint8, device="cuda"),
                fv=torch.zeros(d.n_cand + 1, dtype=torch.int16, device="cuda"))


def _run_lifted(st):
    mpmi.mpmi_tick_lifted(_context(), st["lift"], st["desc"], st["x"], st["u"], out=st["out"],
                          first_violation=st["fv"])
    return st["out"], st["fv"]


def _prepare_refit(case, seed):
    X, U, Y = _car_transitions(np.random.default_rng([seed, 4]), case["n"])
    d = [torch.tensor(v, device="cuda") for v in (X, U, Y)]
    return dict(run=_run_refit, system=_system("car"), data=d)


def _run_refit(st):
    K, cond = mpmi.koopman_fit(_context(), st["system"], *st["data"])
    Kl, _ = mpmi.koopman_fit_lifted(_context(), st["system"], *st["data"])
    return {"K": K, "lifted": Kl, "cond": cond}


_PREPARE = {"tick": _prepare_tick, "loops": _prepare_loops, "learned": _prepare_learned, "train": _prepare_train,
            "stages": _prepare_stages, "lifted": _prepare_lifted, "refit": _prepare_refit}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
# FP32 operations of one predicted, checked state: psi^T K on the basis'
# state-dependent features plus the safety test.  Ticks may stop a candidate
# at its first unsafe state; the counts take the whole horizon.
_STEP_FLOPS = {"bot": 187, "car": 860, "car3": 880}


def work(case):
    k, n, h = case["kind"], case["n"], case.get("h", 0)
    if k == "tick":
        io = 48 + (2 * (n + 1) if case["fv"] else 0)
        if case["gen"] == "explicit":
            io += 4 * n * case["s"] * _SHAPE[case["system"]][1]
        return {"bytes": io + 8 * 64 * 6, "flops": (n + 1) * h * _STEP_FLOPS[case["system"]]}
    if k == "loops":
        sizes = np.random.default_rng(5)
        N = np.rint(np.exp(sizes.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), size=n)))
        H = sizes.integers(case["h_lo"], case["h_hi"] + 1, size=n)
        f = np.where(np.arange(n) < n // 2, _STEP_FLOPS["bot"], _STEP_FLOPS["car"])
        return {"bytes": n * (48 + 48), "flops": float(np.sum((N + 1) * H * f))}
    if k == "learned":
        return {"bytes": 2 * 154448 + 8 * n, "flops": 2 * 153600 + (n + 1) * h * _STEP_FLOPS["car"]}
    if k == "train":
        return {"bytes": n * 40 + 154448 * (2 + 4 + 4 + 3 * 8 + 2), "flops": 2 * n * (3 * 153600 - 2048)}
    if k == "stages":
        return {"bytes": n * h * 24 * 2 + n * (8 + 2 + 4 + 2 + 8), "flops": n * h * _STEP_FLOPS["car"]}
    if k == "lifted":
        return {"bytes": 2 * n, "flops": n * h * (72 + 40)}
    # refit: the Gram matrix (half of it is symmetric), its right-hand sides and the two solves
    return {"bytes": 2 * n * 14 * 8 + 64 * 70 * 8, "flops": n * (64 * 65 + 2 * 64 * 70) + 2 * 64 ** 3}


# ---------------------------------------------------------------------------
# The same in 64 bits, without the library
# ---------------------------------------------------------------------------
def exact(case, seed):
    if case["kind"] == "stages":
        return {"traj": _exact_rollout(case, seed), "fv": None, "margin": None, "record": None}
    if case["kind"] == "train":
        g, loss = _exact_gradient(case, seed)
        return {"grad": g, "loss": loss, "w32": None, "w16": None, "m": None, "v": None}
    if case["kind"] == "refit":
        X, U, Y = _car_transitions(np.random.default_rng([seed, 4]), case["n"])
        P = _psi("car", X, U)
        K = _lstsq(P, np.concatenate([Y, _psi("car", Y, U)], axis=1))
        s = np.linalg.svd(P / np.sqrt(np.mean(P * P, axis=0)), compute_uv=False)
        return {"K": K[:, :6].copy(), "lifted": K[:, 6:].copy(), "cond": float(s[0] / s[-1])}
    return None


def _exact_rollout(case, seed):
    x, _, cand = _stage_inputs(case, seed)
    U = cand[0].double().T
    K = torch.tensor(_fitted("car"), device="cuda")
    s = x.double().expand(case["n"], 6)
    out = torch.empty((case["h"], 6, case["n"]), dtype=torch.float64, device="cuda")
    for k in range(case["h"]):
        s = _psi("car", s, U) @ K
        out[k] = s.T
    return out


def _exact_gradient(case, seed):
    """Mean mixture NLL and its gradient: BF16 weights and FP32 biases as given, everything else in 64 bits."""
    flat, X, T, mean, std, _, _ = _train_inputs(case, seed)
    w32 = torch.tensor(flat.astype(np.float32), device="cuda")
    w16 = w32.to(torch.bfloat16).double()
    Xd, Td = torch.tensor(X, device="cuda").double(), torch.tensor(T, device="cuda").double()
    h = (Xd - torch.tensor(mean, device="cuda").double()) / torch.tensor(std, device="cuda").double()
    p, o = [], 0
    for k, n in _LAYERS:
        p.append(w16[o:o + k * n].reshape(k, n).clone().requires_grad_(True))
        p.append(w32[o + k * n:o + k * n + n].double().clone().requires_grad_(True))
        o += k * n + n
    for i in range(4):
        h = h @ p[2 * i] + p[2 * i + 1]
        if i < 3:
            h = torch.nn.functional.gelu(h, approximate="tanh")
    y = h.reshape(-1, 16, 5)
    ls = y[..., 3:5].clamp(-7.0, 2.0)
    dz = (Td[:, None, :] - y[..., 1:3]) * torch.exp(-ls)
    lp = torch.log_softmax(y[..., 0], dim=1) - 0.5 * (dz * dz).sum(-1) - ls.sum(-1) - math.log(2.0 * math.pi)
    loss = -torch.logsumexp(lp, dim=1).mean()
    g = torch.autograd.grad(loss, p)
    return torch.cat([v.reshape(-1) for v in g]), loss.detach().reshape(1)
