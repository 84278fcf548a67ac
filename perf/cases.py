"""The work that users of this framework have it do, as timed cases.

Every case calls the public entry points of `paper_1811_02512_amd` the way a
program does that solves power flows: analyse a topology once, keep the
handle, then solve.  Kinds:

  newton    Newton-Raphson of one case or a batch of load scenarios
  gradient  the same through torch.autograd, with the gradients
  mixed     grids of different sizes, each with its own analysis, one launch
  screen    N-1 contingency screening (fast decoupled first, the default)
  fdpf      the fast decoupled iteration with shared factors
  estimate  WLS state estimation
  steps     mismatch, Jacobian, factorisation and both solves as separate
            calls (a caller's own Newton loop or sensitivities)
  flows     branch flows of solved states

Grids follow the recipe of the repository's synthetic grids: random points, a
nearest-neighbour tree plus short extra branches up to 1.3 branches a bus, 20 %
PV buses, lognormal load scenarios.  All quantities are float64, the only type
the entry points take.
"""
import functools
import math

import numpy as np
import torch

PQ, PV, SLACK = 1, 2, 3
TOL = 1e-8


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # an operator's study of one small system: launches and latency count
        dict(name="newton_200", kind="newton", n=200, batch=1, spread=0, tail=65536, shunts=False),
        # one case of a large system, shared among 32 CUs as the README shows
        dict(name="newton_10k", kind="newton", n=10000, batch=1, spread=32, tail=65536,
             shunts=False),
        # a planner's load scenarios on a mid-sized system, default launch
        dict(name="newton_2k_x1024", kind="newton", n=2000, batch=1024, spread=0, tail=65536,
             shunts=False),
        # the headline: a large system, 256 scenarios, each with its gradient,
        # in the launch shape that the autotuner picks for it
        dict(name="gradient_10k_x256", kind="gradient", n=10000, batch=256, tail=161792,
             shared_x=True, shunts=False),
        # a training step on a ragged small system, reactances per case, shunts
        dict(name="gradient_487_x33", kind="gradient", n=487, batch=33, tail=65536,
             shared_x=False, shunts=True),
        # a fleet of systems of 500 to 20,000 buses in one launch
        dict(name="mixed_64", kind="mixed", count=64, lo=500, hi=20000, spread=256, tail=161792),
        # a security check: every screened outage of a mid-sized system
        dict(name="screen_2k_x384", kind="screen", n=2000, batch=384, tail=65536),
        # fast decoupled scenarios of a large system
        dict(name="fdpf_10k_x256", kind="fdpf", n=10000, batch=256, tail=161792),
        # one fast decoupled case: the planner's quick look
        dict(name="fdpf_3001", kind="fdpf", n=3001, batch=1, tail=65536),
        # a control room's estimator over telemetry snapshots
        dict(name="estimate_2k_x64", kind="estimate", n=2000, batch=64, tail=65536),
        # a caller's own loop over the linear-algebra entry points
        dict(name="steps_5k_x48", kind="steps", n=5003, batch=48, tail=65536),
        # reporting: flows of every solved scenario
        dict(name="flows_10k_x512", kind="flows", n=10000, batch=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["newton", "newton", "newton", "gradient", "gradient", "mixed", "screen",
                       "fdpf", "estimate", "steps", "flows"])
    if kind == "mixed":
        return dict(kind=kind, count=rng.randint(4, 40), lo=_log_int(rng, 100, 800),
                    hi=_log_int(rng, 1000, 12000), spread=rng.choice([0, 256]),
                    tail=rng.choice([65536, 161792]))
    top = {"estimate": 3000, "screen": 6000}.get(kind, 12000)
    n = _log_int(rng, 60, top)
    # at most what the largest listed case of the kind holds
    cap = {"estimate": 128000, "screen": 760000, "steps": 240000, "flows": 5000000}.get(kind,
                                                                                      2000000)
    most = max(1, min(1024, cap // n))
    batch = 1 if kind in ("newton", "fdpf") and rng.random() < 0.3 else _log_int(rng, 1, most)
    case = dict(kind=kind, n=n, batch=batch)
    if kind == "screen":
        case["batch"] = min(batch, max(1, int(0.2 * n)))
    if kind != "flows":
        case["tail"] = rng.choice([65536, 65536, 114688, 161792])
    if kind == "newton":
        case["spread"] = rng.choice([0, 16, 32]) if batch == 1 else 0
    if kind == "gradient":
        case["shared_x"] = rng.random() < 0.5
    if kind in ("newton", "gradient"):
        case["shunts"] = rng.random() < 0.3
    return case


# ---------------------------------------------------------------------------
# grids and scenarios
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _near(pts, k, earlier):
    """Per point its k nearest others (earlier: its nearest among the points
    before it), in slices of the distance matrix."""
    n, out = len(pts), []
    p = torch.from_numpy(pts).to(_device())
    j = torch.arange(n, device=p.device)
    for i0 in range(0, n, 1024):
        i = j[i0:i0 + 1024]
        d = (p[i, None, 0] - p[None, :, 0]) ** 2 + (p[i, None, 1] - p[None, :, 1]) ** 2
        d[j[None, :] >= i[:, None] if earlier else j[None, :] == i[:, None]] = math.inf
        out.append(d.topk(k, dim=1, largest=False).indices.cpu().numpy())
    return np.concatenate(out)


@functools.lru_cache(maxsize=160)
def _grid(n, shunts=False):
    """Topology, branch data and bus types of the n-bus system; slack at 0."""
    rng = np.random.default_rng(n)
    pts = rng.random((n, 2))
    up = _near(pts, 1, True)[:, 0]
    pairs = {(int(min(i, up[i])), int(max(i, up[i]))) for i in range(1, n)}
    tree = len(pairs)
    near = _near(pts, min(6, n - 1), False)
    cand = sorted({(int(min(i, j)), int(max(i, j))) for i in range(n) for j in near[i]} - pairs)
    extra = rng.permutation(len(cand))[:max(0, int(round(1.3 * n)) - tree)]
    br = np.array(sorted(pairs) + [cand[e] for e in extra], np.int32).reshape(-1, 2)
    m = len(br)
    x = rng.lognormal(math.log(0.05), 0.5, m)
    bus_type = np.full(n, PQ, np.int8)
    bus_type[0] = SLACK
    bus_type[1 + rng.choice(n - 1, max(1, int(round(0.2 * n))) if n > 5 else 0, replace=False)] = PV
    vset = np.ones(n)
    vset[bus_type == PV] = rng.uniform(0.98, 1.05, int((bus_type == PV).sum()))
    ysh = None
    if shunts:
        at = 1 + rng.choice(n - 1, max(1, n // 3), replace=False)
        ysh = np.zeros((n, 2))
        ysh[at, 0] = rng.uniform(0.0, 0.01, len(at))
        ysh[at, 1] = rng.uniform(-0.05, 0.15, len(at))
    return dict(n=n, m=m, tree=tree, pts=pts, f=np.ascontiguousarray(br[:, 0]),
                t=np.ascontiguousarray(br[:, 1]), r=x * rng.uniform(0.05, 0.3, m), x=x,
                b=rng.uniform(0.0, 0.05, m), type=bus_type, vset=vset, ysh=ysh)


def _injections(g, batch, seed):
    """Scheduled P, Q [batch, n]: base loads and generation of the system,
    lognormal load factors per scenario and bus."""
    rng = np.random.default_rng([seed, g["n"], batch])
    n = g["n"]
    Pd = rng.uniform(0.0, 1.0, n) * 0.1
    Qd = Pd * rng.uniform(0.2, 0.5, n)
    gen = np.where(g["type"] == PV, rng.uniform(0.2, 1.0, n), 0.0)
    if gen.sum() > 0:
        gen *= 1.01 * Pd.sum() / gen.sum()
    fac = rng.lognormal(0.0, 0.1, (batch, n))
    return gen - Pd * fac, -Qd * fac


def _put(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(_device())


def _symbolic(g, tail, spread=0):
    from paper_1811_02512_amd import api

    sym = api.Symbolic(g["n"], g["f"], g["t"])
    if tail != 65536:
        sym.set_launch(512, tail, 4)
    if spread:
        sym.set_spread(spread)
    return sym.upload()


def _branches(g):
    return _put(g["r"]), _put(g["x"]), _put(g["b"]), _put(g["ysh"])


def _mixed_sizes(case):
    rng = np.random.default_rng([case["count"], case["lo"], case["hi"]])
    return [int(v) for v in np.round(np.exp(rng.uniform(math.log(case["lo"]),
                                                        math.log(case["hi"]), case["count"])))]


def _states(g, batch, seed):
    """Plausible solved states: |V| near 1, angles falling across the system,
    both smooth along its branches but for a little noise."""
    rng = np.random.default_rng([seed, g["n"], batch, 7])
    across = g["pts"] @ rng.normal(0.0, 0.2, (2, batch))
    wave = np.sin(3.0 * across + rng.uniform(0.0, 6.0, batch))
    Vm = 1.0 + 0.02 * wave.T + rng.normal(0.0, 0.002, (batch, g["n"]))
    Va = (across - across[:1]).T + rng.normal(0.0, 0.002, (batch, g["n"]))
    Va[:, 0] = 0.0
    return Vm, Va


# ---------------------------------------------------------------------------
# power-flow formulas in torch (measurements of the estimator, and exact())
# ---------------------------------------------------------------------------
class _Net:
    """Branch-wise pi-model of one system on the device, fp64."""

    def __init__(self, g):
        self.n, self.m = g["n"], g["m"]
        self.f, self.t = _put(g["f"].astype(np.int64)), _put(g["t"].astype(np.int64))
        self.r, self.x, self.b = _put(g["r"]), _put(g["x"]), _put(g["b"])
        self.ysh = _put(g["ysh"])
        self.type = _put(g["type"])
        self.th = torch.nonzero(self.type != SLACK).flatten()
        self.pq = torch.nonzero(self.type == PQ).flatten()

    def flows(self, Vm, Va, x=None):
        """(Pft, Qft, Ptf, Qtf) of states [..., n]."""
        x = self.x if x is None else x
        den = self.r * self.r + x * x
        g, bs = self.r / den, -x / den
        h = self.b / 2
        vf, vt = Vm[..., self.f], Vm[..., self.t]
        d = Va[..., self.f] - Va[..., self.t]
        c, s = torch.cos(d), torch.sin(d)
        vv = vf * vt
        return (vf * vf * g - vv * (g * c + bs * s), -vf * vf * (bs + h) - vv * (g * s - bs * c),
                vt * vt * g - vv * (g * c - bs * s), -vt * vt * (bs + h) + vv * (g * s + bs * c))

    def injections(self, Vm, Va, x=None):
        pf, qf, pt, qt = self.flows(Vm, Va, x)
        P = torch.zeros_like(Vm).index_add(-1, self.f, pf).index_add(-1, self.t, pt)
        Q = torch.zeros_like(Vm).index_add(-1, self.f, qf).index_add(-1, self.t, qt)
        if self.ysh is not None:
            P = P + Vm * Vm * self.ysh[:, 0]
            Q = Q - Vm * Vm * self.ysh[:, 1]
        return P, Q

    def jacobian(self, Vm, Va):
        """Dense reduced Jacobian (rows P at non-slack, Q at PQ; columns theta
        at non-slack, |V| at PQ) of one state."""
        den = self.r * self.r + self.x * self.x
        y = torch.complex(self.r / den, -self.x / den)
        half = torch.complex(torch.zeros_like(self.b), self.b / 2)
        Y = torch.zeros(self.n, self.n, dtype=torch.complex128, device=y.device)
        for i, j, v in ((self.f, self.f, y + half), (self.t, self.t, y + half),
                        (self.f, self.t, -y), (self.t, self.f, -y)):
            Y.index_put_((i, j), v, accumulate=True)
        if self.ysh is not None:
            k = torch.arange(self.n, device=y.device)
            Y.index_put_((k, k), torch.complex(self.ysh[:, 0], self.ysh[:, 1]), accumulate=True)
        V = torch.polar(Vm, Va)
        cur = Y @ V
        A = V[:, None] * torch.conj(Y) * torch.conj(V)[None, :]
        k = torch.arange(self.n, device=y.device)
        St = -1j * A
        St[k, k] += 1j * V * torch.conj(cur)
        Sv = A / Vm[None, :]
        Sv[k, k] += torch.conj(cur) * V / Vm
        th, pq = self.th, self.pq
        top = torch.cat([St.real[th][:, th], Sv.real[th][:, pq]], 1)
        low = torch.cat([St.imag[pq][:, th], Sv.imag[pq][:, pq]], 1)
        return torch.cat([top, low], 0)


def _solve_exact(net, g, P, Q, x=None):
    """Power-flow solutions [B, n] by Newton steps with the Jacobian at the
    flat start, iterated until the mismatch is at rounding level; returns the
    states and that Jacobian's factors."""
    B = P.shape[0]
    Vm = _put(g["vset"]).expand(B, -1).clone()
    Va = torch.zeros_like(Vm)
    lu = torch.linalg.lu_factor(net.jacobian(Vm[0], Va[0]))
    last = math.inf
    for _ in range(80):
        p, q = net.injections(Vm, Va, x)
        F = torch.cat([(p - P)[:, net.th], (q - Q)[:, net.pq]], 1)
        worst = float(F.abs().max())
        if worst < 1e-12 and worst > 0.5 * last:
            break
        last = worst
        dx = torch.linalg.lu_solve(*lu, F.T.contiguous()).T
        Va[:, net.th] -= dx[:, :len(net.th)]
        Vm[:, net.pq] -= dx[:, len(net.th):]
    return (Vm, Va, lu) if last < 1e-9 else (None, None, None)


def _weights(case, seed):
    return np.random.default_rng([seed, case["n"], 3]).uniform(0.0, 1.0, case["n"])


def _reactances(case, g, seed):
    if case["shared_x"]:
        return g["x"]
    rng = np.random.default_rng([seed, case["n"], 5])
    return g["x"] * rng.uniform(0.95, 1.05, (case["batch"], g["m"]))


def _measurements(g):
    """|V|, P, Q at every bus and P, Q at the from end of every branch."""
    from paper_1811_02512_amd import binding as B

    n, m = g["n"], g["m"]
    kind = np.repeat(np.array([B.PF_MEAS_VM, B.PF_MEAS_P, B.PF_MEAS_Q, B.PF_MEAS_PF,
                               B.PF_MEAS_QF], np.int8), [n, n, n, m, m])
    loc = np.concatenate([np.arange(n)] * 3 + [np.arange(m)] * 2).astype(np.int32)
    return kind, loc


def _h(net, Vm, Va):
    P, Q = net.injections(Vm, Va)
    pf, qf, _, _ = net.flows(Vm, Va)
    return torch.cat([Vm, P, Q, pf, qf], -1)


def _telemetry(case, g, seed):
    """Noisy measurements z [B, M] of plausible states and weights w [M]."""
    net = _Net(g)
    Vm, Va = _states(g, case["batch"], seed)
    h = _h(net, _put(Vm), _put(Va))
    n = g["n"]
    sigma = torch.full((h.shape[-1],), 0.01, dtype=torch.float64, device=h.device)
    sigma[:n] = 0.004
    rng = np.random.default_rng([seed, n, 11])
    return h + sigma * _put(rng.standard_normal(h.shape)), 1.0 / sigma ** 2


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    from paper_1811_02512_amd import api

    kind = case["kind"]
    s = dict(case)
    if kind == "mixed":
        grids = [_grid(n) for n in _mixed_sizes(case)]
        syms = [_symbolic(g, case["tail"]) for g in grids]
        plan = api.MultiPlan(syms)
        if case["spread"]:
            plan.set_spread(case["spread"])
        inj = [_injections(g, 1, seed + k) for k, g in enumerate(grids)]
        bus, br, f8 = "bus", "branch", np.float64
        s.update(plan=plan,
                 r=plan.concat([g["r"] for g in grids], br, f8),
                 x=plan.concat([g["x"] for g in grids], br, f8),
                 b=plan.concat([g["b"] for g in grids], br, f8),
                 type=plan.concat([g["type"] for g in grids], bus, np.int8),
                 P=plan.concat([p[0] for p, _ in inj], bus, f8),
                 Q=plan.concat([q[0] for _, q in inj], bus, f8),
                 Vm0=plan.concat([g["vset"] for g in grids], bus, f8),
                 Va0=plan.concat([np.zeros(g["n"]) for g in grids], bus, f8),
                 yval=torch.empty(int(plan.offs["y"][-1]), dtype=torch.float64, device="cuda"),
                 ws=torch.empty(int(plan.offs["ws"][-1]), dtype=torch.float64, device="cuda"))
        return s
    g = _grid(case["n"], bool(case.get("shunts")))
    B, n = case["batch"], g["n"]
    s["r"], s["x"], s["b"], s["ysh"] = _branches(g)
    s["type"] = _put(g["type"])
    if kind == "flows":
        s["sym"] = api.Symbolic(n, g["f"], g["t"]).upload()
        Vm, Va = _states(g, B, seed)
        s["Vm"], s["Va"] = _put(Vm), _put(Va)
        return s
    if kind == "estimate":
        k, loc = _measurements(g)
        s["est"] = api.StateEstimator(n, g["f"], g["t"], k, loc, tail_lds_budget=case["tail"])
        s["z"], s["w"] = _telemetry(case, g, seed)
        s["Vm0"] = torch.ones(B, n, dtype=torch.float64, device="cuda")
        s["Va0"] = torch.zeros_like(s["Vm0"])
        s["ws"] = s["est"].workspace(B)
        return s
    s["sym"] = sym = _symbolic(g, case["tail"], case.get("spread", 0))
    one = kind == "screen"  # the screened base case is one case
    P, Q = _injections(g, 1 if one else B, seed)
    s["P"], s["Q"] = _put(P[0] if one else P), _put(Q[0] if one else Q)
    s["Vm0"] = _put(g["vset"])
    s["Va0"] = torch.zeros_like(s["Vm0"])
    if kind == "screen":
        rng = np.random.default_rng([seed, n, 9])
        cand = np.arange(g["tree"], g["m"])  # opening one of these never islands a bus
        s["outages"] = np.sort(rng.choice(cand, min(B, len(cand)), replace=False)).tolist()
        return s
    if kind == "gradient":
        s["P"].requires_grad_(True)
        s["Q"].requires_grad_(True)
        s["xg"] = _put(_reactances(case, g, seed)).requires_grad_(True)
        if not case["shared_x"]:
            s["r"], s["b"] = (v.expand(B, -1).contiguous() for v in (s["r"], s["b"]))
        s["w"] = _put(_weights(case, seed)) * (s["type"] == PQ)
        return s
    s["yval"] = sym.build_ybus(s["r"], s["x"], s["b"], s["ysh"])[0]
    if kind == "fdpf":
        s["mat"], _ = sym.fdpf_factors(s["r"], s["x"], s["b"], s["type"])
        s["ws"] = torch.empty(B, sym.info.fd_ws_doubles, dtype=torch.float64, device="cuda")
    elif kind == "newton":
        s["ws"] = sym.workspace(B)
    else:  # steps: states near a solution, a right-hand side for the transposed solve
        Vm, Va = _states(g, B, seed)
        s["Vm"], s["Va"] = _put(Vm), _put(Va)
        info = sym.info
        rng = np.random.default_rng([seed, n, 13])
        s["adj"] = _put(rng.standard_normal((B, 2 * info.nn)))
        s["vals"] = torch.empty(B, info.vals_doubles, dtype=torch.float64, device="cuda")
    return s


def _start(s):
    B, n = s["batch"], s["n"]
    return s["Vm0"].expand(B, n).clone(memory_format=torch.contiguous_format), torch.zeros(
        B, n, dtype=torch.float64, device="cuda")


def run(s):
    from paper_1811_02512_amd import binding as B

    kind = s["kind"]
    if kind == "newton":
        Vm, Va = _start(s)
        it, _, st, _ = s["sym"].newton(s["yval"], s["type"], s["P"], s["Q"], Vm, Va, tol=TOL,
                                       ws=s["ws"])
        return Vm, Va, it, st
    if kind == "gradient":
        from paper_1811_02512_amd.autograd import power_flow

        Vm, Va, st, it = power_flow(s["sym"], s["P"], s["Q"], s["xg"], s["r"], s["b"], s["type"],
                                    s["Vm0"], s["Va0"], tol=TOL, ysh=s["ysh"], with_status=True)
        loss = (s["w"] * (Vm - 1.0) ** 2).sum() + 0.5 * (s["w"] * Va * Va).sum()
        gP, gQ, gx = torch.autograd.grad(loss, (s["P"], s["Q"], s["xg"]))
        return Vm.detach(), Va.detach(), gP, gQ, gx, it, st
    if kind == "mixed":
        p, G = s["plan"], s["count"]
        Vm, Va = s["Vm0"].clone(), s["Va0"].clone()
        it = torch.empty(G, dtype=torch.int32, device="cuda")
        st = torch.empty(G, dtype=torch.int32, device="cuda")
        B.pf_build_ybus_multi(p.p, s["r"], s["x"], s["b"], s["yval"])
        B.pf_newton_multi(p.p, s["yval"], s["type"], s["P"], s["Q"], Vm, Va, TOL, 20, 0, s["ws"],
                          it, None, st)
        return Vm, Va, it, st
    if kind == "screen":
        from paper_1811_02512_amd import contingency

        o = contingency.screen(s["sym"], s["r"], s["x"], s["b"], s["type"], s["P"], s["Q"],
                               s["Vm0"], s["Va0"], s["outages"], tol=TOL)
        return o.Vm, o.Va, o.status, o.method, o.iters, list(o.flows)
    if kind == "fdpf":
        Vm, Va = _start(s)
        it, _, st, _ = s["sym"].fdpf(s["yval"], s["type"], s["P"], s["Q"], Vm, Va, s["mat"],
                                     tol=TOL, ws=s["ws"])
        return Vm, Va, it, st
    if kind == "estimate":
        Vm, Va = s["Vm0"].clone(), s["Va0"].clone()
        it, _, st, _ = s["est"].estimate(s["r"], s["x"], s["b"], s["z"], s["w"], Vm, Va, tol=TOL,
                                         ws=s["ws"])
        return Vm, Va, it, st
    if kind == "steps":
        sym, info, C, n = s["sym"], s["sym"].info, s["batch"], s["n"]
        vals, nn = s["vals"], info.nn
        rhs = torch.empty(C, 2 * nn, dtype=torch.float64, device="cuda")
        norm = torch.empty(C, dtype=torch.float64, device="cuda")
        st = torch.empty(C, dtype=torch.int32, device="cuda")
        lam = s["adj"].clone()
        B.pf_mismatch(sym.h, C, s["yval"], 0, s["type"], 0, s["P"], s["Q"], n, s["Vm"], s["Va"],
                      n, rhs, 2 * nn, norm)
        F = rhs.clone()
        B.pf_jacobian(sym.h, C, s["yval"], 0, s["type"], 0, s["Vm"], s["Va"], n, vals,
                      info.vals_doubles)
        B.pf_factor(sym.h, C, vals, info.vals_doubles, st)
        B.pf_solve(sym.h, C, vals, info.vals_doubles, rhs, 2 * nn)
        B.pf_solve(sym.h, C, vals, info.vals_doubles, lam, 2 * nn, transpose=1)
        return F, norm, vals, rhs, lam, st
    return list(s["sym"].branch_flows(s["r"], s["x"], s["b"], s["Vm"], s["Va"]))


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# Operations per bus: the filled graph of these systems holds about two blocks
# a bus above the diagonal and 2.4 block updates a bus, so assembling and
# factorising a 2 x 2 block matrix and solving with it takes about 300
# operations a bus and a Newton step, 60 with scalar factors kept; the gain
# matrix of the estimator has about 6.7 blocks and 45 block updates a bus.
def work(case):
    kind = case["kind"]
    if kind == "mixed":
        n = sum(_mixed_sizes(case))
        return {"bytes": 8.0 * n * (3 * 1.3 + 2 + 2 + 2), "flops": 5 * 300.0 * n}
    n, B = case["n"], case["batch"]
    m, c = 1.3 * n, float(case["n"]) * case["batch"]
    shared = 8.0 * 3 * m
    if kind == "newton":
        return {"bytes": 8.0 * 2 * 3.6 * n + 32.0 * c, "flops": 4 * 300.0 * c}
    if kind == "gradient":
        x = 2 * 8 * m * (1 if case["shared_x"] else B)
        return {"bytes": shared + x + 48.0 * c, "flops": (5 * 300.0 + 150.0) * c}
    if kind == "screen":
        return {"bytes": shared + 16.0 * n + 16.0 * c + 32.0 * m * B, "flops": 9 * 2 * 60.0 * c}
    if kind == "fdpf":
        return {"bytes": 8.0 * (2 * 3.6 + 2 * 5) * n + 32.0 * c, "flops": 9 * 2 * 60.0 * c}
    if kind == "estimate":
        return {"bytes": shared + 8.0 * (3 * n + 2 * m) * (B + 1) + 32.0 * c,
                "flops": 4 * 3500.0 * c}
    if kind == "steps":
        # voltages, injections and one right-hand side in; mismatch, factors, two solutions out
        return {"bytes": 8.0 * 2 * 3.6 * n + 8.0 * c * (2 + 2 + 2 + 2 + 4 + 2 * 8 + 4),
                "flops": 400.0 * c}
    return {"bytes": shared + 16.0 * c + 32.0 * m * B, "flops": 60.0 * m * B}


# ---------------------------------------------------------------------------
# exact values
# ---------------------------------------------------------------------------
def exact(case, seed):
    kind = case["kind"]
    if kind in ("mixed", "screen"):
        return None
    g = _grid(case["n"], bool(case.get("shunts")))
    net, B = _Net(g), case["batch"]
    if kind == "flows":
        Vm, Va = _states(g, B, seed)
        return list(net.flows(_put(Vm), _put(Va)))
    if kind == "estimate":
        return _estimate_exact(case, g, net, seed)
    if kind == "steps":
        return None  # outputs are in the analysis' elimination order
    if case["n"] > 4000:  # a dense factorisation of all unknowns takes too long
        return None
    P, Q = (_put(v) for v in _injections(g, B, seed))
    if kind in ("newton", "fdpf"):
        Vm, Va, _ = _solve_exact(net, g, P, Q)
        return None if Vm is None else (Vm, Va, None, None)
    # gradients: J(x)^T lam = dL/dx by iterations with the flat start's factors
    x = _put(_reactances(case, g, seed))
    w = _put(_weights(case, seed)) * (net.type == PQ)
    Vm, Va, lu = _solve_exact(net, g, P, Q, x)
    if Vm is None:
        return None
    Vm.requires_grad_(True)
    Va.requires_grad_(True)
    x.requires_grad_(True)
    loss = (w * (Vm - 1.0) ** 2).sum() + 0.5 * (w * Va * Va).sum()
    gv, ga = torch.autograd.grad(loss, (Vm, Va))
    p, q = net.injections(Vm, Va, x)
    th, pq = net.th, net.pq
    goal = torch.cat([ga[:, th], gv[:, pq]], 1)
    lam = torch.zeros_like(goal)

    def vjp(lam, wrt):
        lp, lq = torch.zeros_like(p), torch.zeros_like(q)
        lp[:, th], lq[:, pq] = lam[:, :len(th)], lam[:, len(th):]
        return lp, lq, torch.autograd.grad((p, q), wrt, (lp, lq), retain_graph=True)

    for _ in range(80):
        _, _, (jv, ja) = vjp(lam, (Vm, Va))
        res = goal - torch.cat([ja[:, th], jv[:, pq]], 1)
        if float(res.abs().max()) < 1e-14 * float(goal.abs().max()):
            break
        lam = lam + torch.linalg.lu_solve(*lu, res.T.contiguous(), adjoint=True).T
    gP, gQ, (gx,) = vjp(lam, (x,))
    return Vm.detach(), Va.detach(), gP, gQ, -gx, None, None


def _estimate_exact(case, g, net, seed):
    """Estimates case by case: a Gauss-Newton step from the flat start, then
    steps with the gain matrix at the state that it leads to."""
    if case["n"] > 2200:
        return None
    z, w = _telemetry(case, g, seed)
    n, B = g["n"], case["batch"]
    keep = torch.arange(2 * n, device=z.device) != n  # the slack's angle is fixed
    unit = torch.eye(2 * n, dtype=torch.float64, device=z.device)[keep]

    def h(u):
        return _h(net, u[:n], u[n:])

    def gain(u):
        Ht = torch.func.vmap(lambda e: torch.func.jvp(h, (u,), (e,))[1], chunk_size=512)(unit)
        return torch.linalg.lu_factor((Ht * w) @ Ht.T)

    flat = torch.cat([torch.ones(n, dtype=torch.float64, device=z.device),
                      torch.zeros(n, dtype=torch.float64, device=z.device)])
    first, done = gain(flat), []
    for c in range(B):
        u, lu = flat.clone(), first
        for it in range(60):
            v = u.clone().requires_grad_(True)
            hv = h(v)
            grad, = torch.autograd.grad(hv, v, w * (z[c] - hv).detach())
            dx = torch.linalg.lu_solve(*lu, grad[keep][:, None])[:, 0]
            u[keep] += dx
            if it == 0:
                lu = gain(u)
            worst = float(dx.abs().max())
            if worst < 1e-13:
                break
        if not worst < 1e-11:
            return None
        done.append(u)
    u = torch.stack(done)
    return u[:, :n], u[:, n:], None, None
