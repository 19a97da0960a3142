"""The work that users of this library have it do, as timed cases.

Each case is one pass through the public entry points of
`paper_2503_11674_amd`: a design of a stated size, generated by its netlist
generator with its own library and clock, held by a timing graph (or a
placer) as a user's program holds it, at cell positions drawn from a seed.

`kind` says what the pass does:
  step    one gradient step of timing-driven placement (Secs. III-B to III-D):
          timing update, report_timing_endpoint(n_fail, k) cut to K, the Eq. 9
          pair update, weighted-average wirelength and the pin-to-pin loss,
          forward and backward, into one gradient
  loop    one iteration of the placement loop (Sec. IV) between two timing
          refreshes: wirelength, density, pin-to-pin gradient, Nesterov step
  update  a timing update read back as WNS / TNS and the slack of every pin
  losses  the differentiable objectives through autograd: the pin-to-pin loss
          over exponentially weighted pairs, and the smoothed TNS
  report  a timing update and report_timing_endpoint(n, k), the paths read
          back to the host
  batch   the same over many designs of uneven size in one graph
Further fields: cells / depth / ff / lo (the design; lo: fewest inputs of a
cell), die (um), sigma (um, of the placement's 64 clusters; 0: uniform),
model (0 lumped, 1 Elmore star, 2 spanning-tree wires), prec, k, K, n
(endpoints reported), designs (of a batch).
"""
import functools
import math

import numpy as np
import torch

from paper_2503_11674_amd import netgen
from paper_2503_11674_amd.placer import GlobalPlacer, LoopConfig
from paper_2503_11674_amd.tdp import P2PLoss, SmoothTNS, TimingGraph

GAMMA_WL = 5.0     # um, weighted-average wirelength
GAMMA_TNS = 10.0   # ps, smoothed TNS
BETA = 1e-3        # weight of the pin-to-pin loss in the gradient
JITTER = 5.0       # um: how far a state's positions are from the design's own
FAIL = 0.05        # share of the endpoints that fail


def _case(name, kind, cells, depth, die, k=1, K=1, ff=0.10, lo=1, sigma=30.0, model=0, prec="f32", n=-1, designs=1):
    return dict(name=name, kind=kind, cells=cells, depth=depth, die=die, k=k, K=K, ff=ff, lo=lo, sigma=sigma,
                model=model, prec=prec, n=n, designs=designs)


def listed():
    return [
        # the smallest design, a block of 2,000 cells: launches and latency
        _case("step 2k cells", "step", 2000, 20, 1000.0, k=10, K=100, sigma=0.0),
        # a block of odd size under the fullest net model, few paths
        _case("step 23k cells, tree nets", "step", 23457, 41, 1373.0, k=3, K=777, model=2),
        # an ordinary block
        _case("step 200k cells", "step", 200_000, 60, 4000.0, k=10, K=10_000),
        # the largest design: a gradient step with timing refreshed every step
        _case("step 2M cells", "step", 2_000_000, 100, 10000.0, k=8, K=100_000, ff=0.12, lo=2),
        # the iterations between two timing refreshes, most of a placement run;
        # cells partly spread, as in the middle of one
        _case("loop 500k cells", "loop", 500_000, 60, 5657.0, sigma=350.0),
        _case("loop 60k cells", "loop", 60_123, 40, 1961.0, sigma=120.0),
        # timing alone, for a placer with its own net weighting; the library's
        # fuller wire models
        _case("update 1M cells, tree nets", "update", 1_000_000, 80, 7000.0, model=2),
        # double precision, for checking gradients by finite differences
        _case("update 100k cells, f64", "update", 100_003, 50, 2214.0, model=1, prec="f64"),
        # differentiable objectives
        _case("losses 1M cells", "losses", 1_000_000, 80, 7000.0, k=10, K=50_000),
        # looking at the worst paths of a block
        _case("report 150k cells", "report", 150_001, 57, 2711.0, k=10, K=1000, n=100),
        # many small designs at once
        _case("batch of 24", "batch", 20_000, 48, 1000.0, k=10, K=50, designs=24),
    ]


def draw(rng):
    kind = rng.choice(["step", "step", "step", "loop", "update", "losses", "report", "batch"])
    top = {"step": 900_000, "loop": 450_000, "update": 700_000, "losses": 600_000, "report": 300_000, "batch": 25_000}[kind]
    cells = int(round(2000 * math.exp(rng.random() * math.log(top / 2000))))
    depth = rng.randint(20, 100 if cells > 20_000 else 60)
    lo = rng.choice([1, 1, 2])
    k = rng.choice([1, 2, 3, 5, 8, 10, 12]) if kind in ("step", "losses", "report", "batch") else 1
    nfail = max(1, int(FAIL * 0.1 * cells))
    K = max(1, int(nfail * k * rng.uniform(0.6, 1.0))) if kind in ("step", "losses") else rng.randint(20, 1000)
    die = round(rng.uniform(6.0, 9.0) * math.sqrt(cells), 1)
    sigma = rng.choice([0.0, 30.0]) if kind != "loop" else round(die * rng.uniform(0.04, 0.1), 1)
    model = 0 if kind == "loop" else rng.choice([0, 0, 1, 2])
    prec = "f64" if kind in ("update", "losses") and cells < 150_000 and rng.random() < 0.3 else "f32"
    designs = rng.randint(3, 24) if kind == "batch" else 1
    c = _case("", kind, cells, depth, die, k=k, K=min(K, 100 if kind == "batch" else K), ff=round(rng.uniform(0.08, 0.14), 3),
              lo=lo, sigma=sigma, model=model, prec=prec, n=rng.choice([-1, 10, 100]) if kind == "report" else -1,
              designs=designs)
    del c["name"]
    return c


# ------------------------------------------------------------------ designs
_DESIGN = ("cells", "depth", "die", "ff", "lo", "sigma", "model", "designs")


def _design(case):
    return _designs(*[case[f] for f in _DESIGN])


@functools.lru_cache(maxsize=None)
def _designs(cells, depth, die, ff, lo, sigma, model, designs):
    """(netlists, library): the designs of a case, clocked so that FAIL of
    their endpoints fail at their own positions."""
    lib = dict(netgen.make_library(), net_model=model)
    out = []
    for i in range(designs):
        # the designs of a batch are of uneven size and depth
        f = 1.0 if designs == 1 else 0.5 + 1.5 * ((i * 7) % designs) / designs
        cfg = netgen.NetlistConfig("design", int(cells * f), ff_frac=ff, depth=max(5, depth - (i * 5) % 17), fanin_lo=lo,
                                   fanout_cap=16 if cells * f < 5000 else 32, die=die * math.sqrt(f),
                                   placement="gmm" if sigma > 0 else "uniform", gmm_sigma=max(sigma, 1.0), seed=i)
        nl = netgen.make_netlist(cfg)
        dev = torch.device("cuda", 0)
        t = _Exact(nl, lib, torch.tensor(nl["x"], device=dev), torch.tensor(nl["y"], device=dev),
                   tree_as_star=True)
        t.forward()
        nl["clock_period"] = np.float32(round(netgen.clock_period_for_fail_fraction(t.at[t.d_pin].cpu().numpy(), FAIL), 2))
        out.append(nl)
    return out, lib


def _positions(nls, seed):
    dev = torch.device("cuda", 0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    out = []
    for axis in ("x", "y"):
        base = torch.tensor(np.concatenate([nl[axis] for nl in nls]), device=dev)
        moved = base + JITTER * torch.randn(base.shape, generator=gen, device=dev)
        out.append(torch.minimum(moved.clamp_(min=0.0), base.max()))
    return out


def prepare(case, seed):
    nls, lib = _design(case)
    x, y = _positions(nls, seed)
    kind, k = case["kind"], case["k"]
    s = {"kind": kind, "case": case, "x": x, "y": y}
    if kind == "loop":
        nl = dict(nls[0], x=x.cpu().numpy(), y=y.cpu().numpy())
        bins = 1 << max(4, math.ceil(math.log2(math.sqrt(case["cells"] / 2))))
        p = GlobalPlacer(nl, lib, LoopConfig(die=case["die"], bins=bins, timing_start=0))
        for _ in range(3):  # the first of them times the design and forms the pairs
            p.step()
        s.update(p=p, snap=p.snapshot())
        return s
    g = s["g"] = TimingGraph(nls if kind == "batch" else nls[0], lib, precision=case["prec"], max_paths=max(case["K"], case["n"] * k), max_k=k)
    g.sta_update(x, y)
    if kind == "step":
        s.update(gx=torch.zeros_like(x), gy=torch.zeros_like(y),
                 beta=torch.full((), BETA, dtype=torch.float64, device=x.device))
    elif kind == "update":
        v = g.views()
        s.update(at=v["at"], rat=v["rat"], idx=v["pin_index"].clone())
    elif kind == "losses":
        g.extract_paths(n=-1, k=k, K=case["K"])
        g.pairs_update(rule=1)
        x.requires_grad_(True)
        y.requires_grad_(True)
    return s


def run(s):
    case, x, y, kind = s["case"], s["x"], s["y"], s["kind"]
    if kind == "loop":
        p = s["p"]
        p.resume(s["snap"])
        p.step()
        return {"wl": p.wl_prev, "ux": p.st["ux"], "uy": p.st["uy"], "vx": p.st["vx"], "vy": p.st["vy"], "gx": p.gx, "gy": p.gy}
    g = s["g"]
    if kind == "losses":
        pp = P2PLoss.apply(x, y, g)
        gp = torch.autograd.grad(pp, (x, y))
        st = SmoothTNS.apply(x, y, g, GAMMA_TNS)
        gs = torch.autograd.grad(st, (x, y))
        return {"pp": pp.detach(), "gp": gp, "st": st.detach(), "gs": gs}
    g.sta_update(x, y)
    if kind == "step":
        g.extract_paths(n=-1, k=case["k"], K=case["K"])
        g.pairs_update(rule=0, w0=10.0, w1=0.2)
        s["gx"].zero_()
        s["gy"].zero_()
        wl = g.wa_fwd_bwd_at_update(GAMMA_WL, s["gx"], s["gy"])
        pp = g.p2p_loss_fwd(x, y)
        g.p2p_loss_bwd(x, y, s["beta"], s["gx"], s["gy"])
        return {"wl": wl, "pp": pp, "gx": s["gx"], "gy": s["gy"]}
    if kind == "update":
        wns, tns, nf = g.summary()
        return {"wns": wns, "tns": tns, "nf": nf, "slack": (s["rat"] - s["at"])[s["idx"]]}
    g.extract_paths(n=case["n"], k=case["k"], K=case["K"])
    if kind == "batch":
        w, t, n = g.batch_summary()
        return {"wns": w, "tns": t, "nf": n, "paths": _padded(g)}
    wns, tns, nf = g.summary()
    return {"wns": wns, "tns": tns, "nf": nf, "paths": _padded(g)}


def _padded(g):
    """The reported paths on the host, in arrays of the report's capacity."""
    p, rows = g.paths(), g.max_paths * g.num_inst
    size = {"path_ptr": rows + 1, "path_pins": rows * (2 * g.depth + 2)}
    return {f: v if f == "num_paths" else np.pad(v, (0, size.get(f, rows) - len(v)), constant_values=-1)
            for f, v in p.items()}


def work(case):
    """What a pass cannot do without: the netlist (per sink its driver and pin
    offset, per driver its offset, per cell its type), the positions and the
    clocked results, each read or written once."""
    n = case["cells"] * case["designs"]
    e, m = case["ff"] * n, 1.1 * n
    s = (n - e) * (case["lo"] + 4) / 2 + e
    p, kind = m + s, case["kind"]
    net = 12 * s + 8 * m + n + 8 * n
    val = 8 if case["prec"] == "f64" else 4
    nfail = FAIL * e if case["n"] < 0 else case["n"]
    paths = min(case["K"] * (case["designs"] if kind == "batch" else 1), nfail * case["k"])
    pins = 1.8 * case["depth"] * paths
    b = {"step": net + 2 * val * p + 4 * pins + 8 * n, "loop": net + 4 * n + 16 * n + 48 * n,
         "update": net + 3 * val * p, "losses": net + val * p + 8 * n + 16 * n,
         "report": net + 2 * val * p + 4 * pins, "batch": net + 2 * val * p + 4 * pins}[kind]
    f = {"step": 90, "loop": 60 + 350 * n / p, "update": 40, "losses": 60, "report": 40, "batch": 40}[kind] * p
    return {"bytes": float(b), "flops": float(f)}


# -------------------------------------------------------- the same in 64 bits
class _Exact:
    """Late timing of one design in double precision, level by level."""

    def __init__(self, nl, lib, x, y, tree_as_star=False):
        dev, f64 = x.device, torch.float64
        t = lambda a, dt=torch.int64: torch.as_tensor(np.asarray(a), device=dev).to(dt)
        self.dev, self.lib, self.nl = dev, lib, nl
        self.model = 1 if (lib["net_model"] == 2 and tree_as_star) else int(lib["net_model"])
        self.P = int(nl["num_pins"])
        cell, ox, oy = t(nl["pin_cell"]), t(nl["pin_off_x"], f64), t(nl["pin_off_y"], f64)
        ptr, pins = t(nl["net_ptr"]), t(nl["net_pins"])
        net = torch.repeat_interleave(torch.arange(len(ptr) - 1, device=dev), ptr[1:] - ptr[:-1])
        drv = pins[ptr[:-1]][net]
        self.net, self.net_pins, self.nets = net, pins, len(ptr) - 1
        self.cell, self.ox, self.oy = cell, ox, oy
        m = drv != pins
        self.snk, self.drv = pins[m], drv[m]
        self.typ, self.ff = t(nl["cell_type"]), t(nl["cell_is_ff"]).bool()
        self.out = t(nl["cell_out_pin"])
        c = cell[self.snk]
        self.is_d = self.ff[c]
        self.d_pin = t(nl["cell_in_pins"])[t(nl["cell_in_ptr"])[:-1][self.ff]]
        # levels: one above the highest driver
        lev = torch.zeros(len(self.typ) + 1, dtype=torch.int64, device=dev)  # the last: ports
        ci, cd = c[~self.is_d], cell[self.drv[~self.is_d]]
        while True:
            new = torch.zeros_like(lev).scatter_reduce(0, ci, torch.where(cd >= 0, lev[cd], 0) + 1, "amax")
            if torch.equal(new, lev):
                break
            lev = new
        order = torch.argsort(lev[ci], stable=True)
        self.arcs = torch.nonzero(~self.is_d)[:, 0][order]
        cnt = torch.bincount(lev[ci])[1:].tolist()
        self.levels = torch.split(self.arcs, cnt)
        self.place(x, y)

    def xy(self, x, y, p):
        c = self.cell[p]
        on = c >= 0
        z = torch.zeros((), dtype=torch.float64, device=self.dev)
        return (torch.where(on, x[c.clamp_min(0)], z) + self.ox[p], torch.where(on, y[c.clamp_min(0)], z) + self.oy[p])

    def place(self, x, y):
        """Net delays and loads at positions (x, y) (double; may carry gradients)."""
        x, y = x.double(), y.double()
        lib = self.lib
        r, c, sc = (float(np.float32(lib[q])) for q in ("r_per_um", "c_per_um", "delay_scale"))
        xs, ys = self.xy(x, y, self.snk)
        xd, yd = self.xy(x, y, self.drv)
        ln = (xd - xs).abs() + (yd - ys).abs()
        cap = torch.as_tensor(np.asarray(lib["pin_cap"], np.float64), device=self.dev)[self.typ[self.cell[self.snk]]]
        self.dn = sc * r * c * ln * ln if self.model == 0 else sc * r * ln * (c * ln / 2 + cap)
        self.load = torch.zeros(self.P, dtype=torch.float64, device=self.dev).index_add(0, self.drv, (cap + c * ln).detach())

    def table(self, typ, slew, load):
        lib, dev = self.lib, self.dev
        get = lambda q: torch.as_tensor(np.asarray(lib[q], np.float64), device=dev)
        sa, la = get("slew_axis"), get("load_axis")
        ns, nl = sa.shape[1], la.shape[1]
        s = torch.minimum(torch.maximum(slew, sa[typ, 0]), sa[typ, -1])
        q = torch.minimum(torch.maximum(load, la[typ, 0]), la[typ, -1])
        i = (sa[typ, 1:ns - 1] <= s[:, None]).sum(1)
        j = (la[typ, 1:nl - 1] <= q[:, None]).sum(1)
        u = (s - sa[typ, i]) / (sa[typ, i + 1] - sa[typ, i])
        v = (q - la[typ, j]) / (la[typ, j + 1] - la[typ, j])
        res = []
        for name in ("delay_lut", "slew_lut"):
            d = get(name)
            res.append((1 - u) * (1 - v) * d[typ, i, j] + u * (1 - v) * d[typ, i + 1, j] + (1 - u) * v * d[typ, i, j + 1]
                       + u * v * d[typ, i + 1, j + 1])
        return res

    def forward(self):
        nl, f64 = self.nl, torch.float64
        at = torch.full((self.P,), -math.inf, dtype=f64, device=self.dev)
        slew = torch.zeros(self.P, dtype=f64, device=self.dev)
        port = self.cell < 0
        at[port], slew[port] = 0.0, float(nl["input_slew"])
        q = self.out[self.ff]
        at[q], slew[q] = self.table(self.typ[self.ff], torch.full(q.shape, float(nl["clock_slew"]), dtype=f64, device=self.dev),
                                    self.load[q])
        self.darc = torch.zeros(len(self.snk), dtype=f64, device=self.dev)
        for a in self.levels:
            s, d = self.snk[a], self.drv[a]
            o = self.out[self.cell[s]]
            at[s] = at[d] + self.dn[a]
            sl = slew[d]
            if self.model:
                sl = torch.sqrt(sl * sl + (math.log(9.0) * self.dn[a]) ** 2)
            self.darc[a], tr = self.table(self.typ[self.cell[s]], sl, self.load[o])
            at.scatter_reduce_(0, o, at[s] + self.darc[a], "amax")
            slew.scatter_reduce_(0, o, tr, "amax")
        e = torch.nonzero(self.is_d)[:, 0]
        at[self.snk[e]] = at[self.drv[e]] + self.dn[e]
        self.at = at
        self.req = float(nl["clock_period"] - nl["setup"])
        sl = self.req - at[self.d_pin]
        neg = sl[sl < 0]
        self.wns, self.tns = (neg.min(), neg.sum()) if len(neg) else (torch.zeros((), dtype=f64), torch.zeros((), dtype=f64))

    def slack(self):
        rat = torch.full((self.P,), math.inf, dtype=torch.float64, device=self.dev)
        rat[self.d_pin] = self.req
        e = torch.nonzero(self.is_d)[:, 0]
        rat.scatter_reduce_(0, self.drv[e], rat[self.snk[e]] - self.dn[e], "amin")
        for a in reversed(self.levels):
            s = self.snk[a]
            rat[s] = rat[self.out[self.cell[s]]] - self.darc[a]
            rat.scatter_reduce_(0, self.drv[a], rat[s] - self.dn[a], "amin")
        return rat - self.at

    def smooth(self, gamma):
        """The smoothed TNS from the frozen arc delays and start arrivals."""
        start = torch.cat([torch.nonzero(self.cell < 0)[:, 0], self.out[self.ff]])
        at = torch.zeros_like(self.at).index_copy(0, start, self.at[start])
        for a in self.levels:
            o = self.out[self.cell[self.snk[a]]]
            v = at[self.drv[a]] + self.dn[a] + self.darc[a]
            u, inv = torch.unique(o, return_inverse=True)
            m = torch.full(u.shape, -math.inf, dtype=torch.float64, device=self.dev).scatter_reduce(0, inv, v.detach(), "amax")
            z = torch.zeros(u.shape, dtype=torch.float64, device=self.dev).index_add(0, inv, torch.exp((v - m[inv]) / gamma))
            at = at.index_copy(0, u, m + gamma * torch.log(z))
        e = torch.nonzero(self.is_d)[:, 0]
        z = (at[self.drv[e]] + self.dn[e] - self.req) / gamma
        return -gamma * torch.logaddexp(z, torch.zeros_like(z)).sum()

    def wirelength(self, x, y, gamma):
        total = 0.0
        for v in self.xy(x.double(), y.double(), self.net_pins):
            for sign in (1.0, -1.0):
                w = sign * v
                m = torch.full((self.nets,), -math.inf, dtype=torch.float64, device=self.dev).scatter_reduce(0, self.net, w, "amax")
                ex = torch.exp((w - m[self.net]) / gamma)
                zero = torch.zeros(self.nets, dtype=torch.float64, device=self.dev)
                d = zero.index_add(0, self.net, (w - m[self.net]) * ex) / zero.index_add(0, self.net, ex)
                total = total + (m + d).sum()
        return total


def exact(case, seed):
    kind = case["kind"]
    if kind == "loop":
        return None  # a step of a whole optimiser, with its own history
    nls, lib = _design(case)
    if kind == "batch":
        x, y = _positions(nls, seed)
        w, t, at = [], [], 0
        for nl in nls if lib["net_model"] < 2 else []:
            n = int(nl["num_cells"])
            ex = _Exact(nl, lib, x[at:at + n], y[at:at + n])
            ex.forward()
            w.append(float(ex.wns))
            t.append(float(ex.tns))
            at += n
        return {"wns": np.array(w), "tns": np.array(t), "nf": None, "paths": None} if w else None
    x, y = _positions(nls, seed)
    if kind == "step":
        wl = _Exact(nls[0], lib, x, y, tree_as_star=True).wirelength(x, y, GAMMA_WL)
        return {"wl": wl, "pp": None, "gx": None, "gy": None}
    if lib["net_model"] == 2:
        return None  # its trees are chosen by 32-bit distances
    ex = _Exact(nls[0], lib, x, y)
    ex.forward()
    if kind == "losses":
        xd, yd = x.double().requires_grad_(True), y.double().requires_grad_(True)
        ex.place(xd, yd)
        st = ex.smooth(GAMMA_TNS)
        return {"pp": None, "gp": (None, None), "st": st.detach(), "gs": torch.autograd.grad(st, (xd, yd))}
    out = {"wns": ex.wns, "tns": ex.tns, "nf": None}
    return dict(out, slack=ex.slack()) if kind == "update" else dict(out, paths=None)
