"""What a user of this framework has it do, as measurable cases.

A pass is a stretch of a melting (or solidification) run between two
outputs: advance the handle by some steps, then read the whole fields back
and log the diagnostics.  The initial state is a partly melted cavity (hot
liquid next to the heated wall, a wavy front, solid beyond), so every
branch of the enthalpy method and the flow are exercised from the first
step on.

`exact` is the same run in plain torch in 64 bits: the method of
arXiv:1701.00702 with dense moment transforms, without this repository's
code.
"""
import math

import numpy as np
import torch

from paper_1701_00702_amd import lbm

# Dimensionless groups of the problems (Eq. 54).  "cavity" is the Sec. IV B
# cavity (hot left, cold right wall) of the benchmark sizes; "paper" the
# paper's own Ra = 1e6 run; "corner" the solidification in a corner of
# Sec. IV A (cold left and bottom walls, no flow).
_BASE = dict(bc_x=0, gravity_axis=1, porosity=0.9, Ra=1e6, Pr=50.0, Da=1e-4, Ste=1.0, k_ratio=100.0,
             cap_ratio=1.0, Nu_i=5.0, F_phi=-1.0, dp_over_L=0.0, k_f=0.0, cf_ref=0.0, cm_ref=0.0, J=0.0,
             T_hot=1.0, T_cold=0.0, T_init=0.0, T_solidus=0.0, T_liquidus=0.002, thermal_lattice=9,
             thermal_collision=0, varpi=0.0, zeta_e=0.0, wall_type=(0, 0, 0, 0), wall_T=(0.0, 0.0, 0.0, 0.0),
             L_char=0.0, solid_treatment=0, band_rows=0, pcm_even_rates=0)
_PROBLEMS = {
    "cavity": {},
    "paper": dict(porosity=0.8, k_ratio=1000.0, Nu_i=5.9, F_phi=0.068, k_f=5e-4, cf_ref=0.2, cm_ref=1.0, J=1.0,
                  T_solidus=0.299, T_liquidus=0.301),
    "corner": dict(porosity=0.8, Ra=0.0, Pr=1.0, Da=1.0, Ste=4.0, k_ratio=10.0, Nu_i=5.9, F_phi=0.068, k_f=0.01,
                   cf_ref=0.5, cm_ref=1.0, T_hot=0.0, T_cold=-1.0, T_init=0.3, T_solidus=-0.05,
                   T_liquidus=0.05, wall_type=(1, 2, 1, 2), wall_T=(-1.0, 0.0, -1.0, 0.0)),
}
_STATE_BYTES = {("f64", 9): 224, ("f32", 9): 112, ("f32h64", 9): 116, ("f16split", 9): 76, ("f64", 5): 160,
                ("f32", 5): 80, ("f32h64", 5): 84}  # per node: populations and the previous source
_FLOP = {9: 420, 5: 290}  # multiplies and adds of one node update (three coupled fields)
_LOG = ("liquid_fraction", "Nu_hot", "Nu_cold", "E_int", "M_int", "x_front_mid", "max_dT_LTNE", "u_max")
_FIELDS = ("ux", "uy", "T_pcm", "T_mf", "f_l", "rho")


def listed():
    c = _case
    return [
        # a live monitor of a small run: ten steps, then the diagnostics; launches and waits count
        c("monitor 256", 256, 256, "f32h64", 10, read="log"),
        # the small checking run of the test suite, in full precision
        c("cavity 64 f64", 64, 64, "f64", 2000),
        # the paper's own grid (Sec. IV B), full precision
        c("paper 151 f64", 151, 151, "f64", 2000, problem="paper"),
        # Sec. IV A: isothermal walls left and bottom, no flow
        c("corner 200 f64", 200, 200, "f64", 1000, problem="corner"),
        # the A/B size of the 32-bit forms
        c("cavity 256 f32h64", 256, 256, "f32h64", 2500),
        # 32-bit production run, odd sides, Appendix B's five-velocity thermal lattice
        c("ragged 1001x613 f32 q5", 1001, 613, "f32", 2000, lattice=5),
        # 32-bit production run
        c("cavity 1024 f32h64", 1024, 1024, "f32h64", 3000),
        # reference run in full precision
        c("cavity 1024 f64", 1024, 1024, "f64", 1000),
        # a parameter study: many uneven cavities (sides log-uniform in [64, 512]) in one handle;
        # the table of all diagnostics and the fields of eight of them come back
        c("study of 256 f32", 0, 0, "f32", 600, cavities=256),
        # half the memory: the split 16-bit store
        c("cavity 4096 f16split", 4096, 4096, "f16split", 1000),
        # the large cavity of the benchmark
        c("cavity 8192 f32h64", 8192, 8192, "f32h64", 600, Ra=1e7, Da=1e-5, Ste=0.5, k_ratio=1000.0),
    ]


def _case(name, nx, ny, precision, steps, problem="cavity", lattice=9, cavities=1, read="fields", **groups):
    return dict(dict(name=name, nx=nx, ny=ny, precision=precision, steps=steps, problem=problem, lattice=lattice,
                     cavities=cavities, read=read), **groups)


def draw(rng):
    """A run of any size, form and length in between."""
    kind = rng.choice(["single"] * 5 + ["study", "log"])
    precision, lattice = rng.choice([("f32h64", 9), ("f32h64", 9), ("f32", 9), ("f64", 9), ("f16split", 9),
                                     ("f32", 5), ("f32h64", 5), ("f64", 5)])
    groups = dict(porosity=round(rng.uniform(0.85, 0.97), 4), Ra=10 ** rng.uniform(4, 6), Da=10 ** rng.uniform(-5, -3),
                  Ste=round(rng.uniform(0.2, 2.0), 4), Nu_i=round(rng.uniform(1, 20), 4))
    if kind == "study":
        return _case_without_name(0, 0, precision, rng.randint(60, 600), lattice=lattice, cavities=rng.randint(9, 200))
    nx = int(round(math.exp(rng.uniform(math.log(40), math.log(4000)))))
    ny = max(24, min(4000, int(round(nx * rng.uniform(0.5, 2.0)))))
    if kind == "log":
        return _case_without_name(min(nx, 900), min(ny, 900), precision, rng.randint(4, 40), lattice=lattice, read="log",
                                  **groups)
    most = max(60.0, min(3000.0, 1.2e10 / (nx * ny)))  # node updates well below the largest listed case's
    return _case_without_name(nx, ny, precision, int(rng.uniform(0.3, 1.0) * most), lattice=lattice, **groups)


def _case_without_name(*a, **kw):
    c = _case("", *a, **kw)
    del c["name"]
    return c


def _problems(case):
    """The parameters of each cavity of a case."""
    own = {k: case[k] for k in ("porosity", "Ra", "Da", "Ste", "k_ratio", "Nu_i") if k in case}
    if case["cavities"] == 1:
        p = dict(_BASE, **dict(_PROBLEMS[case["problem"]], **own))
        p.update(nx=case["nx"], ny=case["ny"], thermal_lattice=case["lattice"])
        if case["problem"] == "corner":
            p["L_char"] = case["nx"] / 2.0
        return [p]
    # a fixed design of uneven cavities: sides, aspects and groups spread over the study's ranges
    rng = np.random.default_rng(7)
    out = []
    for _ in range(case["cavities"]):
        n = int(round(math.exp(rng.uniform(math.log(64), math.log(512)))))
        out.append(dict(_BASE, nx=n, ny=n * int(rng.integers(1, 3)), porosity=rng.uniform(0.85, 0.97),
                        Ra=10.0 ** rng.uniform(4, 6), Da=10.0 ** rng.uniform(-5, -3), Ste=rng.uniform(0.2, 2.0),
                        Nu_i=rng.uniform(1, 20), thermal_lattice=case["lattice"]))
    return out


def _initial(p, rng):
    """Initial temperature of PCM and foam: melted up to a wavy front, with small noise."""
    nx, ny = p["nx"], p["ny"]
    if p["wall_type"][0] == 1:  # solidification: everything liquid at T_init
        T = np.full((ny, nx), p["T_init"])
    else:
        at, waves = rng.uniform(0.25, 0.4), rng.integers(1, 5)
        y = np.arange(ny) / (ny - 1.0)
        front = (nx - 1.0) * (at + 0.05 * np.sin(2 * np.pi * (waves * y + rng.uniform())))
        T = np.arange(nx)[None, :] * (-1.0 / front)[:, None]
        T += 1.0
        np.maximum(T, 0.0, out=T)
        if p["T_hot"] - p["T_cold"] != 1.0 or p["T_cold"] != 0.0:
            T *= p["T_hot"] - p["T_cold"]
            T += p["T_cold"]
    noise = rng.random((ny, nx), dtype=np.float32)
    noise -= 0.5
    noise *= 2e-6
    T += noise
    return T


def prepare(case, seed):
    ps = _problems(case)
    rng = np.random.default_rng([seed, 1701])
    s = lbm.Solver(ps if len(ps) > 1 else ps[0], case["precision"])
    for c, p in enumerate(ps):
        T = _initial(p, rng)
        s.set_initial(c, T, T)
    return {"solver": s, "steps": case["steps"], "read": case["read"],
            "shown": range(0, len(ps), max(1, -(-len(ps) // 8))) if len(ps) > 1 else range(1)}


def run(state):
    s = state["solver"]
    s.step(state["steps"])
    n = len(s.params)
    if n > 1:
        log = [s.diagnostics(c) for c in range(n)]
        return {"log": {k: np.array([d[k] for d in log]) for k in _LOG},
                "fields": [s.fields(c) for c in state["shown"]]}
    d = s.diagnostics()
    log = {k: d[k] for k in _LOG}
    return {"log": log} if state["read"] == "log" else {"log": log, "fields": s.fields()}


def work(case):
    # the state crosses memory at least once each way in a pass; the fields read (six doubles a node) come on top
    per = 2 * _STATE_BYTES[case["precision"], case["lattice"]]
    sizes = [p["nx"] * p["ny"] for p in _problems(case)]
    shown = sizes[::max(1, -(-len(sizes) // 8))] if len(sizes) > 1 else sizes
    back = 0 if case["read"] == "log" else 48 * sum(shown)
    return {"bytes": per * sum(sizes) + back, "flops": _FLOP[case["lattice"]] * sum(sizes) * case["steps"]}


# ---------------------------------------------------------------------------
# The same run in 64 bits.
# ---------------------------------------------------------------------------
_E = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_W = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_M9 = [[1, 1, 1, 1, 1, 1, 1, 1, 1], [-4, -1, -1, -1, -1, 2, 2, 2, 2], [4, -2, -2, -2, -2, 1, 1, 1, 1],
       [0, 1, 0, -1, 0, 1, -1, -1, 1], [0, -2, 0, 2, 0, 1, -1, -1, 1], [0, 0, 1, 0, -1, 1, 1, -1, -1],
       [0, 0, -2, 0, 2, 1, 1, -1, -1], [0, 1, -1, 1, -1, 0, 0, 0, 0], [0, 0, 0, 0, 0, 1, -1, 1, -1]]
_M5 = [[1, 1, 1, 1, 1], [0, 1, 0, -1, 0], [0, 0, 1, 0, -1], [0, 1, 1, 1, 1], [0, 1, -1, 1, -1]]


def exact(case, seed):
    updates = sum(p["nx"] * p["ny"] for p in _problems(case)) * case["steps"]
    if case["cavities"] > 1 or 2e-3 * case["steps"] + 1.2e-9 * updates > 18:
        return None
    p = _problems(case)[0]
    run_ = _Exact(p, _initial(p, np.random.default_rng([seed, 1701])))
    for _ in range(case["steps"]):
        run_.step()
    f = run_.fields()
    inner = {k: f[k][1:-1, 1:-1] for k in _FIELDS}
    log = dict.fromkeys(_LOG)
    log["liquid_fraction"] = float(inner["f_l"].mean())
    log["max_dT_LTNE"] = float((inner["T_pcm"] - inner["T_mf"]).abs().max())
    log["u_max"] = float((inner["ux"] ** 2 + inner["uy"] ** 2).sqrt().max())
    return {"log": log} if case["read"] == "log" else {"log": log, "fields": f}


class _Exact:
    def __init__(self, p, T0):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.p, self.q = p, p["thermal_lattice"]
        self.col = lambda v: torch.tensor(v, dtype=torch.float64, device=dev).reshape(-1, 1)
        nx, ny = self.shape = p["nx"], p["ny"]
        phi = self.phi = p["porosity"]
        self.cf, self.cm = p["cf_ref"] if p["cf_ref"] > 0 else 0.2, p["cm_ref"] if p["cm_ref"] > 0 else 1.0
        J, L = (p["J"] if p["J"] > 0 else 1.0), (p["L_char"] if p["L_char"] > 0 else nx - 1.0)
        d_p = (p["dp_over_L"] if p["dp_over_L"] > 0 else 0.0135) * L
        self.varpi = p["varpi"] if p["varpi"] > 0 else 2 / 3
        cs2 = 1 / 3 if self.q == 9 else self.varpi / 2
        rho_m, Nu = p["cap_ratio"], p["Nu_i"]
        per = 1 / phi + 1 / ((1 - phi) * rho_m)
        kf = p["k_f"]
        if kf <= 0:  # the largest value with every relaxation time <= 2 and the exchange number <= 0.5
            kf = min(0.5 / (J * p["Pr"]), 1.5 * cs2 * self.cf, 1.5 * cs2 * rho_m * self.cm / p["k_ratio"],
                     0.5 * d_p * d_p / (Nu * per))
        nu, h_v, K = p["Pr"] * kf, Nu * kf / d_p ** 2, p["Da"] * L * L
        F_phi = p["F_phi"] if p["F_phi"] >= 0 else 1.75 / math.sqrt(150 * phi ** 3)
        dT = p["T_hot"] - p["T_cold"]
        self.gbeta = p["Ra"] * nu * kf / (dT * L ** 3)
        self.Hs, self.Hl = p["T_solidus"], p["T_liquidus"] + dT / p["Ste"]
        self.lin, self.quad = phi * nu / K, phi * F_phi / math.sqrt(K)
        self.l0, self.l1 = 0.5 * (1 + 0.5 * self.lin), 0.5 * self.quad
        self.hf, self.hm = h_v / phi, h_v / ((1 - phi) * rho_m)
        sv, za, ea = 1 / (0.5 + 3 * J * nu), 1 / (0.5 + kf / self.cf / cs2), 1 / (0.5 + p["k_ratio"] * kf / (rho_m * self.cm) / cs2)
        self.s = self.col([1, 1.1, 1.1, 1, 1.2, 1, 1.2, sv, sv])
        if self.q == 9:
            self.z, self.e = self.col([1, 2 - za, 2 - za, za, za, za, za, 1.2, 1.2]), self.col([1, 1.1, 1.1, ea, ea, ea, ea, 1.2, 1.2])
        else:
            self.z, self.e = self.col([1, za, za, 2 - za, 2 - za]), self.col([1, ea, ea, 1.1, 1.1])
        self.M = torch.tensor(_M9, dtype=torch.float64, device=dev)
        self.Mt = self.M if self.q == 9 else torch.tensor(_M5, dtype=torch.float64, device=dev)
        self.Mi, self.Mti = (m.cpu().inverse().to(dev) for m in (self.M, self.Mt))
        self.w = self.col(_W)
        self.wt = self.w if self.q == 9 else self.col([0] + [self.varpi / 4] * 4)
        self.rest = 5 / 9 if self.q == 9 else self.varpi
        # wall nodes: their inward partners and, on isothermal walls, their temperatures
        kinds = [t if t else (1, 1, 2, 2)[i] for i, t in enumerate(p["wall_type"])]
        temps = [p["wall_T"][i] if p["wall_type"][i] else (p["T_hot"], p["T_cold"], 0, 0)[i] for i in range(4)]
        x, y = np.meshgrid(np.arange(nx), np.arange(ny))
        wall = (x == 0) | (x == nx - 1) | (y == 0) | (y == ny - 1)
        Tw = np.full((ny, nx), np.nan)
        for i, on in ((3, y == ny - 1), (2, y == 0), (1, x == nx - 1), (0, x == 0)):
            if kinds[i] == 1:
                Tw[on] = temps[i]
        t = lambda a: torch.as_tensor(a, device=dev)  # noqa: E731
        self.wall = t((y * nx + x)[wall])
        self.partner = t((np.clip(y, 1, ny - 2) * nx + np.clip(x, 1, nx - 2))[wall])
        self.Tw = t(Tw[wall])
        self.iso = ~torch.isnan(self.Tw)
        T = torch.where(torch.isnan(t(Tw)), t(T0), t(Tw)).reshape(-1)
        one = torch.ones_like(T)
        self.f = self.w * one
        self.g, self.h = self._rest(self._H(T), T, self.cf), self._rest(T, T, self.cm)
        self.before = self.hf * 0 * T

    def _H(self, T):
        p = self.p
        mid = self.Hs + (T - p["T_solidus"]) / (p["T_liquidus"] - p["T_solidus"]) * (self.Hl - self.Hs)
        return torch.where(T <= p["T_solidus"], T, torch.where(T >= p["T_liquidus"], T - p["T_liquidus"] + self.Hl, mid))

    def _rest(self, H, T, c):
        q = self.wt * (c * T)
        q[0] = H - self.rest * c * T
        return q

    def _macros(self, f, g, h):
        p, H = self.p, g.sum(0)
        fl = ((H - self.Hs) / (self.Hl - self.Hs)).clamp(0, 1)
        T = torch.where(H <= self.Hs, H, torch.where(H >= self.Hl, p["T_liquidus"] + (H - self.Hl),
                                                     p["T_solidus"] + fl * (p["T_liquidus"] - p["T_solidus"])))
        rho = f.sum(0)
        jx, jy = (sum(e[a] * f[i] for i, e in enumerate(_E) if e[a]) * fl for a in (0, 1))
        G = self.gbeta * (T - p["T_cold"]) * fl
        vx, vy = jx / rho, jy / rho + 0.5 * self.phi * G
        d = self.l0 + (self.l0 ** 2 + self.l1 * (vx * vx + vy * vy).sqrt()).sqrt()
        return dict(H=H, fl=fl, T=T, Tm=h.sum(0), rho=rho, G=G, ux=vx / d, uy=vy / d)

    def step(self):
        m, phi = self._macros(self.f, self.g, self.h), self.phi
        fl, T, Tm, rho, ux, uy = (m[k] for k in ("fl", "T", "Tm", "rho", "ux", "uy"))
        f = fl * self.f + (1 - fl) * self.w * rho
        uu = ux * ux + uy * uy
        drag = self.lin + self.quad * uu.sqrt()
        Fx, Fy = -drag * ux, -drag * uy + phi * m["G"]
        uF = ux * Fx + uy * Fy
        eq = rho * torch.stack([torch.ones_like(T), -2 + 3 * uu / phi, 1 - 3 * uu / phi, ux, -ux, uy, -uy,
                                (ux * ux - uy * uy) / phi, ux * uy / phi])
        src = rho * torch.stack([0 * T, 6 * uF / phi, -6 * uF / phi, Fx, -Fx, Fy, -Fy,
                                 2 * (ux * Fx - uy * Fy) / phi, (ux * Fy + uy * Fx) / phi])
        d = self.M @ f
        f = self.Mi @ (d - self.s * (d - eq) + (1 - self.s / 2) * src)
        sr = self.hf * (Tm - T)
        S = sr + 0.5 * (sr - self.before)
        self.before = sr
        jx, jy, o = T * ux / phi, T * uy / phi, 0 * T
        cf, cm, vp = self.cf * T, self.cm * Tm, self.varpi
        if self.q == 9:
            eg = torch.stack([m["H"], -4 * m["H"] + 2 * cf, 4 * m["H"] - 3 * cf, jx, -jx, jy, -jy, o, o])
            eh = torch.stack([Tm, -4 * Tm + 2 * cm, 4 * Tm - 3 * cm, o, o, o, o, o, o])
            unit = self.col([1, -2, 1, 0, 0, 0, 0, 0, 0])
        else:
            eg, eh = torch.stack([m["H"], jx, jy, vp * cf, o]), torch.stack([Tm, o, o, vp * cm, o])
            unit = self.col([1, 0, 0, vp, 0])
        d = self.Mt @ self.g
        g = self.Mti @ (d - self.z * (d - eg) + unit * S)
        d = self.Mt @ self.h
        h = self.Mti @ (d - self.e * (d - eh) - unit * (S * (self.hm / self.hf)))
        nx, ny = self.shape
        self.f, self.g, self.h = (torch.stack([torch.roll(q[i].reshape(ny, nx), (_E[i][1], _E[i][0]), (0, 1))
                                               for i in range(len(q))]).reshape(len(q), -1) for q in (f, g, h))
        self._walls()

    def _walls(self):
        """Non-equilibrium extrapolation from the inward neighbour (Eq. 52 and its thermal analogues)."""
        f, g, h = (q[:, self.partner] for q in (self.f, self.g, self.h))
        m, phi = self._macros(f, g, h), self.phi
        T, H, Tm = (torch.where(self.iso, a, b) for a, b in ((self.Tw, m["T"]), (self._H(self.Tw), m["H"]), (self.Tw, m["Tm"])))
        eu = torch.stack([e[0] * m["ux"] + e[1] * m["uy"] for e in _E])
        uu = m["ux"] ** 2 + m["uy"] ** 2
        f = f - self.w * m["rho"] * (3 * eu + 4.5 * eu * eu / phi - 1.5 * uu / phi)
        cs2 = 1 / 3 if self.q == 9 else self.varpi / 2
        move = self.wt * (m["T"] / (cs2 * phi)) * eu[:self.q]
        g = g + self._rest(H, T, self.cf) - self._rest(m["H"], m["T"], self.cf) - move
        h = h + self._rest(Tm, Tm, self.cm) - self._rest(m["Tm"], m["Tm"], self.cm)
        self.f[:, self.wall], self.g[:, self.wall], self.h[:, self.wall] = f, g, h

    def fields(self):
        m = self._macros(self.f, self.g, self.h)
        nx, ny = self.shape
        if not self.gbeta:  # nothing drives the flow: its rounding is not the solution
            m["ux"] = m["uy"] = torch.zeros_like(m["ux"])
        return {k: m[n].reshape(ny, nx) for k, n in zip(_FIELDS, ("ux", "uy", "T", "Tm", "fl", "rho"))}
