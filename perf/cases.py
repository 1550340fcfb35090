"""Workloads for timing the patch-group solver through its public entry points.

Each case is one pass of something a simulation program does over and over:

  box     one step of a periodic box held in patch-group order: hydro.step_box with the time step on the device, then the FP64 time step
          and conserved sums of the new state (hydro.cfl_dt_sums);
  groups  the ghosted-groups interface: hydro.fill_ghosts_periodic, then hydro.solve_groups with the fluxes on the group faces;
  serve   one tick of the continuous-batching server's GPU backend over a mix of resident simulations;
  amr     one step of the patch groups of three refinement levels: hydro.fill_groups_amr, then one hydro.solve_batch over all levels, with
          face fluxes;
  sync    the end of a coarse AMR step: a box step that stores the fluxes on every patch face, the average of the fine fluxes over two
          sub-steps (hydro.accumulate) and the coarse-grid correction (hydro.amr_correct).

Inputs are seeded smooth random fields of the kind of workloads.lognormal_blast_box (lognormal density, velocities of about Mach 1, hot
spheres), formed on the GPU, so that large boxes are quick to make.  exact() evaluates the published schemes in FP64 with plain torch
operations on whole arrays.
"""
import math
import time

import numpy as np
import torch

from paper_1103_3373_amd import hydro as H
from paper_1103_3373_amd import serve as S
from paper_1103_3373_amd import workloads as W

MHM, VL, CTU = 0, 1, 2
PLM, PPM = 0, 1
ROE, HLLC, HLLE, EXACT = 0, 1, 2, 3
GMINMOD, VANLEER, VANALBADA, HYBRID = 0, 1, 2, 3
CFL = {MHM: 0.3, VL: 0.3, CTU: 0.5}
GHOST = {(MHM, PLM): 2, (MHM, PPM): 3, (VL, PLM): 3, (VL, PPM): 4, (CTU, PLM): 2, (CTU, PPM): 3}


def _box(name, nx, ny, nz, scheme, recon=PPM, riemann=HLLC, limiter=VANLEER, char=True, f64=False, ic="blast", gamma=1.4, kind="box"):
    return {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "scheme": scheme, "recon": recon, "riemann": riemann,
            "limiter": limiter, "char": char, "f64": f64, "ic": ic, "gamma": gamma}


def listed():
    return [
        # The parity set-up: a Sod tube on 8 groups in FP64, primitive PLM and Roe at gamma 5/3.  Latency and launches.
        _box("sod_32_f64", 32, 32, 32, MHM, PLM, ROE, char=False, f64=True, ic="sod", gamma=5.0 / 3.0),
        # The smallest boxes of the request stream, one step each.
        _box("box_32", 32, 32, 32, CTU),
        _box("box_64_vl_roe", 64, 64, 64, VL, riemann=ROE, ic="smooth"),
        # Its largest.
        _box("box_128_mhm", 128, 128, 128, MHM),
        # Unequal sides, another limiter on primitive variables, PLM.
        _box("box_ragged_plm", 80, 48, 144, CTU, PLM, HLLE, VANALBADA, char=False),
        # A reference run in FP64.
        _box("box_96_f64", 96, 96, 96, CTU, f64=True),
        # The uniform-mesh benchmark.
        _box("box_256", 256, 256, 256, CTU),
        # A program that prepares its ghost cells itself and keeps the boundary fluxes.
        _box("groups_vl_flux", 128, 96, 80, VL, riemann=HLLE, kind="groups"),
        # Reference solutions with the exact Riemann solver.
        _box("groups_exact", 32, 32, 64, MHM, PLM, EXACT, f64=True, ic="smooth", kind="groups"),
        # A server tick with ten simulations of all sizes, schemes and solvers (n:scheme:riemann).
        {"name": "serve_tick", "kind": "serve", "sims": "32:2:1,64:0:0,128:1:1,32:0:1,64:2:0,64:1:0,32:1:1,128:2:1,64:0:1,32:2:0"},
        # The AMR benchmark: 2048, 6144 and 12288 groups on three levels.
        {"name": "amr_step", "kind": "amr", "n0": 2048, "n1": 6144, "n2": 12288, "base": 256, "coarse": 64, "scheme": CTU, "recon": PPM,
         "riemann": ROE, "f64": False},
        # The coarse-grid correction of a complete 256^3 coarse level under 6144 fine groups.
        {"name": "sync_256", "kind": "sync", "n": 256, "fine": 6144, "riemann": ROE, "f64": False},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choices(("box", "groups", "serve", "amr", "sync"), (10, 4, 2, 3, 2))[0]
    if kind in ("box", "groups"):
        # The production options mostly; every scheme, solver, limiter and mode now and then.
        usual = rng.random() < 0.6
        f64 = rng.random() < 0.3
        scheme = rng.choice((MHM, VL, CTU))
        recon = PPM if usual else rng.choice((PLM, PPM))
        riemann = rng.choice((ROE, HLLC) if usual else (ROE, HLLC, HLLE))
        limiter = VANLEER if usual else rng.choice((GMINMOD, VANLEER, VANALBADA, HYBRID))
        char = True if usual else rng.random() < 0.5
        most = 512 if f64 else (1500 if kind == "groups" else 4096)
        if kind == "groups" and rng.random() < 0.2:
            riemann, f64, most = EXACT, True, 64
        while True:
            m = _log(rng, 8, most) ** (1 / 3)
            g = [max(1, min(16, round(m * _log(rng, 0.6, 1.67)))) for _ in range(3)]
            if 4 <= g[0] * g[1] * g[2] <= most:
                break
        c = _box("", 16 * g[0], 16 * g[1], 16 * g[2], scheme, recon, riemann, limiter, char, f64,
                 rng.choice(("blast", "smooth")), 1.4, kind)
        del c["name"]
        return c
    if kind == "serve":
        sims = ["%d:%d:%d" % (rng.choice((32, 64, 128)), rng.choice((MHM, VL, CTU)), rng.choice((ROE, HLLC))) for _ in range(rng.randint(2, 16))]
        return {"kind": "serve", "sims": ",".join(sims)}
    if kind == "amr":
        base = rng.choice((64, 128, 256))
        most = min(2048, (base // 16) ** 3)
        n0 = int(_log(rng, 8, most))
        return {"kind": "amr", "n0": n0, "n1": int(n0 * rng.uniform(1, 3)), "n2": int(n0 * rng.uniform(1, 6)), "base": base,
                "coarse": rng.choice((32, 64)), "scheme": CTU, "recon": rng.choice((PLM, PPM)), "riemann": rng.choice((ROE, HLLC)),
                "f64": rng.random() < 0.25 and n0 < 400}
    n = 16 * rng.randint(4, 16)
    return {"kind": "sync", "n": n, "fine": int(_log(rng, 8, 0.2 * (n // 8) ** 3 + 10)), "riemann": rng.choice((ROE, HLLC)),
            "f64": rng.random() < 0.25 and n <= 128}


# ---- inputs -----------------------------------------------------------------
def _rng(seed):
    return np.random.default_rng(int(seed))


def _modes(shape, rng, count, kmax=8, modes=20):
    """`count` smooth periodic random fields [count, nz, ny, nx] of unit variance: sums of plane waves."""
    out = []
    for _ in range(count):
        k = rng.integers(-kmax // 2, kmax // 2 + 1, size=(modes, 3))
        k[np.all(k == 0, axis=1), 0] = 1
        ph, amp = rng.uniform(0, 2 * np.pi, modes), rng.uniform(0.5, 1.5, modes)
        amp *= np.sqrt(2.0 / np.sum(amp * amp))
        e = []
        for ax in range(3):
            x = (torch.arange(shape[ax], dtype=torch.float64, device="cuda") + 0.5) / shape[ax]
            e.append(torch.from_numpy(2 * np.pi * k[:, ax].astype(np.float64)).cuda()[:, None] * x)
        pz = e[0] + torch.from_numpy(ph).cuda()[:, None]
        zy = (pz[:, :, None] + e[1][:, None, :]).reshape(modes, -1)
        a = torch.from_numpy(amp).cuda()[:, None]
        f = (a * torch.cos(zy)).t().contiguous() @ torch.cos(e[2]) - (a * torch.sin(zy)).t().contiguous() @ torch.sin(e[2])
        out.append(f.reshape(shape))
    return torch.stack(out)


def _state(shape, seed, ic, gamma):
    """Conserved FP64 state [5, nz, ny, nx] of a seeded initial condition."""
    rng = _rng(seed)
    nz, ny, nx = shape
    if ic == "sod":
        x = (torch.arange(nx, device="cuda") + 0.5) / nx
        left = (x < 0.5).expand(shape)
        noise = torch.from_numpy(rng.uniform(-1e-3, 1e-3, size=shape)).cuda()
        rho = torch.where(left, 1.0, 0.125).double() * (1 + noise)
        p = torch.where(left, 1.0, 0.1).double()
        vel = torch.zeros((3,) + tuple(shape), dtype=torch.float64, device="cuda")
    else:
        f = _modes(shape, rng, 4)
        rho = torch.exp(0.5 * f[0] - 0.125)
        vel = f[1:] * math.sqrt(gamma / 3.0)
        p = torch.ones_like(rho)
        if ic == "blast":  # four hot spheres
            r = min(8.0, min(shape) / 6.0)
            ax = [torch.arange(n, device="cuda") + 0.5 for n in shape]
            for _ in range(4):
                d2 = 0.0
                for q in range(3):
                    d = (ax[q] - rng.uniform(0, shape[q])).abs()
                    d = torch.minimum(d, shape[q] - d) ** 2
                    d2 = d2 + d.reshape([-1 if a == q else 1 for a in range(3)])
                p = torch.where(d2 <= r * r, 100.0, p)
    E = p / (gamma - 1) + 0.5 * rho * (vel * vel).sum(0)
    return torch.cat([rho[None], rho * vel, E[None]])


def _grouped(box):
    _, nz, ny, nx = box.shape
    return box.reshape(5, nz // 16, 16, ny // 16, 16, nx // 16, 16).permute(1, 3, 5, 0, 2, 4, 6).reshape(-1, 5, 16, 16, 16).contiguous()


def _ungrouped(g, shape):
    nz, ny, nx = shape
    return g.reshape(nz // 16, ny // 16, nx // 16, 5, 16, 16, 16).permute(3, 0, 4, 1, 5, 2, 6).reshape(5, nz, ny, nx)


def _signal(U, gamma):
    """The largest max_d |v_d| + c over a conserved FP64 state with its variables along the first axis."""
    v = U[1:4] / U[0]
    p = (gamma - 1) * (U[4] - 0.5 * (U[1:4] * v).sum(0))
    return (v.abs().amax(0) + torch.sqrt(gamma * p / U[0])).max()


def _dtype(case):
    return torch.float64 if case["f64"] else torch.float32


def _options(case):
    return {"scheme": case["scheme"], "recon": case["recon"], "riemann": case["riemann"], "limiter": case["limiter"], "char": case["char"]}


def _box_input(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    box = _state(shape, seed, case["ic"], case["gamma"]).to(_dtype(case))
    dh = 1.0 / max(shape)
    dt = CFL[case["scheme"]] * dh / _signal(box.double(), case["gamma"]).reshape(1)
    return box, dh, dt


def _serve_sims(case, seed):
    """(request, initial box) of every simulation."""
    ics, found = ("sod", "blast", "smooth"), []
    for i, text in enumerate(case["sims"].split(",")):
        n, scheme, riemann = (int(v) for v in text.split(":"))
        ic = ics[i % 3] if scheme != CTU else ics[1 + i % 2]
        req = S.Request(id=i, arrival=0.0, n=n, scheme=scheme, riemann=riemann, ic=ic, seed=1000 * int(seed) + i, steps=1 << 30)
        found.append((req, _state((n, n, n), req.seed, ic, 1.4).float()))
    return found


def _trilinear(field, layout, lo, hi, dh_of_level, cn):
    """Trilinear interpolation of a periodic field [5, cn, cn, cn] at the centres of cells lo..hi-1 of every group: [5, n, z, y, x]."""
    c = torch.arange(lo, hi, device=field.device)
    ix, w = [], []
    for ax in (3, 2, 1):  # z, y, x
        X = (layout[:, ax, None].double() + c + 0.5) * dh_of_level[layout[:, 0].long(), None] * cn - 0.5
        f = torch.floor(X)
        ix.append((f.long() % cn, (f.long() + 1) % cn))
        w.append((1 - (X - f), X - f))
    out = 0.0
    for a in (0, 1):
        for b in (0, 1):
            for d in (0, 1):
                v = field[:, ix[0][a][:, :, None, None], ix[1][b][:, None, :, None], ix[2][d][:, None, None, :]]
                out = out + v * (w[0][a][:, :, None, None] * w[1][b][:, None, :, None] * w[2][d][:, None, None, :])
    return out


ALPHA = (0.5, 0.25, 0.875)  # sub-step times within the coarse step, by level
AMR_GAMMA = 1.4


def _amr_input(case, seed):
    cn, base = case["coarse"], case["base"]
    c0 = _state((cn,) * 3, seed, "blast", AMR_GAMMA)
    c1 = 0.97 * c0 + 0.03 * _state((cn,) * 3, seed + 500009, "smooth", AMR_GAMMA)
    c0, c1 = c0.to(_dtype(case)), c1.to(_dtype(case))
    layout = torch.from_numpy(W.amr_layout((case["n0"], case["n1"], case["n2"]), base_n=base, seed=int(seed))).cuda()
    dhs = torch.tensor([1.0 / (base << l) for l in range(3)], dtype=torch.float64, device="cuda")
    fine = torch.empty((layout.shape[0], 5, 16, 16, 16), dtype=_dtype(case), device="cuda")
    for q in range(0, layout.shape[0], 1024):
        mid = (0.7 * c0 + 0.3 * c1).double()
        fine[q:q + 1024] = _trilinear(mid, layout[q:q + 1024], 0, 16, dhs, cn).transpose(0, 1)
    dt = 0.5 / base / _signal(c0.double(), AMR_GAMMA).reshape(1)
    return c0, c1, layout, dhs, fine, dt


def _sync_input(case, seed):
    n, dt_ = case["n"], _dtype(case)
    coarse = _grouped(_state((n,) * 3, seed, "blast", AMR_GAMMA).to(dt_))
    dt = 0.5 / n / float(_signal(coarse.double().transpose(0, 1), AMR_GAMMA))
    layout = torch.from_numpy(W.amr_layout((0, case["fine"]), base_n=n, seed=int(seed))).cuda()
    layout[:, 0] = 0
    gen = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))
    fine = torch.rand((case["fine"], 5, 16, 16, 16), dtype=dt_, device="cuda", generator=gen) + 0.5
    flux = [torch.randn((case["fine"], 3, 2, 5, 16, 16), dtype=dt_, device="cuda", generator=gen) for _ in range(2)]
    return coarse, dt, layout, fine, flux


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("box", "groups"):
        box, dh, dt = _box_input(case, seed)
        s.update(dh=dh, dt=dt, dt_host=float(dt))
        G = (case["nx"] // 16) * (case["ny"] // 16) * (case["nz"] // 16)
        s["out"] = torch.empty((G, 5, 16, 16, 16), dtype=box.dtype, device="cuda")
        if kind == "box":
            s["in"] = _grouped(box)
            s["new_dt"] = torch.empty(1, dtype=torch.float64, device="cuda")
            s["sums"] = torch.empty(5, dtype=torch.float64, device="cuda")
        else:
            s["in"] = box.contiguous()
            N = 16 + 2 * GHOST[case["scheme"], case["recon"]]
            s["ghosted"] = torch.empty((G, 5, N, N, N), dtype=box.dtype, device="cuda")
            s["flux"] = torch.empty((G, 3, 2, 5, 16, 16), dtype=box.dtype, device="cuda")
    elif kind == "serve":
        sims = _serve_sims(case, seed)
        cache = {(r.ic, r.n, r.seed): _grouped(b).cpu().pin_memory() for r, b in sims}
        s["backend"] = S.GpuBackend(gamma=1.4, ic_cache=cache)
        s["backend"].start(time.perf_counter, time.perf_counter())
        s["handles"] = [s["backend"].admit(r) for r, _ in sims]
    elif kind == "amr":
        c0, c1, layout, dhs, fine, dt = _amr_input(case, seed)
        n, g = layout.shape[0], GHOST[case["scheme"], case["recon"]]
        s.update(c0=c0, c1=c1, layout=layout, fine=fine, dt=dt, g=g, ng0=case["base"] // 16, n=n)
        s["map"] = H.build_group_map(layout, s["ng0"], 3)
        s["ghosted"] = torch.empty((n, 5) + (16 + 2 * g,) * 3, dtype=fine.dtype, device="cuda")
        s["out"] = torch.empty_like(fine)
        s["flux"] = torch.empty((n, 3, 2, 5, 16, 16), dtype=fine.dtype, device="cuda")
        rows, first = [], 0
        for lev, count in enumerate((case["n0"], case["n1"], case["n2"])):
            at = slice(first, first + count)
            rows.append((s["ghosted"][at], s["out"][at], s["flux"][at], dt, 0.5 ** lev, 1.0 / (case["base"] << lev), first, count))
            first += count
        s["table"] = H.seg_table(rows, "cuda")
        s["spec"] = H.make_spec(case["scheme"], case["recon"], case["riemann"], gamma=AMR_GAMMA, char=True, f64=case["f64"])
    else:
        coarse, dt, layout, fine, flux = _sync_input(case, seed)
        n, G = case["n"], coarse.shape[0]
        s.update(coarse=coarse, dt_host=dt, layout=layout, fine=fine, fine_flux=flux, n=n)
        s["dt"] = torch.tensor([dt], dtype=torch.float64, device="cuda")
        s["map"] = H.build_group_map(layout, n // 8, 1)
        s["new"] = torch.empty_like(coarse)
        s["flux"] = torch.empty((G, 3, 3, 5, 16, 16), dtype=coarse.dtype, device="cuda")
        s["mean"] = torch.empty_like(flux[0])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "box":
        H.step_box(s["in"], s["out"], (case["nx"], case["ny"], case["nz"]), s["dt"], dh=s["dh"], gamma=case["gamma"], **_options(case))
        H.cfl_dt_sums(s["out"], s["dh"], case["gamma"], CFL[case["scheme"]], dt_out=s["new_dt"], sums_out=s["sums"])
        return s["out"], s["new_dt"], s["sums"]
    if kind == "groups":
        H.fill_ghosts_periodic(s["in"], GHOST[case["scheme"], case["recon"]], out=s["ghosted"])
        H.solve_groups(s["ghosted"], s["out"], s["flux"], dt=s["dt_host"], dh=s["dh"], gamma=case["gamma"], **_options(case))
        return s["ghosted"], s["out"], s["flux"]
    if kind == "serve":
        s["backend"].tick(s["handles"])
        return [(h.b if h.flip else h.a, h.dt) for h in s["handles"]]
    if kind == "amr":
        H.fill_groups_amr(s["fine"], s["layout"], s["map"], s["ng0"], ALPHA, s["c0"], s["c1"], s["g"], out=s["ghosted"])
        H.solve_batch(s["table"], 3, s["n"], s["spec"])
        return s["ghosted"], s["out"], s["flux"]
    n = s["n"]
    H.step_box(s["coarse"], s["new"], (n, n, n), s["dt"], dh=1.0 / n, gamma=AMR_GAMMA, scheme=CTU, recon=PPM, riemann=case["riemann"],
               char=True, flux=s["flux"], flux_mid=True)
    s["mean"].zero_()
    for x in s["fine_flux"]:
        H.accumulate(s["mean"], x, 0.5)
    H.amr_correct(s["new"], n, s["flux"], s["fine"], s["layout"], s["map"], s["mean"], s["dt_host"], 1.0 / n)
    return s["new"], s["mean"], s["flux"]


# Operations per cell update with HLLC on primitive variables, counted on a periodic box; characteristic limiting and the other solvers add
# to it (oracle/opcounts.json).
_OPS = {(MHM, PLM): 1043.3, (MHM, PPM): 1486.8, (VL, PLM): 1211.3, (VL, PPM): 1654.8, (CTU, PLM): 1904.3, (CTU, PPM): 2572.8}
_SOLVES = {MHM: 3, VL: 6, CTU: 6}
_SOLVE_OPS = {HLLC: 0.0, HLLE: 15.0, ROE: 136.0, EXACT: 600.0}


def _ops(scheme, recon, riemann, char):
    return _OPS[scheme, recon] + (0.0 if not char else 121.1 if recon == PPM else 241.3) + _SOLVES[scheme] * _SOLVE_OPS[riemann]


def work(case):
    kind = case["kind"]
    if kind == "serve":
        sims = [tuple(int(v) for v in t.split(":")) for t in case["sims"].split(",")]
        return {"bytes": sum(40.0 * n ** 3 for n, _, _ in sims), "flops": sum((_ops(a, PPM, b, True) + 25) * n ** 3 for n, a, b in sims)}
    e = 8.0 if case["f64"] else 4.0
    if kind in ("box", "groups"):
        cells = case["nx"] * case["ny"] * case["nz"]
        flops = cells * _ops(case["scheme"], case["recon"], case["riemann"], case["char"])
        if kind == "box":
            return {"bytes": 10 * e * cells, "flops": flops + 25 * cells}
        N = 16 + 2 * GHOST[case["scheme"], case["recon"]]
        return {"bytes": e * cells * (10 + 5 * N ** 3 / 4096 + 30 * 256 / 4096), "flops": flops}
    if kind == "amr":
        n, N = case["n0"] + case["n1"] + case["n2"], 16 + 2 * GHOST[case["scheme"], case["recon"]]
        return {"bytes": n * e * (10 * 4096 + 5 * N ** 3 + 30 * 256), "flops": n * 4096 * _ops(case["scheme"], case["recon"], case["riemann"], True)}
    cells = case["n"] ** 3
    return {"bytes": e * (10 * cells + cells // 4096 * 45 * 256 + case["fine"] * (5 * 4096 + 3 * 30 * 256)),
            "flops": cells * _ops(CTU, PPM, case["riemann"], True) + case["fine"] * (5 * 4096 + 4 * 30 * 256)}


# ---- the same in 64 bits, on whole arrays -------------------------------------
class _Reference:
    """One step of a scheme on conserved FP64 arrays [5, ..., z, y, x]; every array is treated as periodic, so with ghost layers the
    interior alone is meant."""

    def __init__(self, scheme, recon, riemann, limiter, char, gamma):
        self.scheme, self.recon, self.rs, self.lim, self.char, self.g = scheme, recon, riemann, limiter, char, gamma

    @staticmethod
    def at(a, d, k):
        return torch.roll(a, -k, dims=a.dim() - 1 - d)

    def prim(self, U):
        v = U[1:4] / U[0]
        return torch.cat([U[:1], v, ((self.g - 1) * (U[4] - 0.5 * (U[1:4] * v).sum(0)))[None]])

    def cons(self, W):
        return torch.cat([W[:1], W[0] * W[1:4], (W[4] / (self.g - 1) + 0.5 * W[0] * (W[1:4] ** 2).sum(0))[None]])

    @staticmethod
    def floor(W):
        W[0].clamp_(min=1e-10)
        W[4].clamp_(min=1e-10)
        return W

    def flux(self, W, d):
        U = self.cons(W)
        F = U * W[1 + d]
        F[1 + d] += W[4]
        F[4] += W[4] * W[1 + d]
        return F

    def limit(self, a, b):
        c, t = 0.5 * (a + b), 1.5
        if self.lim == VANLEER:
            r = 2 * a * b / (a + b)
        elif self.lim == VANALBADA:
            r = a * b * (a + b) / (a * a + b * b)
        else:
            r = torch.minimum(torch.minimum(t * a.abs(), t * b.abs()), c.abs())
            if self.lim == HYBRID:
                r = torch.minimum(r, (2 * a * b / (a + b)).abs())
            r = r * torch.sign(c)
        return torch.where(a * b > 0, r, 0.0)

    # Amplitudes: slot 0 the wave u - c, slot 1 + d the wave u + c, slot 4 the entropy wave, the transverse velocities as they are.
    def project(self, W, c, d, x):
        a, n = x.clone(), 1 + d
        p, v = 0.5 * x[4] / c ** 2, 0.5 * W[0] / c * x[n]
        a[0], a[n], a[4] = p - v, p + v, x[0] - x[4] / c ** 2
        return a

    def expand(self, W, c, d, a):
        x, n = a.clone(), 1 + d
        x[0], x[n], x[4] = a[0] + a[4] + a[n], c / W[0] * (a[n] - a[0]), c ** 2 * (a[0] + a[n])
        return x

    def faces(self, W, d):
        c = torch.sqrt(self.g * W[4] / W[0])
        lo, hi = W - self.at(W, d, -1), self.at(W, d, 1) - W
        if self.char:
            s = self.expand(W, c, d, self.limit(self.project(W, c, d, lo), self.project(W, c, d, hi)))
        else:
            s = self.limit(lo, hi)
        del lo, hi
        if self.recon == PPM:
            up = self.at(W, d, 1)
            e = 0.5 * (W + up) - (self.at(s, d, 1) - s) / 6
            e = torch.maximum(torch.minimum(e, torch.maximum(W, up)), torch.minimum(W, up))
            l, r = self.at(e, d, -1), e
            peak = (r - W) * (W - l) <= 0
            x, y = r - l, 6 * (W - 0.5 * (l + r))
            l2 = torch.where(peak, W, torch.where(x * y > x * x, 3 * W - 2 * r, l))
            r2 = torch.where(peak, W, torch.where(x * y < -x * x, 3 * W - 2 * l, r))
            l, r = l2, r2
        else:
            l, r = W - 0.5 * s, W + 0.5 * s
            if self.char:
                for f, k in ((l, -1), (r, 1)):
                    nb = self.at(W, d, k)
                    f.copy_(torch.maximum(torch.minimum(f, torch.maximum(W, nb)), torch.minimum(W, nb)))
        return l, r, c

    def trace(self, W, l, r, c, d, h):
        """Characteristic tracing to the half step; h = dt / dh."""
        x = r - l
        six = 6 * (W - 0.5 * (l + r)) if self.recon == PPM else torch.zeros_like(W)
        u = W[1 + d]
        speed = {0: (u - c) * h, 1 + d: (u + c) * h}
        top, low = speed[1 + d].clamp(min=0), speed[0].clamp(max=0)
        R = r - 0.5 * top * (x - (1 - 2 / 3 * top) * six)
        L = l - 0.5 * low * (x + (1 + 2 / 3 * low) * six)
        dx, d6 = self.project(W, c, d, x), self.project(W, c, d, six)
        aR, aL = torch.zeros_like(W), torch.zeros_like(W)
        for k in range(5):
            s = speed.get(k, u * h)
            v = 0.5 * (top - s) * (dx[k] - d6[k]) + (top * top - s * s) / 3 * d6[k]
            aR[k] = torch.where(s > 0, v, 0.0)
            v = 0.5 * (low - s) * (dx[k] + d6[k]) + (low * low - s * s) / 3 * d6[k]
            aL[k] = torch.where(s < 0, v, 0.0)
        return L + self.expand(W, c, d, aL), R + self.expand(W, c, d, aR)

    def solve(self, L, R, d):
        if self.rs == EXACT:
            return self.exact(L, R, d)
        n, g = 1 + d, self.g
        UL, UR = self.cons(L), self.cons(R)
        FL, FR = self.flux(L, d), self.flux(R, d)
        sl, sr = torch.sqrt(L[0]), torch.sqrt(R[0])
        v = (sl * L[1:4] + sr * R[1:4]) / (sl + sr)
        Hm = ((UL[4] + L[4]) / sl + (UR[4] + R[4]) / sr) / (sl + sr)
        c2 = (g - 1) * (Hm - 0.5 * (v * v).sum(0))
        c, u = torch.sqrt(c2.clamp(min=0)), v[d]
        SL = torch.minimum(L[n] - torch.sqrt(g * L[4] / L[0]), u - c)
        SR = torch.maximum(R[n] + torch.sqrt(g * R[4] / R[0]), u + c)
        if self.rs == HLLC:
            mL, mR = L[0] * (SL - L[n]), R[0] * (SR - R[n])
            star = (R[4] - L[4] + mL * L[n] - mR * R[n]) / (mL - mR)
            F = torch.where(star >= 0, self._star(L, UL, FL, SL, mL, star, n), self._star(R, UR, FR, SR, mR, star, n))
            return torch.where(SL >= 0, FL, torch.where(SR <= 0, FR, F))
        lo, hi = SL.clamp(max=0), SR.clamp(min=0)
        hlle = (hi * FL - lo * FR + hi * lo * (UR - UL)) / (hi - lo)
        if self.rs == HLLE:
            return hlle
        dU = UR - UL
        t = [k for k in (1, 2, 3) if k != n]
        q2 = (v * v).sum(0)
        at = {k: dU[k] - v[k - 1] * dU[0] for k in t}
        dE = dU[4] - sum(at[k] * v[k - 1] for k in t)
        a2 = (g - 1) / c ** 2 * (dU[0] * (Hm - u * u) + u * dU[n] - dE)
        a1 = (dU[0] * (u + c) - dU[n] - c * a2) / (2 * c)
        a5 = dU[0] - a1 - a2

        def wave(sign):
            K = torch.stack([torch.ones_like(u), v[0], v[1], v[2], Hm + sign * u * c])
            K[n] += sign * c
            return K
        K1, K5 = wave(-1.0), wave(1.0)
        ok = c2 > 0
        for X in (UL + a1 * K1, UR - a5 * K5):
            ok &= (X[0] > 0) & (self.prim(X)[4] > 0)
        D = (u - c).abs() * a1 * K1 + (u + c).abs() * a5 * K5
        K2 = torch.stack([torch.ones_like(u), v[0], v[1], v[2], 0.5 * q2])
        D += u.abs() * a2 * K2
        for k in t:
            D[k] += u.abs() * at[k]
            D[4] += u.abs() * at[k] * v[k - 1]
        return torch.where(ok, 0.5 * (FL + FR - D), hlle)

    def _star(self, Q, U, F, Sp, m, star, n):
        f = m / (Sp - star)
        X = f * Q
        X[0] = f
        X[n] = f * star
        X[4] = f * (U[4] / Q[0] + (star - Q[n]) * (star + Q[4] / m))
        return F + Sp * (X - U)

    def exact(self, L, R, d):
        """Flux of the exact solution of the Riemann problem, sampled on the face."""
        n, g = 1 + d, self.g
        G1, G2 = (g - 1) / (2 * g), (g + 1) / (2 * g)
        cL, cR = torch.sqrt(g * L[4] / L[0]), torch.sqrt(g * R[4] / R[0])
        du = R[n] - L[n]

        def curve(p, Q, c):
            A, B = 2 / ((g + 1) * Q[0]), (g - 1) / (g + 1) * Q[4]
            q = torch.sqrt(A / (p + B))
            shock = p > Q[4]
            f = torch.where(shock, (p - Q[4]) * q, 2 * c / (g - 1) * ((p / Q[4]) ** G1 - 1))
            return f, torch.where(shock, q * (1 - 0.5 * (p - Q[4]) / (B + p)), (p / Q[4]) ** -G2 / (Q[0] * c))
        p = torch.maximum(0.5 * (L[4] + R[4]) - 0.125 * du * (L[0] + R[0]) * (cL + cR), 1e-8 * torch.minimum(L[4], R[4]))
        for _ in range(40):
            (fL, dL), (fR, dR) = curve(p, L, cL), curve(p, R, cR)
            new = p - (fL + fR + du) / (dL + dR)
            p = torch.where(new < 0, 1e-12 * p, new)
        fL, fR = curve(p, L, cL)[0], curve(p, R, cR)[0]
        u = 0.5 * (L[n] + R[n]) + 0.5 * (fR - fL)

        def side(Q, c, sign):  # sign -1: the left state, +1: the right one
            vn = -sign * Q[n]  # velocity away from the wave, as on the left
            us, shock, pr = -sign * u, p > Q[4], p / Q[4]
            g6 = (g - 1) / (g + 1)
            rho = torch.where(shock, Q[0] * (pr + g6) / (g6 * pr + 1), Q[0] * pr ** (1 / g))
            head = torch.where(shock, vn - c * torch.sqrt(G2 * pr + G1), vn - c)
            tail = torch.where(shock, head, us - c * pr ** G1)
            b = (2 / (g + 1) + (g - 1) / ((g + 1) * c) * vn).clamp(min=0)
            fan = (head < 0) & (tail >= 0)
            star = (head < 0) & (tail < 0)
            X = Q.clone()
            X[0] = torch.where(star, rho, torch.where(fan, Q[0] * b ** (2 / (g - 1)), Q[0]))
            X[n] = -sign * torch.where(star, us, torch.where(fan, 2 / (g + 1) * (c + 0.5 * (g - 1) * vn), vn))
            X[4] = torch.where(star, p, torch.where(fan, Q[4] * b ** (2 * g / (g - 1)), Q[4]))
            return X
        return self.flux(torch.where(u >= 0, side(L, cL, -1.0), side(R, cR, 1.0)), d)

    def step(self, U, h):
        """The new state and the three fluxes (at the upper face of every cell) for h = dt / dh."""
        W0 = self.prim(U)
        at, diff = self.at, lambda F, d: F - self.at(F, d, -1)
        if self.scheme == VL:
            X = U.clone()
            for d in range(3):
                X -= 0.5 * h * diff(self.solve(W0, at(W0, d, 1), d), d)
            W0 = self.floor(self.prim(X))
            del X
        l, r = [None] * 3, [None] * 3
        for d in range(3):
            l[d], r[d], c = self.faces(W0, d)
            if self.scheme == CTU:
                l[d], r[d] = self.trace(W0, l[d], r[d], c, d, h)
            self.floor(l[d]), self.floor(r[d])
        if self.scheme == MHM:
            X = sum(self.flux(r[d], d) - self.flux(l[d], d) for d in range(3))
            for d in range(3):
                l[d], r[d] = (self.floor(self.prim(self.cons(f) - 0.5 * h * X)) for f in (l[d], r[d]))
            del X
        if self.scheme == CTU:
            D = [diff(self.solve(r[d], at(l[d], d, 1), d), d) for d in range(3)]
            for d in range(3):
                X = 0.5 * h * (D[(d + 1) % 3] + D[(d + 2) % 3])
                l[d], r[d] = (self.floor(self.prim(self.cons(f) - X)) for f in (l[d], r[d]))
            del D, X
        F = []
        for d in range(3):
            F.append(self.solve(r[d], at(l[d], d, 1), d))
            l[d] = r[d] = None
        out = U - h * sum(diff(F[d], d) for d in range(3))
        return out, F


def _group_fluxes(F, g, planes):
    """Fluxes [5, n, z, y, x] at upper cell faces of ghosted groups -> [n, 3, planes, 5, 16, 16]; plane offsets 0, 16 (and 8)."""
    out = []
    for d in range(3):
        f = F[d].transpose(0, 1)
        for ax in range(3):
            if ax != d:
                f = f.narrow(f.dim() - 1 - ax, g, 16)
        out.append(torch.stack([f.select(f.dim() - 1 - d, g + o - 1) for o in (0, 16, 8)[:planes]], 1))
    return torch.stack(out, 1)


def _solve_ghosted(ref, groups, g, h, planes=2, chunk=512):
    """Updated interiors and face fluxes of ghosted FP64 groups [n, 5, N, N, N] (h per group)."""
    outs, fluxes = [], []
    for q in range(0, groups.shape[0], chunk):
        U = groups[q:q + chunk].transpose(0, 1).contiguous()
        o, F = ref.step(U, h[q:q + chunk].reshape(-1, 1, 1, 1))
        outs.append(o[..., g:g + 16, g:g + 16, g:g + 16].transpose(0, 1).contiguous())
        fluxes.append(_group_fluxes(F, g, planes))
    return torch.cat(outs), torch.cat(fluxes)


def _windows(box, g):
    """Ghosted groups [G, 5, N, N, N] of a periodic box [5, nz, ny, nx]."""
    for d in range(3):
        n = box.shape[1 + 2 * d]
        i = (16 * torch.arange(n // 16, device=box.device)[:, None] + torch.arange(-g, 16 + g, device=box.device)) % n
        box = box.index_select(1 + 2 * d, i.reshape(-1)).unflatten(1 + 2 * d, tuple(i.shape))
    return box.permute(1, 3, 5, 0, 2, 4, 6).reshape(-1, 5, 16 + 2 * g, 16 + 2 * g, 16 + 2 * g)


def _ghosted_amr(case, c0, c1, layout, dhs, fine, lo, hi):
    """The padded input of groups lo..hi-1 in FP64."""
    g = GHOST[case["scheme"], case["recon"]]
    lay, out = layout[lo:hi].long(), None
    for lev in range(3):
        pick = (lay[:, 0] == lev).nonzero().reshape(-1)
        if not len(pick):
            continue
        ng = (case["base"] << lev) // 16
        all_ = (layout[:, 0] == lev).nonzero().reshape(-1)
        where = torch.full((ng, ng, ng), -1, dtype=torch.long, device="cuda")
        o = layout[all_].long() // 16
        where[o[:, 3], o[:, 2], o[:, 1]] = all_
        L = lay[pick]
        c = torch.arange(-g, 16 + g, device="cuda")
        z, y, x = ((L[:, ax, None] + c) % (16 * ng) for ax in (3, 2, 1))
        z, y, x = z[:, :, None, None], y[:, None, :, None], x[:, None, None, :]
        owner = where[z // 16, y // 16, x // 16]
        near = fine[owner.clamp(min=0), :, z % 16, y % 16, x % 16].movedim(-1, 1).double()
        blend = (1 - ALPHA[lev]) * c0.double() + ALPHA[lev] * c1.double()
        far = _trilinear(blend, L, -g, 16 + g, dhs, case["coarse"]).transpose(0, 1)
        v = torch.where((owner >= 0)[:, None], near, far)
        out = torch.empty((hi - lo,) + v.shape[1:], dtype=torch.float64, device="cuda") if out is None else out
        out[pick] = v
    return out


def _correct(U, h, F, fine, layout, mean):
    """Refluxing and restriction on an FP64 box [5, n, n, n] with the coarse fluxes F at the upper faces of its cells."""
    n = U.shape[-1]
    K = 0 * U[0].long()
    o = layout.long() // 2
    c8 = torch.arange(8, device="cuda")
    at = tuple((o[:, ax, None] + c8).reshape([-1] + [8 if a == q else 1 for a in range(3)]) for q, ax in ((0, 3), (1, 2), (2, 1)))
    K[at] = 1
    f = fine.double().reshape(-1, 5, 8, 2, 8, 2, 8, 2).mean((3, 5, 7))
    avg = mean.reshape(-1, 3, 2, 5, 8, 2, 8, 2).mean((5, 7))  # [fine, dir, side, var, slow, fast]
    out = U.clone()
    for d in range(3):
        ax = [k for k in (0, 1, 2) if k != 2 - d]  # slow and fast transverse axes of (z, y, x)
        for side in (0, 1):
            pos = [None] * 3
            for j, k in enumerate(ax):
                pos[k] = (o[:, 3 - k, None] + c8)[:, :, None] if j == 0 else (o[:, 3 - k, None] + c8)[:, None, :]
            edge = o[:, 1 + d, None, None]
            cell, face = (edge - 1, edge - 1) if side == 0 else (edge + 8, edge + 7)
            pos[2 - d] = cell % n
            idx = tuple(torch.broadcast_tensors(*pos))
            pos[2 - d] = face % n
            fc = F[d][(slice(None),) + tuple(torch.broadcast_tensors(*pos))]
            ff = avg[:, d, side].transpose(0, 1)
            keep = (K[idx] == 0).double()
            out.permute(1, 2, 3, 0).index_put_(idx, ((-1.0 if side == 0 else 1.0) * h * (ff - fc) * keep).movedim(0, -1), accumulate=True)
    out.permute(1, 2, 3, 0)[at] = f.permute(0, 2, 3, 4, 1)
    return out


def _grouped_fluxes(F):
    """Fluxes [5, n, n, n] at upper cell faces of a periodic box -> [G, 3, 3, 5, 16, 16] on the patch faces."""
    G = torch.stack([_grouped(f) for f in F], 1)  # upper faces
    low = torch.stack([_grouped(torch.roll(f, 1, dims=3 - d)) for d, f in enumerate(F)], 1)
    out = []
    for d in range(3):
        ax = 4 - d
        out.append(torch.stack([low[:, d].select(ax, 0), G[:, d].select(ax, 15), G[:, d].select(ax, 7)], 1))
    return torch.stack(out, 1)


@torch.no_grad()
def exact(case, seed):
    kind = case["kind"]
    if kind in ("box", "groups"):
        box, dh, dt = _box_input(case, seed)
        ref = _Reference(case["scheme"], case["recon"], case["riemann"], case["limiter"], case["char"], case["gamma"])
        if kind == "box":
            new, _ = ref.step(box.double(), dt / dh)
            return (_grouped(new), CFL[case["scheme"]] * dh / _signal(new, case["gamma"]).reshape(1),
                    dh ** 3 * torch.stack([v.sum() for v in new]))
        g = GHOST[case["scheme"], case["recon"]]
        groups = _windows(box, g).double()
        out, flux = _solve_ghosted(ref, groups, g, (dt / dh).expand(groups.shape[0]))
        return groups, out, flux
    if kind == "serve":
        outs = []
        for r, box in _serve_sims(case, seed):
            U, dh = box.double(), 1.0 / r.n
            dt = CFL[r.scheme] * dh / _signal(U, 1.4).reshape(1)
            new, _ = _Reference(r.scheme, PPM, r.riemann, VANLEER, True, 1.4).step(U, dt / dh)
            outs.append((_grouped(new), CFL[r.scheme] * dh / _signal(new, 1.4).reshape(1)))
        return outs
    if kind == "amr":
        c0, c1, layout, dhs, fine, dt = _amr_input(case, seed)
        ref = _Reference(case["scheme"], case["recon"], case["riemann"], VANLEER, True, AMR_GAMMA)
        parts = []
        for q in range(0, layout.shape[0], 512):
            e = min(q + 512, layout.shape[0])
            groups = _ghosted_amr(case, c0, c1, layout, dhs, fine, q, e)
            h = dt / dhs[0] + 0 * dhs[layout[q:e, 0].long()]  # dt and dh halve together from level to level
            parts.append((groups,) + _solve_ghosted(ref, groups, GHOST[case["scheme"], case["recon"]], h))
        return tuple(torch.cat(p) for p in zip(*parts))
    coarse, dt, layout, fine, flux = _sync_input(case, seed)
    n = case["n"]
    U = _ungrouped(coarse.double(), (n, n, n))
    new, F = _Reference(CTU, PPM, case["riemann"], VANLEER, True, AMR_GAMMA).step(U, dt * n)
    mean = 0.5 * flux[0].double() + 0.5 * flux[1].double()
    return _grouped(_correct(new, dt * n, F, fine, layout, mean)), mean, _grouped_fluxes(F)
