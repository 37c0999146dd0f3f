"""Performance cases of the library: what a program does with it, through the public entry points of
``paper_2603_15920_amd.binding``, over the range of sizes, types and options that its own workloads use.

Kinds of case

``explicit``  the explicit finite-volume operators on given fields: gradients, Laplacian, divergence,
              face interpolation and (FP64) the deferred correction; results in the user's order.
``poisson``   assembly of a diffusion system and its solve by CG (Jacobi or AMG), the manufactured
              Poisson workload.
``momentum``  assembly of the implicit momentum system, its BiCGStab solve (three components on one
              matrix), a transposed product.
``step``      PISO time steps from a given state, optionally followed by a passive scalar step or made
              in graph mode; the new state comes back.
``window``    a recorded window of steps and its reverse sweep.

Each function below works from plain case dicts; a drawn case is one more of the same kinds and ranges.
"""
import functools
import math

import numpy as np
import torch

from paper_2603_15920_amd import binding as B
from paper_2603_15920_amd import meshgen as mg

DEV = "cuda:0"


def listed():
    return [
        # the smallest whole run: the lid-driven cavity of 2,048 prisms, ten steps with the default
        # (Jacobi) pressure preconditioner; launches and round trips to the host are its time
        dict(name="cavity", kind="step", mesh="cavity", n=32, precond="jacobi", steps=10, graph=False, conv="upwind",
             time="backward_euler", scalar=False),
        # the same case as a program that steps it for long runs it: AMG, the step as a replayed graph
        dict(name="cavity_graph", kind="step", mesh="cavity", n=33, precond="amg", steps=10, graph=True, conv="upwind",
             time="backward_euler", scalar=False),
        # a straight tube of 50k cells with the higher-order options: QUICK, Crank-Nicolson, a
        # transported scalar after the steps
        dict(name="tube_options", kind="step", mesh="tube", n=43, precond="amg", steps=2, graph=False, conv="quick",
             time="crank_nicolson", scalar=True),
        # an ordinary channel between the small cases and the benchmark's
        dict(name="channel_163k", kind="step", mesh="channel", n=30, m=31, precond="amg", steps=2, graph=False,
             conv="upwind", time="backward_euler", scalar=False),
        # the benchmark's channel of 1,053,696 cells
        dict(name="channel_1m", kind="step", mesh="channel", n=56, m=56, precond="amg", steps=1, graph=False,
             conv="upwind", time="backward_euler", scalar=False),
        # many small simulations packed into one mesh, each with its own Reynolds number and outlet
        dict(name="batch", kind="step", mesh="batch", n=10, precond="jacobi", steps=1, graph=False, conv="upwind",
             time="backward_euler", scalar=False),
        # the differentiated form on a bifurcating tube: a recorded window and its reverse sweep
        dict(name="window_51k", kind="window", mesh="ybif", n=51000, precond="amg", steps=4, every=2),
        # the paper's Poisson verification sizes: its smallest with Jacobi, its largest with AMG
        dict(name="poisson_10k", kind="poisson", mesh="box", n=12, m=12, precond="jacobi"),
        dict(name="poisson_94k", kind="poisson", mesh="box", n=25, m=25, precond="amg"),
        # one implicit momentum system of ordinary size
        dict(name="momentum_163k", kind="momentum", mesh="channel", n=30, m=31),
        # the operators alone, at the benchmark's size in FP64 and at a smaller one in FP32
        dict(name="explicit_1m_f64", kind="explicit", mesh="channel", n=56, m=56, dtype="float64", scheme="upwind"),
        dict(name="explicit_94k_f32", kind="explicit", mesh="channel", n=25, m=25, dtype="float32", scheme="linear"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["explicit", "poisson", "momentum", "step", "step", "step", "window"])
    n, m = _log_int(rng, 8, 50), _log_int(rng, 8, 50)  # a box of n x n x m hexes, six tets each
    if kind == "explicit":
        return dict(kind=kind, mesh="channel", n=n, m=m, dtype=rng.choice(["float64", "float32"]),
                    scheme=rng.choice(["upwind", "linear"]))
    if kind == "poisson":
        amg = rng.random() < 0.5
        return dict(kind=kind, mesh="box", n=n if amg else min(n, 26), m=m if amg else min(m, 26),
                    precond="amg" if amg else "jacobi")
    if kind == "momentum":
        return dict(kind=kind, mesh="channel", n=n, m=m)
    if kind == "window":
        amg = rng.random() < 0.7
        return dict(kind=kind, mesh="ybif", n=_log_int(rng, 9000, 60000 if amg else 12000), precond="amg" if amg else "jacobi",
                    steps=4, every=rng.choice([2, 4]))
    shape = rng.choice(["cavity", "tube", "channel", "batch"])
    size = {"cavity": lambda: _log_int(rng, 10, 60), "tube": lambda: _log_int(rng, 10, 80), "channel": lambda: n,
            "batch": lambda: rng.randint(3, 12)}[shape]()
    c = dict(kind="step", mesh=shape, n=size, precond=rng.choice(["jacobi", "amg"]), steps=rng.randint(1, 3),
             graph=rng.random() < 0.25, conv=rng.choice(["upwind", "upwind", "linear", "sou", "quick"]),
             time=rng.choice(["backward_euler", "backward_euler", "crank_nicolson"]), scalar=rng.random() < 0.25)
    if shape == "channel":
        c["m"] = m
        if n * n * m > 10000:
            c["precond"] = "amg"
    if shape == "batch":
        c["precond"] = "jacobi"
        c["graph"] = c["scalar"] = False
    return c


# ------------------------------------------------------------------------------------------------
# meshes (host, made once per size; a program keeps its mesh)
# ------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=3)
def _source(shape, n, m):
    """(mesh, setup): the host mesh and, for flow cases, nu, dt, Ub, Windkessel rows per outlet, segments."""
    if shape == "box":
        # Dirichlet on every side
        return mg.kuhn_cube(n, patches="walls", nxyz=(n, n, m), seed=2603007), {}
    if shape == "channel":
        mesh = mg.kuhn_cube(n, patches="channel", nxyz=(n, n, m), seed=2603002)
        Ub = mg.box_channel_inlet(mesh)
        q = mg.inlet_flow(mesh, Ub)
        # the largest cells of a drawn box are coarse: the diffusion number stays in the stable range
        return mesh, dict(nu=0.005, dt=1e-3, Ub=Ub, wk=np.array([[1 / (9 * q), 0.1 * q, 1 / q]]))
    if shape == "cavity":
        mesh = mg.cavity(n)
        Ub = np.zeros((mesh.n_boundary_faces, 3))
        lid = mesh.patch("lid")
        Ub[lid.start - mesh.n_internal_faces:lid.start - mesh.n_internal_faces + lid.size, 0] = 1.0
        return mesh, dict(nu=0.01, dt=1e-3, Ub=Ub, wk=np.zeros((0, 3)))
    if shape == "tube":
        mesh = mg.tube(n=8, m=4, layers=n, L=0.05 * n, outlet="wk")
        Ub = np.zeros((mesh.n_boundary_faces, 3))
        p = mesh.patch("inlet")
        Ub[p.start - mesh.n_internal_faces:p.start - mesh.n_internal_faces + p.size] = \
            mg.parabolic_inlet(mesh.Cf[p.start:p.start + p.size], (0, 0, 0), 0.5, 1.0)
        wk = mg.windkessel_nominal(mesh, mg.inlet_flow(mesh, Ub), outlets=("outlet",))
        return mesh, dict(nu=1e-3, dt=1e-3, Ub=Ub, wk=wk)
    if shape == "ybif":
        mesh = mg.ybif(h=0.0519 * (401484 / n) ** (1 / 3))
        Ub = np.zeros((mesh.n_boundary_faces, 3))
        p = mesh.patch("inlet")
        Ub[p.start - mesh.n_internal_faces:p.start - mesh.n_internal_faces + p.size] = \
            mg.parabolic_inlet(mesh.Cf[p.start:p.start + p.size], (0, 0, 0), 0.5, 1.0)
        return mesh, dict(nu=1e-3, dt=1e-3, Ub=Ub, wk=mg.windkessel_nominal(mesh, mg.inlet_flow(mesh, Ub)))
    # n members of 2,000 to 30,000 cells side by side
    members = mg.batch_members(n, n_lo=2e3, n_hi=3e4)
    mesh, starts = mg.pack([b["mesh"] for b in members])
    nb = np.concatenate([[0], np.cumsum([b["mesh"].n_boundary_faces for b in members])])
    Ub = np.zeros((mesh.n_boundary_faces, 3))
    for k, b in enumerate(members):
        Ub[nb[k]:nb[k + 1]] = b["Ub"]
    return mesh, dict(nu=[b["nu"] for b in members], dt=1e-3, Ub=Ub, wk=np.concatenate([b["wk"] for b in members]),
                      starts=starts)


def _src(case):
    return _source(case["mesh"], case["n"], case.get("m", 0))


@functools.lru_cache(maxsize=1)
def _ctx():
    return B.Context(0)


@functools.lru_cache(maxsize=2)
def _mesh(shape, n, m):
    src, setup = _source(shape, n, m)
    return B.Mesh(_ctx(), src, seg_cell_start=setup.get("starts"))


def _dev(a, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device=DEV, dtype=dtype)


# ------------------------------------------------------------------------------------------------
# fields (from the seed alone)
# ------------------------------------------------------------------------------------------------

def _waves(x, seed, k):
    """The k-th smooth random field of this seed at the points x [n, 3]: six sines of low wave number."""
    r = np.random.default_rng([seed, k])
    a = r.standard_normal(6) / math.sqrt(6.0)
    kv = 2 * math.pi * r.integers(-3, 4, size=(6, 3))
    th = r.uniform(0, 2 * math.pi, 6)
    out = torch.zeros(x.shape[0], dtype=torch.float64, device=x.device)
    for q in range(6):
        out += float(a[q]) * torch.sin(x[:, 0] * float(kv[q, 0]) + x[:, 1] * float(kv[q, 1]) +
                                       x[:, 2] * float(kv[q, 2]) + float(th[q]))
    return out


def _waves3(x, seed, k):
    return torch.stack([_waves(x, seed, k + c) for c in range(3)], 1)


def _start_flow(case, seed, x):
    """A developed-looking state: the inlet's profile along the axis (none in the cavity), with a
    smooth perturbation, and a falling pressure."""
    lo, hi = x.min(0).values, x.max(0).values
    if case["mesh"] in ("cavity", "batch", "ybif"):
        U = torch.zeros_like(x)
    elif case["mesh"] == "tube":
        U = torch.zeros_like(x)
        U[:, 0] = (1 - 4 * (x[:, 1] ** 2 + x[:, 2] ** 2)).clamp(min=0)
    else:
        U = torch.zeros_like(x)
        U[:, 0] = 16 * x[:, 1] * (1 - x[:, 1]) * x[:, 2] * (1 - x[:, 2])
    pert = 0.02 * _waves3(x / (hi - lo).max(), seed, 20)
    if case["mesh"] == "cavity":
        pert[:, 2] = 0.0
    p = 0.1 * (hi[0] - x[:, 0]) + 0.01 * _waves(x / (hi - lo).max(), seed, 30)
    return U + pert, p


def _explicit_inputs(case, seed, C, Cf, Sf, nfi):
    """phi, phi_b, U, U_b and the flux of a smooth velocity, in user order and FP64 before rounding."""
    phi, phib = _waves(C, seed, 0), _waves(Cf[nfi:], seed, 0)
    U, Ub = _waves3(C, seed, 1), _waves3(Cf[nfi:], seed, 1)
    flux = (_waves3(Cf, seed, 1) * Sf).sum(1)
    dt = getattr(torch, case["dtype"])
    return [t.to(dt) for t in (phi, phib, U, Ub, flux)]


def _momentum_inputs(seed, C, Cf, Sf):
    U = _waves3(C, seed, 1)
    return U, (_waves3(Cf, seed, 1) * Sf).sum(1), _waves3(C, seed, 5)


# ------------------------------------------------------------------------------------------------
# prepare and run
# ------------------------------------------------------------------------------------------------

NU, DT = 0.005, 1e-3  # of the momentum system


def prepare(case, seed):
    src, setup = _src(case)
    M = _mesh(case["mesh"], case["n"], case.get("m", 0))
    kind = case["kind"]
    nc, nfi, nf = src.n_cells, src.n_internal_faces, src.n_faces
    empty = lambda *s, dtype=torch.float64: torch.empty(s, dtype=dtype, device=DEV)  # noqa: E731
    st = dict(case=case, M=M, src=src, setup=setup)
    if kind == "explicit":
        dt = getattr(torch, case["dtype"])
        phi, phib, U, Ub, flux = _explicit_inputs(case, seed, _dev(src.C), _dev(src.Cf), _dev(src.Sf), nfi)
        st.update(phi=M.to_internal(phi, B.KIND_CELL), phib=M.to_internal(phib, B.KIND_BFACE),
                  U=M.to_internal(U, B.KIND_CELL), Ub=M.to_internal(Ub, B.KIND_BFACE),
                  flux=M.to_internal(flux, B.KIND_FACE_FLUX), g=empty(nc, 3, dtype=dt), gU=empty(nc, 3, 3, dtype=dt),
                  lap=empty(nc, dtype=dt), div=empty(nc, 3, dtype=dt), face=empty(nf, dtype=dt), dc=empty(nc, 3, dtype=dt))
    elif kind == "poisson":
        amp = 1.0 + 0.5 * np.random.default_rng(seed).random()
        st.update(phib=M.to_internal(_dev(amp * mg.poisson_mms_solution(src.Cf[nfi:])), B.KIND_BFACE),
                  g=M.to_internal(_dev(amp * mg.poisson_mms_gradient(src.C)), B.KIND_CELL),
                  source=M.to_internal(_dev(amp * src.V * mg.poisson_mms_source(src.C)), B.KIND_CELL),
                  d=empty(nc), u=empty(nfi), rbc=empty(nc), lap=empty(nc), zero=torch.zeros(nc, dtype=torch.float64, device=DEV),
                  x=empty(nc), amg=None)
        st["A"] = B.ldu(st["d"], st["u"])
        if case["precond"] == "amg":
            B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, st["phib"], st["A"], st["rbc"])
            st["amg"] = _Amg(M, st["A"])
    elif kind == "momentum":
        U, flux, x0 = _momentum_inputs(seed, _dev(src.C), _dev(src.Cf), _dev(src.Sf))
        st.update(U=M.to_internal(U, B.KIND_CELL), flux=M.to_internal(flux, B.KIND_FACE_FLUX),
                  Ub=M.to_internal(_dev(setup["Ub"]), B.KIND_BFACE), x0=M.to_internal(x0, B.KIND_CELL), d=empty(nc),
                  u=empty(nfi), low=empty(nfi), b=empty(nc, 3), x=empty(nc, 3), y=empty(nc, 3))
        st["A"] = B.ldu(st["d"], st["u"], st["low"])
    else:
        window = kind == "window"
        prm = B.piso_params(setup["nu"] if np.isscalar(setup["nu"]) else 0.01, setup["dt"], maxit_p=20000, maxit_u=2000,
                            precond=case["precond"], conv=case.get("conv", "upwind"),
                            time=case.get("time", "backward_euler"))
        P = B.Piso(M, prm)
        if not np.isscalar(setup["nu"]):
            P.set_viscosity(setup["nu"])
        P.set_boundary(_dev(setup["Ub"]), torch.zeros(src.n_boundary_faces, dtype=torch.float64, device=DEV))
        x = _dev(src.C)
        U, p = _start_flow(case, seed, x)
        st.update(P=P, U=U.contiguous(), p=p.contiguous())
        if case.get("scalar"):
            st.update(c=torch.exp(-8 * ((x - x.mean(0)) ** 2).sum(1)) + 0.1 * _waves(x, seed, 40), cw=empty(nc),
                      cb=torch.zeros(src.n_boundary_faces, dtype=torch.float64, device=DEV))
        _load(st)
        if case.get("graph"):
            P.set_graph(True)
        # the solver as a running program has it: its hierarchy built, its step captured
        P.step(case["steps"] if case.get("graph") else 1)
        if window:
            st.update(T=_Tape(P, case["steps"], case["every"]), gU=_waves3(x, seed, 50), gp=_waves(x, seed, 60),
                      gphi=_waves(_dev(src.Cf), seed, 61), gpc=np.random.default_rng([seed, 62]).standard_normal(len(setup["wk"])),
                      oU=empty(nc, 3), op=empty(nc), ophi=empty(nf))
    return st


class _Amg:
    def __init__(self, M, A):
        self.M, self.h = M, B.difvm_amg_create(M.h, A)

    def __del__(self):
        B.difvm_amg_destroy(self.h)


class _Tape:
    def __init__(self, P, steps, every):
        self.P, self.h = P, B.difvm_tape_create(P.h, steps, every)

    def __del__(self):
        B.difvm_tape_destroy(self.h)


def _load(st):
    """Starts a run: the state, the flux from the velocity, empty outlets' capacitors."""
    st["P"].set_state(st["U"], st["p"], None)
    for j, row in enumerate(st["setup"]["wk"]):
        st["P"].set_windkessel(j, *row, 0.0)


def run(st):
    case, M = st["case"], st["M"]
    kind = case["kind"]
    if kind == "explicit":
        B.difvm_op_grad(M.h, 1, B.BC_P, st["phi"], st["phib"], st["g"])
        B.difvm_op_laplacian(M.h, B.BC_P, None, st["phi"], st["g"], st["phib"], st["lap"])
        B.difvm_op_interp(M.h, 1, B.BC_P, st["phi"], st["phib"], st["face"])
        B.difvm_op_grad(M.h, 3, B.BC_U, st["U"], st["Ub"], st["gU"])
        scheme = B.SCHEME_UPWIND if case["scheme"] == "upwind" else B.SCHEME_LINEAR
        B.difvm_op_div(M.h, scheme, 3, B.BC_U, st["flux"], st["U"], st["Ub"], st["div"])
        out = dict(g=M.to_user(st["g"], B.KIND_CELL), lap=M.to_user(st["lap"], B.KIND_CELL),
                   face=M.to_user(st["face"], B.KIND_FACE), gU=M.to_user(st["gU"], B.KIND_CELL),
                   div=M.to_user(st["div"], B.KIND_CELL))
        if case["dtype"] == "float64":
            B.difvm_op_deferred_correction(M.h, "sou", 3, st["flux"], st["U"], st["gU"], st["dc"])
            out["dc"] = M.to_user(st["dc"], B.KIND_CELL)
        return out
    if kind == "poisson":
        B.difvm_ldu_assemble_laplace(M.h, B.BC_ALL_FIXED, None, st["phib"], st["A"], st["rbc"])
        B.difvm_op_laplacian(M.h, B.BC_ALL_FIXED, None, st["zero"], st["g"], st["phib"], st["lap"])
        rhs = st["lap"].sub_(st["source"])
        st["x"].zero_()
        if st["amg"] is None:
            B.difvm_solve_pcg(M.h, st["A"], rhs, st["x"], 1e-12, 20000)
        else:
            B.difvm_solve_pcg_amg(st["amg"].h, st["A"], rhs, st["x"], 1e-12, 500)
        return dict(d=M.to_user(st["d"], B.KIND_CELL), rhs=M.to_user(rhs, B.KIND_CELL), x=M.to_user(st["x"], B.KIND_CELL))
    if kind == "momentum":
        B.difvm_ldu_assemble_momentum(M.h, NU, DT, st["flux"], st["U"], st["Ub"], st["A"], st["b"])
        st["x"].copy_(st["U"])
        B.difvm_solve_bicgstab(M.h, st["A"], 3, st["b"], st["x"], 1e-10, 500)
        B.difvm_ldu_spmv(M.h, 3, 1, st["A"], st["x0"], st["y"])
        return dict(d=M.to_user(st["d"], B.KIND_CELL), b=M.to_user(st["b"], B.KIND_CELL),
                    x=M.to_user(st["x"], B.KIND_CELL), y=M.to_user(st["y"], B.KIND_CELL))
    P = st["P"]
    _load(st)
    if kind == "window":
        n = case["steps"]
        B.difvm_piso_forward_record(P.h, st["T"].h, n)
        U, p, phi, pc = P.get_state()
        _, gpc, gwk = B.difvm_piso_adjoint(P.h, st["T"].h, st["gU"], st["gp"], st["gphi"], st["gpc"], 1e-8, st["oU"],
                                           st["op"], st["ophi"], len(st["setup"]["wk"]))
        return dict(U=U, p=p, phi=phi, pc=pc, gU=st["oU"], gp=st["op"], gphi=st["ophi"], gpc=gpc, gwk=gwk)
    P.step(case["steps"])
    out = {}
    if case["scalar"]:
        st["cw"].copy_(st["c"])
        P.transport_scalar(1e-4, B.BC_U, st["cb"], st["cw"])
        out["c"] = st["cw"]
    U, p, phi, pc = P.get_state()
    out.update(U=U, p=p, phi=phi)
    if len(pc):
        out["pc"] = pc
    return out


# ------------------------------------------------------------------------------------------------
# the bytes and operations that a pass cannot do without: the mesh, the inputs and the outputs once
# (a solve: one product's worth of its matrix and vectors; its iterations are the method's choice)
# ------------------------------------------------------------------------------------------------

def _sizes(case):
    if case["mesh"] in ("box", "channel"):
        n, m = case["n"], case["m"]
        nc = 6 * n * n * m
        nfb = 2 * (2 * n * n + 4 * n * m)
        return nc, (4 * nc - nfb) // 2, nfb
    src, _ = _src(case)
    return src.n_cells, src.n_internal_faces, src.n_boundary_faces


def work(case):
    nc, nfi, nfb = _sizes(case)
    kind = case["kind"]
    if kind == "explicit":
        w = 8 if case["dtype"] == "float64" else 4
        # owner, neighbour; S, w, k, delta, flux read and the face value written; boundary faces; cells:
        # phi, V, U read, gradients, Laplacian, divergence written (and the deferred correction)
        b = nfi * (8 + 10 * w) + nfb * (4 + 10 * w) + nc * w * (5 + 16)
        f = nfi * 150 + nc * 30
        if w == 8:
            b += nfi * 6 * w + nc * 3 * w
            f += nfi * 60
        return dict(bytes=b, flops=f)
    if kind == "poisson":
        return dict(bytes=nfi * (8 + 7 * 8) + nfb * 28 + nc * 8 * 8, flops=nfi * 30 + nc * 20)
    if kind == "momentum":
        return dict(bytes=nfi * (8 + 10 * 8) + nfb * 60 + nc * 8 * 14, flops=nfi * 120 + nc * 60)
    steps = case["steps"]
    # per step: the mesh once, the state in and out, the momentum and two pressure systems once each
    b = nfi * (8 + 12 * 8) + nfb * 60 + nc * 8 * 30
    f = nfi * 300 + nc * 200
    return dict(bytes=steps * b * (3 if kind == "window" else 1), flops=steps * f * (3 if kind == "window" else 1))


# ------------------------------------------------------------------------------------------------
# the same in 64 bits with plain torch and numpy, face loops in user order
# ------------------------------------------------------------------------------------------------

class _Plain:
    def __init__(self, src):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).double()  # noqa: E731
        self.nfi, self.nc = src.n_internal_faces, src.n_cells
        self.O = torch.from_numpy(src.owner.astype(np.int64))
        self.N = torch.from_numpy(src.neighbour.astype(np.int64))
        self.Oi, self.Ob = self.O[:self.nfi], self.O[self.nfi:]
        self.S, self.Cf, self.C, self.V, self.w = t(src.Sf), t(src.Cf), t(src.C), t(src.V), t(src.w)
        Si, Sb = self.S[:self.nfi], self.S[self.nfi:]
        d = self.C[self.N] - self.C[self.Oi]
        db = self.Cf[self.nfi:] - self.C[self.Ob]
        self.delta = (Si * Si).sum(1) / (Si * d).sum(1)
        self.k = Si - self.delta[:, None] * d
        self.deltab = (Sb * Sb).sum(1) / (Sb * db).sum(1)
        self.mask = {k: torch.from_numpy(mg.boundary_mask(src, k)) for k in "up"}

    def faces(self, phi, phib, table):
        """Face values of phi [nc, ...] by linear interpolation, boundary by the table."""
        e = (slice(None),) + (None,) * (phi.dim() - 1)
        fi = self.w[e] * phi[self.Oi] + (1 - self.w)[e] * phi[self.N]
        code = self.mask[table][e]
        fb = torch.where(code == 0, phib, torch.where(code == 1, phi[self.Ob], torch.zeros_like(phib)))
        return torch.cat([fi, fb])

    def sum(self, q):
        """Cell sums of a face quantity: + at the owner, - at the neighbour."""
        out = torch.zeros((self.nc,) + q.shape[1:], dtype=torch.float64)
        out.index_add_(0, self.O, q)
        return out.index_add_(0, self.N, -q[:self.nfi])

    def grad(self, phi, phib, table):
        f = self.faces(phi, phib, table)
        q = f[..., None] * (self.S if f.dim() == 1 else self.S[:, None, :])
        s = self.sum(q)
        return s / (self.V[:, None] if s.dim() == 2 else self.V[:, None, None])

    def correction(self, g):
        """k . interp(g) per internal face, g [nc, 3] or [nc, c, 3]."""
        e = (slice(None),) + (None,) * (g.dim() - 1)
        gf = self.w[e] * g[self.Oi] + (1 - self.w)[e] * g[self.N]
        k = self.k if g.dim() == 2 else self.k[:, None, :]
        return (k * gf).sum(-1)

    def matrix(self, d, up, low):
        """CSR matrix of the LDU coefficients (upper: row owner)."""
        i = torch.cat([torch.arange(self.nc), self.Oi, self.N])
        j = torch.cat([torch.arange(self.nc), self.N, self.Oi])
        return torch.sparse_coo_tensor(torch.stack([i, j]), torch.cat([d, up, low]), (self.nc, self.nc)).to_sparse_csr()


def _cg(A, d, b, x, tol=3e-15, maxit=4000):
    r = b - A @ x
    z = r / d
    p, rz, bn = z.clone(), r @ z, b.norm()
    for _ in range(maxit):
        if r.norm() <= tol * bn:
            break
        q = A @ p
        a = rz / (p @ q)
        x = x + a * p
        r = r - a * q
        z = r / d
        rz, old = r @ z, rz
        p = z + (rz / old) * p
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "window"):
        return None  # hundreds of solves: no plain counterpart within seconds
    src, setup = _src(case)
    G = _Plain(src)
    nfi = G.nfi
    if kind == "explicit":
        phi, phib, U, Ub, flux = (t.double() for t in _explicit_inputs(case, seed, G.C, G.Cf, G.S, nfi))
        g, gU = G.grad(phi, phib, "p"), G.grad(U, Ub, "u")
        lf = G.delta * (phi[G.N] - phi[G.Oi]) + G.correction(g)
        lb = torch.where(G.mask["p"] == 0, G.deltab * (phib - phi[G.Ob]), torch.zeros_like(phib))
        Uf = G.faces(U, Ub, "u")
        pos = (flux[:nfi] >= 0)
        up = torch.where(pos, G.Oi, G.N)
        if case["scheme"] == "upwind":
            Uf[:nfi] = U[up]
        out = dict(g=g, lap=G.sum(torch.cat([lf, lb])), face=G.faces(phi, phib, "p"), gU=gU, div=G.sum(flux[:, None] * Uf))
        if case["dtype"] == "float64":
            q = torch.zeros_like(Uf)
            q[:nfi] = -flux[:nfi, None] * (gU[up] * (G.Cf[:nfi] - G.C[up])[:, None, :]).sum(-1)
            out["dc"] = G.sum(q)
        return out
    if kind == "poisson":
        amp = 1.0 + 0.5 * np.random.default_rng(seed).random()
        phib = torch.from_numpy(amp * mg.poisson_mms_solution(src.Cf[nfi:]))
        g = torch.from_numpy(amp * mg.poisson_mms_gradient(src.C))
        source = torch.from_numpy(amp * src.V * mg.poisson_mms_source(src.C))
        d = torch.zeros(G.nc, dtype=torch.float64)
        d.index_add_(0, G.O, torch.cat([G.delta, G.deltab])).index_add_(0, G.N, G.delta)
        rhs = G.sum(torch.cat([G.correction(g), G.deltab * phib])) - source
        if G.nc > 200000:
            return dict(d=d, rhs=rhs, x=None)  # the solve takes too long here
        x = _cg(G.matrix(d, -G.delta, -G.delta), d, rhs, torch.zeros_like(rhs))
        return dict(d=d, rhs=rhs, x=x)
    U, flux, x0 = _momentum_inputs(seed, G.C, G.Cf, G.S)
    Ub = torch.from_numpy(setup["Ub"])
    F, Fb = flux[:nfi], flux[nfi:]
    fixed, free = G.mask["u"] == 0, G.mask["u"] == 1
    up, low = F.clamp(max=0) - NU * G.delta, -F.clamp(min=0) - NU * G.delta
    d = G.V / DT
    d.index_add_(0, G.Oi, F.clamp(min=0) + NU * G.delta).index_add_(0, G.N, -F.clamp(max=0) + NU * G.delta)
    d.index_add_(0, G.Ob, torch.where(fixed, NU * G.deltab, torch.where(free, Fb, torch.zeros_like(Fb))))
    b = (G.V / DT)[:, None] * U
    b += G.sum(torch.cat([NU * G.correction(G.grad(U, Ub, "u")),
                          torch.where(fixed[:, None], (NU * G.deltab - Fb)[:, None] * Ub, torch.zeros_like(Ub))]))
    A = G.matrix(d, up, low)
    x = U.clone()
    for _ in range(400):  # the time term dominates: Jacobi steps converge quickly
        r = b - A @ x
        if r.norm() <= 1e-15 * b.norm():
            break
        x += r / d[:, None]
    At = G.matrix(d, low, up)
    return dict(d=d, b=b, x=x, y=At @ x0)
