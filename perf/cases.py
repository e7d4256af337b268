"""The work that a user of the planning library has it do, as measured cases.

A patient is a voxel phantom shaped like the head-and-neck workloads of the
framework's benchmark: an ellipsoidal body at 2.5 mm, two targets and four
organs at risk, three coplanar beams with a 5 mm lateral spot grid and nine
energy layers at a position, 3 mm shifts and 3.5 % range errors as scenarios.  `n` spots, the
body's size and the number of scenarios come from the case, everything else
(where targets and organs lie, spot jitter, plans, weights) from the seed.
"""
import math

import numpy as np
import torch

import paper_2304_14568_amd as A

SPACING, SIGMA, H_MM, LAYERS, BEAMS = 5.0, 2.5, 2.5, 9, (0.0, 120.0, 240.0)
#: nonzeros of a spot's column per voxel of the body's longest semi-axis, roughly (the exact number depends on the seed)
NNZ_PER_SPOT = 47.0
FEATURES = 15  # 8 geometric and 7 dose features of the warm-start network


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # a single-field check plan: 100 spots, where launches and host waits are all there is
        dict(name="solve_tiny", kind="solve", n=100, body=13, scen=3),
        # the benchmark's patient, solved to the paper's stopping rule with the default options
        dict(name="solve_hn13", kind="solve", n=2981, body=50, scen=13),
        # the largest patient of the paper's Table 1, iterated in chunks with a checkpoint after each
        dict(name="iterate_large", kind="iterate", n=5762, body=50, scen=13, k=20),
        # several uneven patients in one context, as a planning queue runs them
        dict(name="iterate_batch", kind="batch", n=1883, body=40, scen=8, patients=6, k=30),
        # more spots than the cached inverses take (n > 8128): the library chooses the sparse CG form by itself
        dict(name="solve_cg_huge", kind="solve", n=8501, body=50, scen=3),
        # CG asked for with bf16 values, the reduced-precision option of the precision study
        dict(name="solve_cg_bf16", kind="solve", n=1493, body=40, scen=13, xupdate="cg", precision="bf16"),
        # the comparison method on the benchmark's patient: a fixed budget of projected-gradient steps
        dict(name="pgd_hn13", kind="pgd", n=2981, body=50, scen=13, k=150),
        # a new patient: set-up from host arrays, then the first iterations
        dict(name="setup_mid", kind="setup", n=1700, body=42, scen=13, k=5),
        # dose-volume evaluation of a finished plan over every scenario
        dict(name="evaluate_hn13", kind="evaluate", n=2981, body=50, scen=13, nbins=2048),
        # objective and gradient of a plan, on the paper's smallest patient
        dict(name="gradient_small", kind="gradient", n=707, body=30, scen=13),
        # learned warm start of a patient: features, network, new penalty and duals
        dict(name="warm_start_mid", kind="warm", n=2003, body=45, scen=13, hidden=128),
        # one pass of the network's training over eight patients
        dict(name="train_mlp", kind="train", rows=2981, hidden=128, steps=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "iterate", "batch", "solve_cg", "pgd", "setup", "evaluate", "gradient", "warm",
                       "train"])
    if kind == "train":
        return dict(kind="train", rows=_log(rng, 200, 6000), hidden=rng.choice([32, 64, 100, 128, 160]),
                    steps=rng.randint(2, 8))
    n = _log(rng, 120, 3400)
    c = dict(kind=kind, n=n, body=min(50, max(16, int(round(50 * (n / 3000.0) ** (1 / 3.0))) + rng.randint(-4, 4))),
             scen=rng.choice([1, 3, 5, 9, 13, 21]))
    if n > 2000:
        c["scen"] = min(c["scen"], 13)
    if kind == "solve_cg":
        c.update(kind="solve", xupdate="cg", precision=rng.choice(["fp32", "bf16", "fp16"]))
    elif kind in ("iterate", "setup"):
        c["k"] = rng.randint(5, 40)
    elif kind == "batch":
        c.update(n=min(n, 1700), scen=min(c["scen"], 9), patients=rng.randint(2, 6), k=rng.randint(5, 40))
    elif kind == "pgd":
        c["k"] = rng.randint(20, 150)
    elif kind == "evaluate":
        c["nbins"] = rng.choice([256, 1000, 2048])
    elif kind == "warm":
        c["hidden"] = 128
    return c


# ---------------------------------------------------------------------------
# patients
# ---------------------------------------------------------------------------

class _Csr:
    def __init__(self, row_ptr, col, val):
        self.row_ptr, self.col, self.val = row_ptr, col, val


class _Patient:
    """The arrays `Solver` takes; `dev` keeps the matrices on the GPU for exact()."""

    def __init__(self, **kw):
        self.__dict__.update(kw)


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _shifts(scen, gen):
    s, r = 3.0, 0.035
    base = [(0, 0, 0, 0), (s, 0, 0, 0), (-s, 0, 0, 0), (0, s, 0, 0), (0, -s, 0, 0), (0, 0, s, 0), (0, 0, -s, 0),
            (0, 0, 0, -r), (0, 0, 0, r), (s, 0, 0, r), (-s, 0, 0, -r), (0, s, 0, r), (0, -s, 0, -r)]
    while len(base) < scen:
        u = gen.uniform(-1.0, 1.0, 4)
        base.append((s * u[0], s * u[1], s * u[2], r * u[3]))
    return base[:scen]


def _spots(n, layers):
    """(beam, u, v, layer) of n spots: discs of lateral positions on the 5 mm
    grid, the positions of each beam in (u, v) order with their layers together."""
    per = [n // 3 + (1 if b < n % 3 else 0) for b in range(3)]
    out = []
    for b, nb in enumerate(per):
        pos = -(-nb // layers)
        g = int(math.sqrt(pos)) + 2
        cand = sorted(((u * u + v * v, u, v) for u in range(-g, g + 1) for v in range(-g, g + 1)))[:pos]
        cand = sorted((u, v) for _, u, v in cand)
        lst = [(b, u, v, k) for u, v in cand for k in range(layers)][:nb]
        out += lst
    return np.asarray(out, dtype=np.float64).reshape(-1, 4)


def _patient(n, body, scen, seed):
    dev, gen = _device(), np.random.default_rng([seed, n, body, scen])
    semi = np.array([1.0, 0.8, 0.6]) * body * H_MM
    ax = [torch.arange(-math.ceil(s / H_MM), math.ceil(s / H_MM) + 1, device=dev, dtype=torch.float64) * H_MM for s in semi]
    Z, Y, X = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    pts = torch.stack([X.reshape(-1), Y.reshape(-1), Z.reshape(-1)], 1)
    semi_t = torch.tensor(semi, device=dev)
    pts = pts[((pts / semi_t) ** 2).sum(1) <= 1.0]
    m = pts.shape[0]
    layers = LAYERS if n >= 200 else 4
    sp = _spots(n, layers)
    radius = SPACING * (math.sqrt(np.max(sp[:, 1] ** 2 + sp[:, 2] ** 2)) + 0.7)
    iso = gen.uniform(-0.15, 0.15, 3) * semi

    # structures: 0 normal, 1-2 targets, 3-6 organs at risk
    iso_t = torch.tensor(iso, device=dev)
    sid = torch.zeros(m, dtype=torch.uint8, device=dev)
    presc = torch.zeros(m, dtype=torch.float64, device=dev)
    for k in range(4):
        d = gen.normal(size=3)
        c = iso + d / np.linalg.norm(d) * radius * gen.uniform(0.9, 1.5)
        e = (pts - torch.tensor(c, device=dev)) / torch.tensor(gen.uniform(0.25, 0.5, 3) * radius, device=dev)
        sid[(e * e).sum(1) <= 1.0] = 3 + k
    for k, p in ((1, 0.85), (0, 1.0)):
        c = iso + gen.uniform(-0.3, 0.3, 3) * radius
        e = (pts - torch.tensor(c, device=dev)) / torch.tensor(gen.uniform(0.5, 0.85, 3) * radius, device=dev)
        inside = (e * e).sum(1) <= 1.0
        sid[inside] = 1 + k
        presc[inside] = p

    key = [tuple(r) for r in sp[:, :3]]
    first = {}
    for j, k in enumerate(key):
        first.setdefault(k, j)
    pos = np.array([[*k, j] for k, j in sorted(first.items(), key=lambda kv: kv[1])])  # beam, u, v, first spot
    nl = np.diff(np.append(pos[:, 3], n)).astype(np.int64)
    uv = pos[:, 1:3] * SPACING + gen.uniform(-0.5, 0.5, (len(pos), 2))
    th = np.deg2rad(np.asarray(BEAMS))[pos[:, 0].astype(int)]
    D = np.stack([np.cos(th), np.sin(th), 0 * th], 1)
    E1 = np.stack([-np.sin(th), np.cos(th), 0 * th], 1)
    centre = iso + uv[:, :1] * E1 + uv[:, 1:] * np.array([0.0, 0.0, 1.0])

    def enter(q):  # depth of the body's surface along each axis, from its centre point
        qs, ds = q / semi, D / semi
        a, b, c = (ds * ds).sum(1), 2 * (qs * ds).sum(1), (qs * qs).sum(1) - 1.0
        return (-b - np.sqrt(np.maximum(b * b - 4 * a * c, 0.0))) / (2 * a)

    depth0 = -enter(centre)
    off = (np.arange(layers) - (layers - 1) / 2) / max(1, layers - 1) * 2.0 * radius
    R = np.maximum(depth0[:, None] + off[None, :], 8.0)  # range of layer k at each position

    t = lambda a: torch.tensor(a, device=dev)  # noqa: E731
    D_t, nl_t, first_t, R_t = t(D), t(nl), t(pos[:, 3].astype(np.int64)), t(R)
    rmax2 = 2.0 * SIGMA * SIGMA * math.log(1e4)
    mats = []
    for sx, sy, sz, rr in _shifts(scen, gen):
        c_np = centre + np.array([sx, sy, sz])
        c_t, tin = t(c_np), t(enter(c_np))
        rows, posi = [], []
        for lo in range(0, m, 65536):
            q = pts[lo:lo + 65536]
            along = q @ D_t.T - (c_t * D_t).sum(1)
            r2 = (q * q).sum(1, keepdim=True) - 2 * (q @ c_t.T) + (c_t * c_t).sum(1) - along * along
            keep = (r2 <= rmax2) & (along >= tin)
            i, p = torch.nonzero(keep, as_tuple=True)
            rows.append(i + lo)
            posi.append(torch.stack([p.double(), along[i, p] - tin[p], r2[i, p]], 1))
        i, pdr = torch.cat(rows), torch.cat(posi)
        p, d, r2 = pdr[:, 0].long(), pdr[:, 1:2], pdr[:, 2:3]
        Rk = (R_t * (1.0 + rr))[p]
        x = torch.where(d <= Rk, 0.3 + 0.2 * d / Rk + 0.5 * torch.exp(-0.5 * ((Rk - d) / (0.04 * Rk + 1.0)) ** 2),
                        torch.exp(-0.5 * ((d - Rk) / (0.012 * Rk + 0.8)) ** 2))
        x = (x * torch.exp(-0.5 * r2.clamp_min(0) / SIGMA ** 2)).float()
        keep = (x >= 1e-4) & (torch.arange(layers, device=dev)[None, :] < nl_t[p][:, None])
        a, k = torch.nonzero(keep, as_tuple=True)
        rp = torch.zeros(m + 1, dtype=torch.int64, device=dev)
        rp[1:] = torch.cumsum(torch.bincount(i[a], minlength=m), 0)
        mats.append(_Csr(rp, (first_t[p[a]] + k).int(), x[a, k].contiguous()))
    return _Patient(m=m, n=n, A=mats, prob=np.ones(scen), struct_id=sid.cpu().numpy(),
                    struct_weight=np.array([0.1, 1.0, 1.0, 0.5, 0.5, 0.5, 0.5]), presc=presc.cpu().numpy(),
                    lb=np.zeros(n), ub=np.full(n, 10.0), plan=gen.uniform(0.0, 0.15, n) * (gen.random(n) < 0.7))


def _sizes(case):
    """(n, body, seed offset) of every patient of a case."""
    if case["kind"] != "batch":
        return [(case["n"], case["body"], 0)]
    f = [1.0, 0.55, 1.6, 0.8, 0.37, 1.25]
    return [(max(60, int(case["n"] * f[k])), max(14, int(case["body"] * f[k] ** (1 / 3.0))), 101 * k)
            for k in range(case["patients"])]


def _patients(case, seed):
    return [_patient(n, b, case["scen"], seed + o) for n, b, o in _sizes(case)]


def _host(P):
    """The same patient with its matrices in host memory."""
    q = _Patient(**P.__dict__)
    q.A = [_Csr(a.row_ptr.cpu().numpy(), a.col.cpu().numpy(), a.val.cpu().numpy()) for a in P.A]
    return q


def _options(case):
    return {k: case[k] for k in ("xupdate", "precision") if k in case}


def _train_data(case, seed):
    """Feature rows, targets and penalties of the case's patients (uneven numbers of spots)."""
    g = np.random.default_rng([seed, case["rows"], case["hidden"]])
    out = []
    for s in range(case["steps"]):
        rows = max(8, int(case["rows"] * (0.7 + 0.6 * ((5 * s + 2) % 8) / 8.0)))
        X = g.normal(size=(rows, FEATURES)).astype(np.float32)
        y = np.abs(0.5 * X[:, 0] + 0.3 * X[:, 9] * X[:, 3] + 0.2 * g.normal(size=rows)).astype(np.float32)
        out.append((X, y, float(g.choice([0.0, math.log(0.5)]))))
    return out


def _theta(hidden, seed):
    """He-uniform weights of the network."""
    g = np.random.default_rng([seed, hidden, 7])
    u = lambda lim, *s: g.uniform(-lim, lim, s).reshape(-1)  # noqa: E731
    H, F = hidden, FEATURES
    return np.concatenate([u(math.sqrt(6 / F), H, F), np.zeros(H), u(math.sqrt(6 / H), H, H), np.zeros(H),
                           u(math.sqrt(3 / H), H), np.zeros(1), 0.1 * u(math.sqrt(3 / H), H), np.zeros(1)]).astype(np.float32)


def _classes(P):
    return np.where(P.struct_id == 0, 0, np.where(P.struct_id <= 2, 1, 2)).astype(np.uint8)


def _geometry(n, seed):
    return np.random.default_rng([seed, n, 3]).normal(size=(n, 8)).astype(np.float32)


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

LR, LAM = 2e-3, 0.05
ALPHA_STEPS = 30


def prepare(case, seed):
    if case["kind"] == "train":
        net = A.Mlp(FEATURES, case["hidden"], seed=1)
        return dict(case=case, net=net, theta=_theta(case["hidden"], seed), data=_train_data(case, seed))
    Ps = _patients(case, seed)
    if case["kind"] == "setup":
        return dict(case=case, P=_host(Ps[0]))
    S = A.Solver(Ps, **_options(case))
    st = dict(case=case, S=S, plan=Ps[0].plan)
    if case["kind"] == "evaluate":
        st["group"] = Ps[0].struct_id
    if case["kind"] == "warm":
        st.update(cls=_classes(Ps[0]), geom=_geometry(case["n"], seed), rho=[S.rho() * 0.8, S.rho() * 1.25], turn=0,
                  net=A.Mlp(FEATURES, case["hidden"], seed=1), ub=Ps[0].ub)
        st["net"].set_params(_theta(case["hidden"], seed))
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "train":
        net = st["net"]
        net.set_params(st["theta"])
        losses = []
        for X, y, lr_t in st["data"]:
            L, grad = net.loss_grad(X, y, lr_t, LAM)
            net.adam_step(lr=LR)
            losses.append(L)
        return dict(losses=np.array(losses), grad=grad, params=net.get_params())
    if kind == "setup":
        with A.Solver(st["P"]) as S:
            info = S.iterate(case["k"])
            return dict(z=S.z(), obj=info[0]["obj"], rho=S.rho())
    S = st["S"]
    if kind == "solve":
        S.reset()
        z, info, _ = S.solve()
        return dict(z=z[0], obj=info[0]["obj"])
    if kind == "iterate":
        S.reset()
        info = S.iterate(case["k"])
        s = S.get_state()
        return dict(z=s["z"], y=s["y"], d=s["d"], obj=info[0]["obj"])
    if kind == "batch":
        S.reset()
        info = S.iterate(case["k"])
        return dict(z=[S.z(p) for p in range(S.num_patients)], obj=[i["obj"] for i in info])
    if kind == "pgd":
        x, info, _ = S.pgd(0, obj_rel_tol=0.0, max_iter=case["k"])
        return dict(x=x, obj=info["obj"])
    if kind == "evaluate":
        counts, sums, maxes, _ = S.dose_stats(st["plan"], st["group"], 7, case["nbins"], 2.0)
        return dict(counts=counts, sums=sums, maxes=maxes)
    if kind == "gradient":
        g, f = S.gradient(st["plan"])
        return dict(g=g, f=f)
    # warm: features, network, then a start with its plan, its duals and a new penalty
    f = S.spot_features(st["cls"])
    y, lr = st["net"].forward(np.concatenate([st["geom"], f], axis=1), precision="bf16")
    S.warm_start(0, np.clip(0.1 * y.astype(np.float64), 0.0, st["ub"]), st["rho"][0], dual_init=True)
    S.warm_start(0, np.clip(0.1 * y.astype(np.float64), 0.0, st["ub"]), st["rho"][1], dual_init=True)
    s = S.get_state()
    info = S.iterate(1)
    return dict(features=f, y=y, log_rho=lr, z=s["z"], dual=s["y"], obj=info[0]["obj"], z1=S.z())


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    if case["kind"] == "train":
        H, F = case["hidden"], FEATURES
        rows = sum(len(y) for _, y, _ in _train_data(case, 0))
        par = H * F + 2 * H + H * H + 2 * H + 2
        return dict(bytes=rows * (F + 1) * 4.0 + case["steps"] * par * 4.0 * 8, flops=rows * 6.0 * (H * F + H * H + 2 * H))
    N, total, flops = case["scen"], 0.0, 0.0
    for n, body, _ in _sizes(case):
        nnz = NNZ_PER_SPOT * body * n * N
        dense = case.get("xupdate") != "cg" and n <= 8128
        # per ADMM iteration: the packed inverses (CG: eight operator passes and one gradient pass) and the vectors
        values = 2.0 if case.get("precision") in ("bf16", "fp16") else 4.0
        it = (2.0 * n * n * (N + 1.5) + 28.0 * N * n) if dense else nnz * (8 * (values + 2) + 6)
        fl = 2.0 * n * n * (N + 1) if dense else 36.0 * nnz
        kind = case["kind"]
        if kind == "solve":
            total, flops = total + 230 * it, flops + 230 * fl
        elif kind in ("iterate", "batch"):
            total, flops = total + case["k"] * it + 24.0 * N * n, flops + case["k"] * fl
        elif kind == "pgd":
            total, flops = total + (case["k"] + 1 + ALPHA_STEPS) * 4.0 * n * n, flops + case["k"] * 16.0 * n * n
        elif kind in ("setup", "warm"):
            total += nnz * 8 + 2.0 * n * n * N
            flops += 2.0 * nnz * 30 + 1.0 * n ** 3 * N
            if kind == "setup":
                total, flops = total + case["k"] * it, flops + case["k"] * fl
            else:
                total += nnz * 6 * 2
        elif kind == "evaluate":
            total += nnz * 6 + 4.0 * N * 7 * case["nbins"]
            flops += 2.0 * nnz
        elif kind == "gradient":
            total += nnz * 6
            flops += 4.0 * nnz
    return dict(bytes=total, flops=flops)


def tolerance(case):
    kind = case["kind"]
    if kind == "solve":
        # a run may end an iteration sooner or later: the stopping rule leaves the intensities 1e-4 from the minimiser
        return {"rel": 5e-4, "max": 2e-2}
    if kind == "iterate":
        # fp32 inverses of a system with condition 1e4: 1e-6 in z and the duals, 2.5e-4 in the small d = x - z
        return {"rel": 1e-3, "max": 4e-2}
    if kind in ("batch", "setup"):
        return {"rel": 1e-5, "max": 1e-3}  # 2.4e-6 seen in z against 64 bits
    if kind == "pgd":
        return {"rel": 4e-7, "max": 2e-5}  # 9.4e-8 seen: the order of the power iteration's sums moves the first step
    if kind == "evaluate":
        # fp32 doses of fp64 row sums (3e-8 seen); a dose on a bin's edge may change its bin
        return {"rel": 2e-7, "max": 1e-6, "differ": 1e-3}
    if kind == "gradient":
        return {"rel": 5e-7, "max": 1e-5}  # 8e-8 seen: fp32 column sums of each tile, added in fp64
    if kind == "warm":
        # bf16 hidden layers: a sum in another order moves an activation by one bf16 step (1/256)
        return {"rel": 2e-3, "max": 5e-2}
    # training: gradients 3e-7 and weights 8e-8 from 64 bits, but Adam makes a whole step of a near-zero gradient's sign
    return {"rel": 5e-5, "max": 5e-2}


# ---------------------------------------------------------------------------
# the same in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _sparse(a, m, n):
    return torch.sparse_csr_tensor(a.row_ptr, a.col.long(), a.val.double(), size=(m, n))


def _weights(P):
    dev = P.A[0].val.device
    w = torch.tensor(P.struct_weight, device=dev)[torch.tensor(P.struct_id, device=dev).long()]
    return w, torch.tensor(P.presc, device=dev)


def _gram(P):
    """(G_s, b_s, const) of every scenario, dense, row blocks at a time."""
    w, p = _weights(P)
    out, const = [], 0.0
    for a in P.A:
        G = torch.zeros(P.n, P.n, dtype=torch.float64, device=w.device)
        b = torch.zeros(P.n, dtype=torch.float64, device=w.device)
        len_ = a.row_ptr[1:] - a.row_ptr[:-1]
        ids = torch.nonzero(len_ > 0)[:, 0]
        step = max(1, min(32768, int(4e8 // P.n)))
        for lo in range(0, len(ids), step):
            r = ids[lo:lo + step]
            L = len_[r]
            local = torch.repeat_interleave(torch.arange(len(r), device=w.device), L)
            start = torch.cumsum(L, 0) - L
            e = a.row_ptr[r][local] + torch.arange(int(L.sum()), device=w.device) - start[local]
            B = torch.zeros(len(r), P.n, dtype=torch.float64, device=w.device)
            B[local, a.col[e].long()] = a.val[e].double()
            WB = B * w[r][:, None]
            G += B.t().contiguous() @ WB
            b += WB.t() @ p[r]
        const += float((w * p * p).sum())
        out.append((G, b))
    return out, const


def _admm(P, rho=None, k=None, z=None, dual_at_z=False, tight=False):
    """ADMM with the Barzilai-Borwein dual step in 64 bits: k iterations, or on to the minimiser."""
    gs, const = _gram(P)
    dev = gs[0][0].device
    N, n = len(gs), P.n
    if rho is None:
        rho = 2.0 * float(torch.stack([G.diagonal().mean() for G, _ in gs]).mean())
    S = torch.stack([G for G, _ in gs]).sum(0)
    g0 = 2.0 * torch.stack([b for _, b in gs]).sum(0)
    lb, ub = torch.tensor(P.lb, device=dev), torch.tensor(P.ub, device=dev)
    f = lambda v: float(v @ (S @ v) - g0 @ v + const)  # noqa: E731
    z = torch.zeros(n, dtype=torch.float64, device=dev) if z is None else torch.minimum(torch.maximum(z, lb), ub)
    y = torch.stack([-2.0 * (G @ z - b) for G, b in gs]) if dual_at_z else torch.zeros(N, n, dtype=torch.float64, device=dev)
    z_start, y_start = z.clone(), y.clone()
    inv = torch.stack([torch.linalg.inv(G + 0.5 * rho * torch.eye(n, dtype=torch.float64, device=dev)) for G, _ in gs])
    bs = torch.stack([b for _, b in gs])
    tau, dp = rho, torch.zeros(N, n, dtype=torch.float64, device=dev)
    for it in range(k if k is not None else 4000):
        c = bs + 0.5 * rho * z - 0.5 * y
        x = torch.bmm(inv, c[:, :, None])[:, :, 0]
        zn = torch.minimum(torch.maximum((x + y / rho).mean(0), lb), ub)
        d = x - zn
        dd = d - dp
        dd2 = float((dd * dd).sum())
        tau_n = rho
        if it >= 1 and dd2 > 0:
            beta = -tau * float((dd * dp).sum()) / dd2
            tau_n = beta if math.isfinite(beta) and beta > 0 else rho
        tau = tau_n
        y = y + tau * d
        move = float((zn - z).norm()) / max(1e-30, float(zn.norm()))
        z, dp = zn, d
        if tight and it > 20 and move < 1e-10 and float(d.norm()) < 1e-9 * float(x.norm()):
            break
    return dict(z=z, y=y, d=dp, obj=f(z), rho=rho, z_start=z_start, y_start=y_start)


def _np(t):
    return t.double().cpu().numpy()


def _mlp64(th, X, hidden):
    H, F = hidden, FEATURES
    o = np.cumsum([0, H * F, H, H * H, H, H, 1, H, 1])
    W1, b1, W2, b2, w3, b3, wr, br = (th[o[i]:o[i + 1]] for i in range(8))
    h1 = torch.relu(X @ W1.reshape(H, F).t() + b1)
    h2 = torch.relu(h1 @ W2.reshape(H, H).t() + b2)
    return torch.nn.functional.softplus(h2 @ w3 + b3), (h2.mean(0) @ wr + br)[0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        th = torch.tensor(_theta(case["hidden"], seed).astype(np.float64))
        m, v, losses = torch.zeros_like(th), torch.zeros_like(th), []
        for t, (X, y, lr_t) in enumerate(_train_data(case, seed), 1):
            q = th.clone().requires_grad_(True)
            out, lr = _mlp64(q, torch.tensor(X.astype(np.float64)), case["hidden"])
            L = ((out - torch.tensor(y.astype(np.float64))) ** 2).mean() + LAM * (lr - lr_t) ** 2
            (g,) = torch.autograd.grad(L, q)
            losses.append(float(L.detach()))
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            th = th - LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
        return dict(losses=np.array(losses), grad=g.numpy(), params=th.numpy())
    if case["n"] > 4000:
        return None
    Ps = _patients(case, seed)
    P = Ps[0]
    if kind == "solve":
        r = _admm(P, tight=True)
        return dict(z=_np(r["z"]), obj=r["obj"])
    if kind == "iterate":
        r = _admm(P, k=case["k"])
        return dict(z=_np(r["z"]), y=_np(r["y"]).reshape(-1), d=_np(r["d"]).reshape(-1), obj=r["obj"])
    if kind == "batch":
        rs = [_admm(q, k=case["k"]) for q in Ps]
        return dict(z=[_np(r["z"]) for r in rs], obj=[r["obj"] for r in rs])
    if kind == "setup":
        r = _admm(P, k=case["k"])
        return dict(z=_np(r["z"]), obj=r["obj"], rho=r["rho"])
    w, p = _weights(P)
    dev = w.device
    if kind == "pgd":
        gs, const = _gram(P)
        S, g0 = torch.stack([G for G, _ in gs]).sum(0), 2.0 * torch.stack([b for _, b in gs]).sum(0)
        lb, ub = torch.tensor(P.lb, device=dev), torch.tensor(P.ub, device=dev)
        u = torch.full((P.n,), 1.0 / math.sqrt(P.n), dtype=torch.float64, device=dev)
        for _ in range(ALPHA_STEPS):
            u = 2.0 * (S @ u)
            lam = float(u.norm())
            u = u / lam
        alpha, x = 10.0 / lam, torch.zeros(P.n, dtype=torch.float64, device=dev)
        f = lambda q: float(q @ (S @ q) - g0 @ q + const)  # noqa: E731
        fx = f(x)
        for _ in range(case["k"]):
            g, t = 2.0 * (S @ x) - g0, alpha
            for _ in range(60):
                xt = torch.minimum(torch.maximum(x - t * g, lb), ub)
                ft = f(xt)
                if ft <= fx + 1e-4 * float(g @ (xt - x)):
                    break
                t *= 0.5
            x, fx = xt, ft
        return dict(x=_np(x), obj=fx)
    if kind == "evaluate":
        x = torch.tensor(P.plan.astype(np.float32), device=dev).double()
        grp = torch.tensor(P.struct_id, device=dev).long()
        sums, maxes = [], []
        for a in P.A:
            d = _sparse(a, P.m, P.n) @ x
            sums.append(torch.zeros(7, dtype=torch.float64, device=dev).index_add_(0, grp, d))
            maxes.append(torch.stack([d[grp == g].max() if bool((grp == g).any()) else d.new_tensor(-math.inf)
                                      for g in range(7)]))
        return dict(counts=None, sums=_np(torch.stack(sums)), maxes=_np(torch.stack(maxes)))
    if kind == "gradient":
        x = torch.tensor(P.plan.astype(np.float32), device=dev).double()
        g, f = torch.zeros_like(x), 0.0
        for a in P.A:
            M = _sparse(a, P.m, P.n)
            r = M @ x - p
            f += float((w * r * r).sum())
            g.index_add_(0, a.col.long(), 2.0 * a.val.double() * torch.repeat_interleave(w * r, a.row_ptr.diff()))
        return dict(g=_np(g), f=f)
    # warm: the features (the network's bf16 layers and what follows from them are not 64-bit values)
    cls = torch.tensor(_classes(P), device=dev)
    T, O, M, bs, gd = [], [], [], 0.0, 0.0
    for a in P.A:
        per = lambda u: torch.zeros(P.n, dtype=torch.float64, device=dev).index_add_(  # noqa: E731
            0, a.col.long(), u * torch.repeat_interleave(q, a.row_ptr.diff()))
        v = a.val.double()
        q = (cls == 1).double()
        T.append(per(v))
        q = (cls == 2).double()
        O.append(per(v))
        q = torch.ones(P.m, dtype=torch.float64, device=dev)
        M.append(per(v))
        q = w * p
        bs = bs + per(v)
        q = w
        gd = gd + per(v * v)
    T, O, M = torch.stack(T), torch.stack(O), torch.stack(M)
    ft, fo = torch.where(M > 0, T / M, 0 * M), torch.where(M > 0, O / M, 0 * M)
    feat = torch.stack([ft.mean(0), ft.min(0)[0], ft.max(0)[0], fo.mean(0), fo.max(0)[0], torch.log1p(M.mean(0)),
                        torch.where(gd > 0, bs / gd, 0 * gd)], 1)
    return dict(features=_np(feat), y=None, log_rho=None, z=None, dual=None, obj=None, z1=None)
