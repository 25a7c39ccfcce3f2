"""The work users of the library have it do, as measured cases.

A case is one call sequence through the public binding (`gap.Handle`,
`gap.fit_static`, `gap.cur_select`) on inputs that are resident on the GPU:

  fit      build_knm + solve of one fit on energies: from the 200-configuration
           workload up to the 1e5-configuration one, with the sizes of the
           hyperparameter sweep between them
  forces   build_knm_obs + solve: energies, forces and virials
  predict  energies of 1 .. 4096 configurations against a resident model, the
           serving loop's requests
  cur      sparse-point selection from the descriptor rows of a training set

The low-precision K_NM forms (BF16, FP16) are left out: an FP64 K_NM is built
beside theirs, and the FP32 form is faster and more accurate, so nobody picks
them in earnest.  The derivative inputs have the structure of the recipe in
synth.make_deriv_inputs (12 neighbours per atom, a gradient row per neighbour
and coordinate, six virial components per configuration), drawn on the GPU.
"""
import math

import torch

from paper_2207_03803_amd import gap

DEV = "cuda"
JITTER = 1e-8
NEIGH = 12         # neighbours per atom of the derivative inputs
SIGMA_F = 0.05     # standard deviation of a force component
SIGMA_V = 0.05     # of a virial component, per atom
N_TRUE = 64        # sparse points that carry the weights behind the targets


def listed():
    fit = dict(kind="fit", atoms_lo=8, atoms_hi=64, sigma_per_atom=1e-3, precision="fp64", int8=False, entry="wait")
    pred = dict(kind="predict", atoms_lo=8, atoms_hi=64)
    return [
        # one configuration against a served model: the shortest request there is
        dict(pred, name="predict_one", n_configs=1, d=400, M=4000, zeta=4),
        # a batch of a few hundred (an odd number), mid-sized model
        dict(pred, name="predict_batch", n_configs=333, d=256, M=2250, zeta=3),
        # the largest batch of the serving loop
        dict(pred, name="predict_large", n_configs=4096, d=400, M=4000, zeta=4),
        # the tiny workload: 200 configurations, launches and latency
        dict(fit, name="fit_tiny", n_configs=200, d=64, M=256, zeta=2),
        # the small corner of the sweep, enqueued without waiting, FP32 factor
        dict(fit, name="fit_small_mixed", n_configs=2003, d=128, M=500, zeta=2, precision="fp32", entry="queue"),
        # the allocation-free entry point near its size limit
        dict(fit, name="fit_static", n_configs=6007, d=256, M=1111, zeta=3, entry="static"),
        # the middle of the sweep with its precision
        dict(fit, name="fit_sweep_mixed", n_configs=16001, d=256, M=2250, zeta=3, precision="fp32", entry="queue"),
        # the large corner of the sweep, in FP64
        dict(fit, name="fit_sweep_large", n_configs=30000, d=400, M=4000, zeta=4),
        # mixed precision on the INT8-emulated K_NM, the fastest form of a mid-sized fit
        dict(fit, name="fit_int8", n_configs=10000, d=400, M=2000, zeta=4, precision="fp32", int8=True),
        # the paper-sized training set: 1e5 configurations, about 4e6 atoms, M = 1e4
        dict(fit, name="fit_realistic", n_configs=100000, atoms_lo=16, d=400, M=10000, zeta=4, entry="stream"),
        # energies, forces and virials of a small training set
        dict(kind="forces", name="fit_forces", n_configs=150, atoms_lo=20, atoms_hi=60, d=400, M=1500, zeta=4,
             sigma_per_atom=1e-3, precision="fp64"),
        # sparse-point selection from a quarter of the paper-sized set's rows
        dict(kind="cur", name="cur_select", n_rows=1000000, d=400, M=10000),
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _d(rng):
    """Descriptor lengths: the sweep's, the tiny workload's, or any other."""
    return rng.choice([64, 128, 256, 400, rng.randint(30, 420)])


def draw(rng):
    kind = rng.choice(["predict", "predict", "fit", "fit", "fit", "forces", "cur"])
    if kind == "predict":
        return dict(kind=kind, atoms_lo=8, atoms_hi=64, n_configs=_log(rng, 1, 4096), d=_d(rng),
                    M=_log(rng, 256, 4000), zeta=rng.randint(2, 4))
    if kind == "cur":
        d = _d(rng)
        n = _log(rng, 5000, 1000000)
        return dict(kind=kind, n_rows=n, d=d, M=max(1, n // rng.randint(20, 400)))
    if kind == "forces":
        return dict(kind=kind, n_configs=_log(rng, 12, 300), atoms_lo=20, atoms_hi=60, d=_d(rng),
                    M=_log(rng, 100, 2000), zeta=rng.randint(2, 4), sigma_per_atom=1e-3,
                    precision=rng.choice(["fp64", "fp32"]))
    precision = rng.choice(["fp64", "fp64", "fp32"])
    entry = rng.choice(["wait", "queue", "static"])
    # the allocation-free entry point takes what fits its 256 MiB
    n = _log(rng, 200, 4000 if entry == "static" else 30000)
    M = _log(rng, max(40, n // 60), min(800 if entry == "static" else 4000, n // 2))
    return dict(kind=kind, n_configs=n, atoms_lo=8, atoms_hi=64, d=_d(rng), M=M, zeta=rng.randint(2, 4),
                sigma_per_atom=rng.choice([1e-3, 1e-2]), precision=precision,
                int8=entry != "static" and rng.random() < 0.25, entry=entry)


# ------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _descriptors(n, d, g):
    """Rows of |N(0, 1)| entries scaled to unit length."""
    X = torch.empty((n, d), dtype=torch.float64, device=DEV)
    for a in range(0, n, 1 << 20):
        x = torch.randn((min(n, a + (1 << 20)) - a, d), dtype=torch.float64, device=DEV, generator=g).abs_()
        X[a:a + x.shape[0]] = x / torch.sqrt((x * x).sum(dim=1, keepdim=True))
    return X


def _offsets(case, g):
    counts = torch.randint(case["atoms_lo"], case["atoms_hi"] + 1, (case["n_configs"],), device=DEV, generator=g)
    offs = torch.zeros(case["n_configs"] + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(counts, 0, out=offs[1:])
    return counts, offs


def _segment_sum(v, offs):
    return torch.segment_reduce(v, "sum", lengths=offs[1:] - offs[:-1])


def _power(a, b, zeta):
    """(a b^T)^zeta, entry by entry."""
    return (a @ b.T) ** zeta


def _energies(X, offs, S, cs, zeta):
    """sum_{i in A} sum_j cs_j (x_i . s_j)^zeta."""
    e = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
    for a in range(0, X.shape[0], 1 << 19):
        e[a:a + (1 << 19)] = _power(X[a:a + (1 << 19)], S, zeta) @ cs
    return _segment_sum(e, offs)


def _training_set(case, seed):
    """Descriptors, sparse rows (drawn from them), targets and their deviations."""
    g = _gen(seed)
    counts, offs = _offsets(case, g)
    n = int(offs[-1])
    X = _descriptors(n, case["d"], g)
    pick = torch.randperm(n, device=DEV, generator=g)[:case["M"]].sort().values
    XM = X[pick].contiguous()
    S, cs = XM[:N_TRUE], torch.randn(min(N_TRUE, case["M"]), dtype=torch.float64, device=DEV, generator=g)
    sigma = case["sigma_per_atom"] * counts.to(torch.float64)
    noise = torch.randn(case["n_configs"], dtype=torch.float64, device=DEV, generator=g)
    y = _energies(X, offs, S, cs, case["zeta"]) + sigma * noise
    return dict(counts=counts, offs=offs, X=X, XM=XM, S=S, cs=cs, sigma=sigma, y=y, g=g)


def _derivatives(case, t):
    """Gradient rows (atom i, slot, coordinate): slot 0 is the atom itself, the others its
    neighbours; forces gather the rows of one moved atom and coordinate, virials all rows
    of a configuration weighted by a position coordinate."""
    g, d, n = t["g"], case["d"], t["X"].shape[0]
    cfg = torch.repeat_interleave(torch.arange(case["n_configs"], device=DEV), t["counts"])
    first, size = t["offs"][:-1][cfg], t["counts"][cfg]
    # each atom's neighbours: NEIGH others of its configuration
    order = torch.rand((n, case["atoms_hi"]), device=DEV, generator=g)
    col = torch.arange(case["atoms_hi"], device=DEV)
    own = torch.arange(n, device=DEV) - first
    order[(col[None, :] >= size[:, None]) | (col[None, :] == own[:, None])] = 2.0
    nb = order.argsort(dim=1, stable=True)[:, :NEIGH] + first[:, None]
    moved = torch.cat([torch.arange(n, device=DEV)[:, None], nb], dim=1)      # [n, 1 + NEIGH]
    grad = torch.randn((n, 1 + NEIGH, 3, d), dtype=torch.float64, device=DEV, generator=g) * (0.3 / math.sqrt(d))
    grad[:, 0] = -grad[:, 1:].sum(dim=1)                                       # translations cost nothing
    n_grad = n * (1 + NEIGH) * 3
    axis = torch.arange(3, device=DEV)
    key = (moved[:, :, None] * 3 + axis).reshape(-1)                           # moved atom and coordinate
    f_rows = torch.argsort(key, stable=True)
    f_len = torch.bincount(key, minlength=3 * n)
    # virials: per configuration and pair (a <= b), the rows along b weighted by r_a
    pos = torch.rand((n, 3), dtype=torch.float64, device=DEV, generator=g) * 4.0
    rows = torch.arange(n_grad, device=DEV).reshape(n, 1 + NEIGH, 3)
    v_rows, v_w, v_cfg = [], [], []
    for q, (a, b) in enumerate([(0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)]):
        v_rows.append(rows[:, :, b].reshape(-1))
        v_w.append(-pos[moved, a].reshape(-1))
        v_cfg.append((6 * cfg[:, None] + q).expand(n, 1 + NEIGH).reshape(-1))
    v_rows, v_w, v_cfg = torch.cat(v_rows), torch.cat(v_w), torch.cat(v_cfg)
    v_order = torch.argsort(v_cfg, stable=True)
    lengths = torch.cat([f_len, torch.bincount(v_cfg, minlength=6 * case["n_configs"])])
    offs = torch.zeros(lengths.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lengths, 0, out=offs[1:])
    obs = dict(x_grad=grad.reshape(n_grad, d).contiguous(),
               grad_atom=torch.arange(n, device=DEV).repeat_interleave((1 + NEIGH) * 3).contiguous(),
               obs_offsets=offs, pos_grad=torch.cat([f_rows, v_rows[v_order]]).contiguous(),
               pos_weight=torch.cat([torch.full((n_grad,), -1.0, dtype=torch.float64, device=DEV),
                                     v_w[v_order]]).contiguous())
    sig = torch.cat([torch.full((3 * n,), SIGMA_F, dtype=torch.float64, device=DEV),
                     SIGMA_V * t["counts"].to(torch.float64).repeat_interleave(6)])
    # targets from the same weights as the energies
    w = (t["X"] @ t["S"].T) ** (case["zeta"] - 1) * t["cs"] * case["zeta"]
    e = torch.cat([(obs["x_grad"][a:a + (1 << 19)] @ t["S"].T * w[obs["grad_atom"][a:a + (1 << 19)]]).sum(dim=1)
                   for a in range(0, n_grad, 1 << 19)])
    v = _segment_sum(e[obs["pos_grad"]] * obs["pos_weight"], offs)
    v += sig * torch.randn(v.numel(), dtype=torch.float64, device=DEV, generator=g)
    return obs, torch.cat([t["sigma"], sig]), torch.cat([t["y"], v])


def _params(case):
    fp32 = case.get("precision") == "fp32"
    return gap.params(case["d"], case["zeta"], 1.0, JITTER, precision=gap.GAP_MIXED_FP32 if fp32 else gap.GAP_FP64,
                      flags=gap.GAP_FLAG_KNM_INT8 if case.get("int8") else 0)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "cur":
        g = _gen(seed)
        X = _descriptors(case["n_rows"], case["d"], g)
        draws = torch.empty(case["n_rows"], dtype=torch.float64, device=DEV).exponential_(generator=g)
        ws = torch.empty(gap.cur_workspace_bytes(case["n_rows"], case["d"]), dtype=torch.uint8, device=DEV)
        return dict(kind=kind, X=X, draws=draws, ws=ws, M=case["M"])
    if kind == "predict":
        g = _gen(seed)
        _, offs = _offsets(case, g)
        X = _descriptors(int(offs[-1]), case["d"], g)
        XM = _descriptors(case["M"], case["d"], g)
        c = torch.randn(case["M"], dtype=torch.float64, device=DEV, generator=g)
        h = gap.Handle(_params(case))
        h.set_model(XM)
        return dict(kind=kind, h=h, X=X, offs=offs, XM=XM, c=c,
                    y=torch.empty(case["n_configs"], dtype=torch.float64, device=DEV))
    t = _training_set(case, seed)
    s = dict(kind=kind, p=_params(case), X=t["X"], offs=t["offs"], XM=t["XM"], sigma=t["sigma"], y=t["y"],
             c=torch.empty(case["M"], dtype=torch.float64, device=DEV), entry=case.get("entry", "wait"))
    n_atoms = t["X"].shape[0]
    if kind == "forces":
        s["obs"], s["sigma"], s["y"] = _derivatives(case, t)
        s["h"] = gap.Handle(s["p"])
        s["h"].alloc_workspace_obs(case["n_configs"], n_atoms, s["obs"]["obs_offsets"].numel() - 1,
                                   s["obs"]["pos_grad"].numel(), case["M"])
    elif s["entry"] == "stream":
        # a large fit on a stream of its own, with CUs kept for the panel chain
        s["stream"] = torch.cuda.Stream()
        s["h"] = gap.Handle(s["p"], stream=s["stream"])
        s["h"].set_tuning(qr_free_cus=32)
        s["h"].alloc_workspace(case["n_configs"], n_atoms, case["M"])
    elif s["entry"] != "static":
        s["h"] = gap.Handle(s["p"])
        s["h"].alloc_workspace(case["n_configs"], n_atoms, case["M"])
    return s


# ------------------------------------------------------------------- a pass
def run(s):
    kind = s["kind"]
    if kind == "predict":
        s["h"].predict(s["X"], s["offs"], s["c"], s["y"])
        return s["y"]
    if kind == "cur":
        picked, lev = gap.cur_select(s["X"], s["M"], draws=s["draws"], leverage=True, workspace=s["ws"])
        return dict(picked=picked, leverage=lev)
    if kind == "forces":
        s["h"].build_knm_obs(s["X"], s["offs"], s["obs"], s["XM"], s["sigma"])
        info = s["h"].solve(s["y"], s["c"])
        return dict(c=s["c"], loss=info.residual_norm2)
    if s["entry"] == "static":
        info = gap.fit_static(s["p"], s["X"], s["offs"], s["XM"], s["sigma"], s["y"], s["c"])
        return dict(c=s["c"], loss=info.residual_norm2)
    if s["entry"] == "stream":
        s["stream"].wait_stream(torch.cuda.current_stream())
    s["h"].build_knm(s["X"], s["offs"], s["XM"], s["sigma"])
    if s["entry"] == "queue":
        s["h"].solve(s["y"], s["c"], info=False)
        return dict(c=s["c"])
    info = s["h"].solve(s["y"], s["c"])
    return dict(c=s["c"], loss=info.residual_norm2)


# ------------------------------------------------------------------- bounds
def work(case):
    d, M = case["d"], case["M"]
    if case["kind"] == "cur":
        n = case["n_rows"]
        # the symmetric Gram matrix and the triangular projection
        return dict(bytes=8 * n * d + 8 * n + 8 * n + 8 * M, flops=2.0 * n * d * d)
    N = case["n_configs"]
    atoms = N * (case["atoms_lo"] + case["atoms_hi"]) / 2
    b = 8 * (atoms * d + M * d + N + 1 + M + N)
    f = 2.0 * atoms * M * d
    if case["kind"] == "predict":
        return dict(bytes=b, flops=f)
    rows = N
    if case["kind"] == "forces":
        n_grad, n_obs, n_pos = 39 * atoms, 3 * atoms + 6 * N, 3 * 39 * atoms
        rows += n_obs
        b += 8 * (n_grad * (d + 1) + 3 * n_obs + 2 * n_pos)
        f += 2.0 * n_grad * M * d + 2.0 * n_pos * M + 2.0 * atoms * M * d
    f += 1.0 * M * M * d + M ** 3 / 3.0 + 2.0 * (rows + 1) * M * (M + 1) + 4.0 * (rows + 1) * M + M * M
    return dict(bytes=b + 8 * rows, flops=f)


def exact(case, seed):
    if case["kind"] == "cur":
        s = prepare(case, seed)
        X = s["X"]
        L = torch.linalg.cholesky((X.T @ X).cpu())
        inv = torch.linalg.solve_triangular(L, torch.eye(case["d"], dtype=torch.float64), upper=False).T.to(DEV)
        lev = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
        for a in range(0, X.shape[0], 1 << 18):
            q = X[a:a + (1 << 18)] @ inv
            lev[a:a + (1 << 18)] = (q * q).sum(dim=1)
        keys = s["draws"] / lev
        return dict(picked=torch.topk(keys, case["M"], largest=False).indices.sort().values, leverage=lev)
    if case["kind"] == "predict":
        s = prepare(case, seed)
        return _energies(s["X"], s["offs"], s["XM"], s["c"], case["zeta"])
    if work(case)["flops"] > 6e12:
        return None
    t = _training_set(case, seed)
    M, zeta, N = case["M"], case["zeta"], case["n_configs"]
    blocks, sigma, y = [], t["sigma"], t["y"]
    K = torch.empty((N, M), dtype=torch.float64, device=DEV)
    for a in range(0, M, 128):
        K[:, a:a + 128] = torch.segment_reduce(_power(t["X"], t["XM"][a:a + 128], zeta), "sum",
                                               lengths=t["counts"], axis=0)
    blocks.append(K)
    if case["kind"] == "forces":
        obs, sigma, y = _derivatives(case, t)
        n_obs, n_grad = obs["obs_offsets"].numel() - 1, obs["x_grad"].shape[0]
        W = torch.sparse_csr_tensor(obs["obs_offsets"], obs["pos_grad"], obs["pos_weight"], size=(n_obs, n_grad))
        KD = torch.empty((n_obs, M), dtype=torch.float64, device=DEV)
        for a in range(0, M, 128):
            XM = t["XM"][a:a + 128]
            G = obs["x_grad"] @ XM.T
            G *= (zeta * _power(t["X"], XM, zeta - 1))[obs["grad_atom"]]
            KD[:, a:a + 128] = W @ G
        blocks.append(KD)
    A = torch.cat(blocks)
    A /= sigma[:, None]
    KMM = _power(t["XM"], t["XM"], zeta).cpu()
    KMM.diagonal().add_(JITTER)
    A = torch.cat([A.cpu(), torch.linalg.cholesky(KMM).T])
    b = torch.cat([(y / sigma).cpu(), torch.zeros(M, dtype=torch.float64)])
    R = torch.linalg.qr(torch.cat([A, b[:, None]], dim=1), mode="r").R
    c = torch.linalg.solve_triangular(R[:M, :M], R[:M, M:], upper=True)[:, 0]
    out = dict(c=c)
    if case.get("entry") != "queue":
        out["loss"] = float(R[M, M]) ** 2
    return out
