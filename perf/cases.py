"""The work that a user of this framework has it do, as measurable cases.

A case names a call (a training step, a forward unroll, a solve to tolerance,
a standalone projection with its derivative), a problem class with its sizes,
a data type and the options in use.  `prepare` builds what a program holds
before the call, `run` makes one pass through the public entry points,
`work` counts what the path cannot do without, and `exact` gives the same
outputs from plain float64 torch and numpy.

Sizes follow the repository's own workloads: one max-cut SDP of order 20 over
100 steps; batches of max-cut SDPs of order 30 to 100; Lovasz SDPs of order
64 to 200; Huber regression with up to 2000 x 500 designs and 200 cones;
covariance steering with 4 to 12 states over 30 to 100 steps; one sparse
program per call for the matrix-free linear solve.  Float32 unrolls are kept
short (a rounding in one step travels through all that follow); float64 ones
run longer.
"""
import math

import numpy as np
import torch

import synth
from paper_2606_13825_amd import CosmoBatch
from paper_2606_13825_amd import binding as api

DEV = "cuda:0"
TORCH = {"f32": torch.float32, "f64": torch.float64}
NUMPY = {"f32": np.float32, "f64": np.float64}


def listed():
    return [
        # one small SDP solved by plain forward steps: launches and latency
        {"name": "maxcut20_f64_forward", "call": "forward", "problem": "maxcut", "dtype": "f64", "B": 1, "lo": 20,
         "hi": 20, "K": 100, "form": 0, "graph": False},
        # the training step of a batch of uneven SDPs, buffers kept, launches replayed
        {"name": "maxcut64_f32_train", "call": "train", "problem": "maxcut", "dtype": "f32", "B": 64, "lo": 30,
         "hi": 100, "K": 4, "form": 0, "graph": True},
        # the same step where eigenvalues repeat and the blocks fill the LDS
        {"name": "lovasz8_f32_train", "call": "train", "problem": "lovasz", "dtype": "f32", "B": 8, "lo": 64, "hi": 200,
         "K": 1, "form": 0, "graph": False},
        # robust regression with dense designs in float64 on float32 data
        {"name": "huber4_f64_train", "call": "train", "problem": "huber", "dtype": "f64", "B": 4, "lo": 2000, "hi": 2000,
         "K": 5, "form": 0, "graph": True},
        # covariance steering, the cooperative CG that the autotuner picks for it
        {"name": "covsteer16_f32_train", "call": "train", "problem": "covsteer", "dtype": "f32", "B": 16, "lo": 30,
         "hi": 100, "K": 2, "form": 4, "graph": False},
        # one large sparse program, the matrix-free backward of a single step
        {"name": "sparse10k_f32_train", "call": "train", "problem": "sparse", "dtype": "f32", "B": 1, "lo": 10000,
         "hi": 10000, "K": 1, "form": 4, "graph": False},
        # the penalty policy inside the unroll, forward and backward
        {"name": "policy16_f32_train", "call": "policy", "problem": "maxcut", "dtype": "f32", "B": 16, "lo": 30,
         "hi": 100, "K": 3, "form": 0, "graph": False},
        # the baseline solver to its tolerance, residuals read every 10 steps
        {"name": "maxcut8_f64_solve", "call": "solve", "problem": "maxcut", "dtype": "f64", "B": 8, "lo": 20, "hi": 60,
         "K": 10, "form": 0, "graph": False},
        # standalone projections and their derivatives: many small blocks, as in one steering step
        {"name": "psd_small_f32", "call": "psd", "dtype": "f32", "B": 2000, "lo": 4, "hi": 24},
        {"name": "psd_medium_f64", "call": "psd", "dtype": "f64", "B": 48, "lo": 20, "hi": 100},
        {"name": "psd_large_f32", "call": "psd", "dtype": "f32", "B": 16, "lo": 129, "hi": 200},
        # second-order cones of a robust-regression batch
        {"name": "soc51200_f64", "call": "soc", "dtype": "f64", "B": 51200, "lo": 3, "hi": 10},
    ]


def draw(rng):
    """One more case of the listed ranges."""
    def log_int(a, b):
        return max(a, min(b, int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))))

    dt = rng.choice(["f32", "f64"])
    kind = rng.choice(["forward", "train", "train", "train", "policy", "solve", "psd", "psd", "soc"])
    if kind == "soc":
        return {"call": "soc", "dtype": dt, "B": log_int(100, 51200), "lo": 3, "hi": rng.randint(4, 10)}
    if kind == "psd":
        top = rng.choice([24, 64, 128, 200 if dt == "f32" else 140])
        hi = log_int(6, top)
        lo = rng.randint(max(2, hi // 3), hi)
        return {"call": "psd", "dtype": dt, "B": max(1, min(2000, log_int(4, 96) * 24 // hi + rng.randint(0, 12))),
                "lo": lo, "hi": hi}
    case = {"call": kind, "problem": "maxcut", "dtype": dt, "form": 0, "graph": False}
    if kind == "forward":
        hi = log_int(10, 80)
        case.update(dtype="f64", B=log_int(1, 12), lo=rng.randint(max(4, hi // 2), hi), hi=hi, K=rng.randint(10, 50),
                    graph=rng.random() < 0.5)
    elif kind == "policy":
        hi = log_int(16, 100)
        case.update(B=log_int(1, 24), lo=rng.randint(max(6, hi // 3), hi), hi=hi, K=rng.randint(1, 3))
    elif kind == "solve":
        hi = log_int(12, 60)
        case.update(dtype="f64", B=log_int(1, 8), lo=rng.randint(max(6, hi // 3), hi), hi=hi, K=10)
    else:
        problem = rng.choice(["maxcut", "lovasz", "huber", "covsteer", "sparse"])
        case["problem"] = problem
        if problem == "maxcut":
            hi = log_int(12, 100)
            case.update(B=log_int(1, 64), lo=rng.randint(max(4, hi // 3), hi), hi=hi, K=rng.randint(1, 4),
                        graph=rng.random() < 0.5)
        elif problem == "lovasz":
            hi = log_int(24, 200 if dt == "f32" else 140)
            case.update(B=rng.randint(1, 8), lo=rng.randint(hi // 3, hi), hi=hi, K=1, graph=rng.random() < 0.5)
        elif problem == "huber":
            obs = log_int(120, 2000)
            case.update(dtype="f64", B=max(1, min(16, log_int(1, 64) * 400 // obs)), lo=obs, hi=obs,
                        K=rng.randint(1, 5), graph=rng.random() < 0.5)
        elif problem == "covsteer":
            hi = log_int(8, 100)
            case.update(B=rng.randint(1, 16), lo=rng.randint(max(4, hi // 3), hi), hi=hi, K=rng.randint(1, 2) if hi <= 50 else 1,
                        form=rng.choice([0, 4]) if hi <= 30 else 4)
        else:
            n = log_int(400, 10000)
            case.update(B=1, lo=n, hi=n, K=1, form=rng.choice([0, 4]))
    return case


# ---- sizes and inputs --------------------------------------------------------------


def _spread(case):
    """B sizes spread evenly over [lo, hi], in a mixed order, the same for every seed."""
    B, lo, hi = case["B"], case["lo"], case["hi"]
    at = [lo + (hi - lo) * i // max(1, B - 1) for i in range(B)]
    return [at[i] for i in np.random.default_rng(B).permutation(B)]


def _instance(case, size, i, rng):
    problem = case["problem"]
    if problem == "maxcut":
        return synth.maxcut_sdp(size, synth.erdos_renyi(size, float(rng.uniform(0.1, 0.5)), rng))
    if problem == "lovasz":   # a connection set of a fixed number of distances
        half = (size - 1) // 2
        conn = 1 + rng.permutation(half)[: max(1, int(0.3 * half))]
        return synth.lovasz_theta_sdp(size, synth.circulant(size, [int(d) for d in conn]))
    if problem == "huber":   # cones of dimension 3 to 10, one dimension per instance
        return synth.huber_socp(rng, n_obs=size, n_coef=size // 4, n_soc=max(1, size // 10), soc_dims=(3 + i % 8,) * 2)
    if problem == "covsteer":
        return synth.covsteer_sdp(rng, (4, 6, 8, 10, 12)[i % 5], size)
    P, A, _, b, xstar = synth.appb_instance(size, rng)
    return synth.ConicInstance(P=P.tocsr(), q=-(P @ xstar), A=A.tocsr(), b=b, cones=[synth.Cone("nonneg", A.shape[0])])


def _problem(case, seed):
    """(instances rounded to the data type, rho [K, m], alpha [K, B]) as float64 numpy.
    The Huber batch holds float32 numbers and iterates in float64."""
    npdt = NUMPY[case["dtype"]]
    data = np.float32 if case["problem"] == "huber" else npdt
    insts, rhos, alphas = [], [], []
    rngs = [np.random.default_rng(s) for s in np.random.SeedSequence(seed).spawn(case["B"])]
    for i, (rng, size) in enumerate(zip(rngs, _spread(case))):
        inst = _instance(case, size, i, rng)
        insts.append(inst.astype(data) if data == np.float32 else inst)
        rho, alpha = synth.perturbed_hyper(inst, case["K"], rng)
        rhos.append(rho.astype(npdt).astype(np.float64))
        alphas.append(alpha.astype(npdt).astype(np.float64))
    return insts, np.concatenate(rhos, axis=1), np.stack(alphas, axis=1)


def _blocks(case, seed):
    """Symmetric blocks with some repeated eigenvalues in svec form, and a
    cotangent: (orders, input, cotangent) as float64 numpy."""
    rng = np.random.default_rng(seed)
    orders = _spread(case)
    vs, gs = [], []
    for p in orders:
        Q = np.linalg.qr(rng.standard_normal((p, p)))[0]
        lam = rng.uniform(0.2, 2.0, p) * np.where(rng.random(p) < 0.5, 1.0, -1.0)
        lam[: p // 4] = rng.uniform(0.5, 1.0)
        vs.append(synth.svec_of_dense((Q * lam) @ Q.T))
        G = rng.standard_normal((p, p))
        gs.append(synth.svec_of_dense(G + G.T) / p)
    npdt = NUMPY[case["dtype"]]
    return orders, np.concatenate(vs).astype(npdt).astype(np.float64), np.concatenate(gs).astype(npdt).astype(np.float64)


def _cones(case, seed):
    rng = np.random.default_rng(seed)
    dims = _spread(case)
    m = int(np.sum(dims))
    v, g = rng.standard_normal(m), rng.standard_normal(m)
    first = np.concatenate([[0], np.cumsum(dims)[:-1]])
    v[first] *= 3.0   # inside, outside and in the polar cone
    npdt = NUMPY[case["dtype"]]
    return dims, v.astype(npdt).astype(np.float64), g.astype(npdt).astype(np.float64)


def _policy_theta(case, seed):
    """Parameters of a policy under training: small random last layers."""
    return api.policy_init(seed, head_scale=0.05, dtype=TORCH[case["dtype"]], device=DEV)


def prepare(case, seed):
    dt = TORCH[case["dtype"]]
    if case["call"] in ("psd", "soc"):
        sizes, v, g = (_blocks if case["call"] == "psd" else _cones)(case, seed)
        return {"case": case, "sizes": sizes, "v": torch.from_numpy(v).to(DEV, dt), "g": torch.from_numpy(g).to(DEV, dt)}
    insts, rho, alpha = _problem(case, seed)
    batch = CosmoBatch(insts, K=case["K"], dtype=dt, device=DEV, dense_f32=case["problem"] == "huber")
    batch.set_pcg_form(case["form"])
    batch.set_graph(case["graph"])
    st = {"case": case, "batch": batch, "rho": torch.from_numpy(rho).to(DEV, dt), "alpha": torch.from_numpy(alpha).to(DEV, dt),
          "ws": batch.new_fwd_ws()}
    if case["call"] == "policy":
        st["theta"] = _policy_theta(case, seed)
        st["bws"] = batch.new_bwd_ws()
    elif case["call"] == "train":
        st["z0"] = [torch.zeros(n, dtype=dt, device=DEV, requires_grad=True) for n in (batch.n_tot, batch.m_tot, batch.m_tot)]
        st["rho"].requires_grad_(True)
        st["alpha"].requires_grad_(True)
    if case["graph"]:   # a replayed program keeps its buffers
        like = [torch.empty(n, dtype=dt, device=DEV) for n in (batch.n_tot, batch.m_tot, batch.m_tot)]
        st["out"] = tuple(like)
        if case["call"] == "train":
            st["rho"], st["alpha"] = st["rho"].detach(), st["alpha"].detach()
            st["tape"], st["bws"] = batch.new_tape(), batch.new_bwd_ws()
            st["cot"] = [torch.empty_like(t) for t in like]
            st["grads"] = tuple([torch.empty_like(st["rho"]), torch.empty_like(st["alpha"])] + [torch.empty_like(t) for t in like])
    return st


def run(st):
    case = st["case"]
    if case["call"] == "psd":
        out, lam, U = api.psd_proj(st["v"], st["sizes"])
        return {"out": out, "gin": api.psd_proj_vjp(lam, U, st["g"], st["sizes"])}
    if case["call"] == "soc":
        return {"out": api.socp_proj(st["v"], st["sizes"]), "gin": api.socp_proj_vjp(st["v"], st["g"], st["sizes"])}
    batch = st["batch"]
    if case["call"] == "forward":
        fw = batch.forward(st["rho"], st["alpha"], tape=False, ws=st["ws"], out=st.get("out"))
        return {"x": fw.x, "s": fw.s, "y": fw.y}
    if case["call"] == "solve":
        iters, rho, x, s, y = batch.solve(max_iter=400, ws=st["ws"])
        return {"iters": iters, "rho": rho, "x": x, "s": s, "y": y}
    if case["call"] == "policy":
        fw = batch.policy_forward(st["theta"], ws=st["ws"])
        gtheta, grho, galpha, gx, gs, gy = batch.policy_backward(st["theta"], fw, ws=st["bws"])
        return {"x": fw.x, "s": fw.s, "y": fw.y, "rho": fw.rho, "alpha": fw.alpha, "loss": fw.loss, "gtheta": gtheta}
    if case["graph"]:
        fw = batch.forward(st["rho"], st["alpha"], tape=st["tape"], ws=st["ws"], out=st["out"])
        loss, cot = batch.residual_loss(fw.x, fw.s, fw.y, ws=st["ws"])
        for kept, new in zip(st["cot"], cot):
            kept.copy_(new)
        bw = batch.backward(st["rho"], st["alpha"], fw.tape, *st["cot"], ws=st["bws"], out=st["grads"])
        return {"x": fw.x, "s": fw.s, "y": fw.y, "loss": loss.sum(), "grho": bw.grho, "galpha": bw.galpha, "gx0": bw.gx0,
                "gs0": bw.gs0, "gy0": bw.gy0}
    x, s, y = api.CosmoUnroll.apply(batch, st["rho"], st["alpha"], *st["z0"])
    loss = api.ResidualLoss.apply(batch, x, s, y)
    grads = torch.autograd.grad(loss, [st["rho"], st["alpha"]] + st["z0"])
    return dict(zip(("x", "s", "y", "loss", "grho", "galpha", "gx0", "gs0", "gy0"), (x, s, y, loss) + grads))


# ---- what the path cannot do without -------------------------------------------------


def _counts(case, size, i):
    """(columns, rows, nonzeros read as CSR, dense values, PSD orders) of one instance."""
    problem = case["problem"]
    tri = size * (size + 1) // 2
    if problem == "maxcut":
        return tri, tri + size, tri + size, 0, [size]
    if problem == "lovasz":
        edges = max(1, int(0.3 * ((size - 1) // 2))) * size
        return tri, tri + 1 + edges, tri + size + edges, 0, [size]
    if problem == "huber":
        soc = max(1, size // 10) * (3 + i % 8)
        return size // 4 + 2 * size, 2 * size + soc, 4 * size + soc, size * (size // 4), []
    if problem == "covsteer":
        nx = (4, 6, 8, 10, 12)[i % 5]
        nu, T = nx // 2, size
        ns, ny, b1, b2 = nx * (nx + 1) // 2, nu * (nu + 1) // 2, (nx + nu) * (nx + nu + 1) // 2, nx * (2 * nx + 1)
        nnz = T * (b1 + 2 * ns + nx * nx * (nx + nu))
        return T * (ns + nu * nx + ny), T * (b1 + b2) + ns, nnz, 0, [nx + nu] * T + [2 * nx] * T + [nx]
    return size, size // 2, size * (size // 2) // 100 + size, 0, []


def work(case):
    """Inputs read and outputs written once; 11 p^3 flops for a projection by
    its eigendecomposition, 8 p^3 for its derivative, and one application of
    the operator for a linear solve."""
    esz = 4 if case["dtype"] == "f32" else 8
    sizes = _spread(case)
    if case["call"] == "psd":
        rows = sum(p * (p + 1) // 2 for p in sizes)
        return {"bytes": 4 * rows * esz, "flops": sum(19 * p ** 3 for p in sizes)}
    if case["call"] == "soc":
        return {"bytes": 5 * sum(sizes) * esz, "flops": 12 * sum(sizes)}
    n = m = nnz = dense = cubes = 0
    for i, size in enumerate(sizes):
        a = _counts(case, size, i)
        n, m, nnz, dense = n + a[0], m + a[1], nnz + a[2], dense + a[3]
        cubes += sum(p ** 3 for p in a[4])
    both = case["call"] in ("train", "policy")
    K = case["K"] if case["call"] != "solve" else 40   # a solve takes some tens of steps at least
    data = nnz * (4 + esz) + dense * min(esz, 4) + (n + m) * esz
    steps = K * (m * esz) * (2 if both else 1)         # penalties in, their gradients out
    out = (n + 2 * m) * esz * (3 if both else 1)
    per_step = 11 * cubes + 4 * (nnz + 2 * dense)
    if both:
        per_step += 8 * cubes + 4 * (nnz + 2 * dense)
    if case["call"] == "policy":
        per_step += 7744 * m
    return {"bytes": data + steps + out, "flops": K * per_step}


# ---- the same outputs from plain float64 torch and numpy --------------------------------


def _smat(v, p):
    c, r = np.tril_indices(p)   # svec order: column c holds rows r = 0..c
    S = np.zeros((p, p))
    w = v * np.where(r == c, 1.0, math.sqrt(0.5))
    S[r, c] = w
    S[c, r] = w
    return S


def _svec(S):
    c, r = np.tril_indices(S.shape[0])
    return S[r, c] * np.where(r == c, 1.0, math.sqrt(2.0))


def _psd_project(v, g=None):
    """The projection of one svec block and, for a cotangent, its derivative."""
    p = int((math.isqrt(8 * len(v) + 1) - 1) // 2)
    lam, U = np.linalg.eigh(_smat(v, p))
    pos = np.maximum(lam, 0.0)
    if g is None:
        return _svec((U * pos) @ U.T)
    up = lam > 0
    W = np.where(up[:, None] & up[None, :], 1.0, 0.0)
    mixed = up[:, None] != up[None, :]
    W[mixed] = (np.maximum(pos[:, None], pos[None, :]) / np.maximum(np.abs(lam)[:, None] + np.abs(lam)[None, :], 1e-300))[mixed]
    return _svec(U @ (W * (U.T @ _smat(g, p) @ U)) @ U.T)


class _PsdBlocks(torch.autograd.Function):
    @staticmethod
    def forward(ctx, v, spans):
        ctx.spans, ctx.v = spans, v.detach().cpu().numpy()
        out = np.zeros_like(ctx.v)
        for a, b in spans:
            out[a:b] = _psd_project(ctx.v[a:b])
        return torch.from_numpy(out).to(v.device)

    @staticmethod
    def backward(ctx, g):
        gn = g.detach().cpu().numpy()
        out = np.zeros_like(gn)
        for a, b in ctx.spans:
            out[a:b] = _psd_project(ctx.v[a:b], gn[a:b])
        return torch.from_numpy(out).to(g.device), None


def _soc_project(V):
    """Rows (t, w) of equal dimension, differentiable."""
    t, w = V[:, :1], V[:, 1:]
    nrm = torch.sqrt(torch.clamp((w * w).sum(1, keepdim=True), min=1e-300))
    a = 0.5 * (t + nrm)
    edge = torch.cat([a, a / nrm * w], 1)
    return torch.where(nrm <= t, V, torch.where(nrm <= -t, torch.zeros_like(V), edge))


class _Product(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, M, Mt):
        ctx.pair = (M, Mt)
        return M @ x

    @staticmethod
    def backward(ctx, g):
        M, Mt = ctx.pair
        return _Product.apply(g, Mt, M), None, None


class _Stack:
    """The stacked problem and one differentiable step of the iteration."""

    def __init__(self, insts):
        self.B = len(insts)
        A, self.Arow, self.Acol, self.Aval = self._csr([i.A.tocsr() for i in insts])
        P, _, _, _ = self._csr([i.P.tocsr() for i in insts])
        self.A, self.At = A, torch.sparse_coo_tensor(torch.stack([self.Acol, self.Arow]), self.Aval,
                                                     (A.shape[1], A.shape[0])).to_sparse_csr()
        self.P = P
        to = lambda a: torch.from_numpy(np.concatenate([np.asarray(x, np.float64) for x in a])).to(DEV)  # noqa: E731
        self.q, self.b = to([i.q for i in insts]), to([i.b for i in insts])
        self.pdiag = to([i.P.diagonal() for i in insts])
        rep = lambda ns: torch.from_numpy(np.repeat(np.arange(self.B), ns)).to(DEV)  # noqa: E731
        self.cinst, self.rinst = rep([i.A.shape[1] for i in insts]), rep([i.A.shape[0] for i in insts])
        kind, block, self.psd, soc, row, nb = [], [], [], {}, 0, 0
        for inst in insts:
            for c in inst.cones:
                kind.append(np.full(c.rows, ("zero", "nonneg", "soc", "psd").index(c.kind)))
                if c.kind in ("soc", "psd"):
                    block.append(np.full(c.rows, nb))
                    nb += 1
                else:
                    block.append(nb + np.arange(c.rows))
                    nb += c.rows
                if c.kind == "psd":
                    self.psd.append((row, row + c.rows))
                if c.kind == "soc":
                    soc.setdefault(c.rows, []).append(row)
                row += c.rows
        self.kind = torch.from_numpy(np.concatenate(kind)).to(DEV)
        self.block = torch.from_numpy(np.concatenate(block)).to(DEV)
        self.nb = nb
        self.bsize = torch.zeros(nb, dtype=torch.float64, device=DEV).index_add_(0, self.block, torch.ones_like(self.b))
        self.soc = [torch.from_numpy(np.asarray(r)[:, None] + np.arange(d)).to(DEV) for d, r in soc.items()]
        self.psd_rows, self.nonneg, self.zero = self.kind == 3, self.kind == 1, self.kind == 0

    @staticmethod
    def _csr(mats):
        rows, cols, vals, r0, c0 = [], [], [], 0, 0
        for M in mats:
            rows.append(np.repeat(np.arange(M.shape[0]), np.diff(M.indptr)) + r0)
            cols.append(M.indices.astype(np.int64) + c0)
            vals.append(M.data.astype(np.float64))
            r0, c0 = r0 + M.shape[0], c0 + M.shape[1]
        r, c, v = (torch.from_numpy(np.concatenate(a)).to(DEV) for a in (rows, cols, vals))
        return torch.sparse_coo_tensor(torch.stack([r, c]), v, (r0, c0)).to_sparse_csr(), r, c, v

    def sum_of(self, v, inst):
        return torch.zeros(self.B, dtype=torch.float64, device=DEV).index_add_(0, inst, v)

    def solve(self, rho, rhs, sigma=1e-6):
        """Conjugate gradients in float64, restarted from the true residual."""
        op = lambda x: self.P @ x + sigma * x + self.At @ (rho * (self.A @ x))  # noqa: E731
        dg = (self.pdiag + sigma).index_add(0, self.Acol, rho[self.Arow] * self.Aval ** 2)
        x, bb = torch.zeros_like(rhs), self.sum_of(rhs * rhs, self.cinst)
        for _ in range(3):
            r = rhs - op(x)
            z = r / dg
            p, rz = z.clone(), self.sum_of(r * z, self.cinst)
            for it in range(3000):
                Mp = op(p)
                pMp = self.sum_of(p * Mp, self.cinst)
                a = torch.where(pMp > 0, rz / pMp, torch.zeros_like(rz))[self.cinst]
                x, r = x + a * p, r - a * Mp
                z = r / dg
                new = self.sum_of(r * z, self.cinst)
                p = z + torch.where(rz > 0, new / rz, torch.zeros_like(rz))[self.cinst] * p
                rz = new
                if it % 10 == 9 and bool((self.sum_of(r * r, self.cinst) <= 1e-30 * bb).all()):
                    break
        return x

    def rectify(self, rho):
        mean = torch.zeros(self.nb, dtype=torch.float64, device=DEV).index_add(0, self.block, rho) / self.bsize
        return mean[self.block]

    def product(self, x):
        return _Product.apply(x, self.A, self.At)

    def adjoint(self, y):
        return _Product.apply(y, self.At, self.A)

    def project(self, v):
        out = torch.where(self.zero, torch.zeros_like(v), torch.where(self.nonneg, torch.clamp(v, min=0.0), v))
        for idx in self.soc:
            out = out.index_put((idx.reshape(-1),), _soc_project(v[idx]).reshape(-1))
        return torch.where(self.psd_rows, _PsdBlocks.apply(v, self.psd), out) if self.psd else out

    def step(self, x, s, y, rho, alpha):
        """(x+, s+, y+, s~) of one step with per-row rho and per-instance alpha."""
        rh = self.rectify(rho)
        xi = 1e-6 * x - self.q + self.adjoint(y + rh * (self.b - s))
        xt = _Solve.apply(rh, xi, self)
        st = self.b - self.product(xt)
        ac, ar = alpha[self.cinst], alpha[self.rinst]
        sh = ar * st + (1 - ar) * s
        sn = self.project(sh + y / rh)
        return ac * xt + (1 - ac) * x, sn, y + rh * (sh - sn), st

    def residuals(self, x, s, y):
        Ax, Px, Aty = self.product(x), _Product.apply(x, self.P, self.P), self.adjoint(y)
        return Ax + s - self.b, Px + self.q - Aty, Ax, Px, Aty

    def largest(self, v, inst):
        """Infinity norm per instance, ties sharing the cotangent."""
        cuts = torch.bincount(inst, minlength=self.B).tolist()
        return torch.stack([t.abs().amax() for t in torch.split(v, cuts)])


class _Solve(torch.autograd.Function):
    @staticmethod
    def forward(ctx, rho, rhs, stack):
        x = stack.solve(rho, rhs)
        ctx.stack = stack
        ctx.save_for_backward(rho, x)
        return x

    @staticmethod
    def backward(ctx, g):
        rho, x = ctx.saved_tensors
        w = ctx.stack.solve(rho, g)
        return -(ctx.stack.A @ w) * (ctx.stack.A @ x), w, None


def _mlp(xi, th, n_in):
    sizes = [(n_in, 32), (32,), (32, 32), (32,), (32,), (1,)]
    W1, b1, W2, b2, w3, b3 = (t.reshape(s) for t, s in zip(torch.split(th, [math.prod(s) for s in sizes]), sizes))
    return torch.relu(torch.relu(xi @ W1 + b1) @ W2 + b2) @ w3 + b3[0]


def _policy_exact(S, theta, K, n, m):
    cuts = [7 * 32 + 32 + 32 * 32 + 65, 5 * 32 + 32 + 32 * 32 + 65, 4, 1]
    th_r, th_a, l0, la0 = torch.split(theta, cuts)
    x, s, y = (torch.zeros(k, dtype=torch.float64, device=DEV) for k in (n, m, m))
    lr, la = l0[S.kind], la0.expand(S.B)
    lo, hi = math.log(1e-3), math.log(1e3)
    prev = tilde = None
    rhos, alphas, loss = [], [], torch.zeros(S.B, dtype=torch.float64, device=DEV)
    rp, rd, Ax, Px, Aty = S.residuals(x, s, y)
    Dp, Dd = S.sum_of(rp.detach() ** 2, S.rinst), S.sum_of(rd.detach() ** 2, S.cinst)
    Dp, Dd = (torch.where(D > 0, D, torch.ones_like(D)) for D in (Dp, Dd))
    for k in range(K + 1):
        rp, rd, Ax, Px, Aty = S.residuals(x, s, y)
        if k:
            loss = loss + torch.log(S.sum_of(rd * rd, S.cinst) / Dd + S.sum_of(rp * rp, S.rinst) / Dp)
        if k == K:
            return x, s, y, torch.stack(rhos), torch.stack(alphas), loss
        Np = torch.stack([S.largest(v, S.rinst) for v in (Ax, s, S.b)]).amax(0)
        Nd = torch.stack([S.largest(v, S.cinst) for v in (Px, S.q, Aty)]).amax(0)
        ip, id_ = (torch.where(N > 0, 1 / torch.where(N > 0, N, torch.ones_like(N)), torch.zeros_like(N)) for N in (Np, Nd))
        rbp, rbd = rp * ip[S.rinst], rd * id_[S.cinst]
        dp = torch.zeros_like(s) if tilde is None else s - tilde
        dd = torch.zeros_like(s) if prev is None else s - prev
        log = lambda v, inst: torch.log(S.largest(v, inst) + 1e-12)  # noqa: E731
        gd = log(rbd, S.cinst)
        lr = lr + _mlp(torch.stack([lr, s, y, rbp, gd[S.rinst], dp, dd], 1), th_r, 7)
        la = la + _mlp(torch.stack([la, log(rbp, S.rinst), gd, log(dp, S.rinst), log(dd, S.rinst)], 1), th_a, 5)
        rhos.append(torch.exp(lo + (hi - lo) * torch.sigmoid(lr)))
        alphas.append(2 * torch.sigmoid(la))
        prev = s
        x, s, y, tilde = S.step(x, s, y, rhos[-1], alphas[-1])


def _solve_exact(S, K, n, m, max_iter=400, interval=40, eps=1e-3):
    x, s, y = (torch.zeros(k, dtype=torch.float64, device=DEV) for k in (n, m, m))
    rho, it_of = np.full(S.B, 0.1), np.full(S.B, -1, np.int32)
    kept = [torch.zeros_like(v) for v in (x, s, y)]
    alpha = torch.full((S.B,), 1.6, dtype=torch.float64, device=DEV)

    def keep(mask, src, dst):
        c, r = mask[S.cinst], mask[S.rinst]
        return [torch.where(k, a, d) for k, a, d in zip((c, r, r), src, dst)]

    for it in range(1, max_iter + 1):
        rows = torch.from_numpy(rho).to(DEV)[S.rinst] * torch.where(S.zero, 1e3, 1.0)
        x, s, y, _ = S.step(x, s, y, rows, alpha)
        if it % K:
            continue
        rp, rd, Ax, Px, Aty = S.residuals(x, s, y)
        norm = lambda v, inst: S.largest(v, inst).cpu().numpy()  # noqa: E731
        p, d = norm(rp, S.rinst), norm(rd, S.cinst)
        Np = np.max([norm(v, S.rinst) for v in (Ax, s, S.b)], axis=0)
        Nd = np.max([norm(v, S.cinst) for v in (Px, S.q, Aty)], axis=0)
        now = (p <= eps + eps * Np) & (d <= eps + eps * Nd) & (it_of < 0)
        it_of[now] = it
        kept = keep(torch.from_numpy(now).to(DEV), (x, s, y), kept)
        if (it_of >= 0).all():
            break
        if it % interval == 0:
            for i in np.flatnonzero((it_of < 0) & (Np > 0) & (Nd > 0) & (d > 0)):
                new = min(max(rho[i] * math.sqrt((p[i] / Np[i]) / (d[i] / Nd[i])), 1e-6), 1e6)
                if new > 5 * rho[i] or new < rho[i] / 5:
                    rho[i] = new
    x, s, y = keep(torch.from_numpy(it_of < 0).to(DEV), (x, s, y), kept)
    return {"iters": it_of, "rho": rho, "x": x, "s": s, "y": y}


def exact(case, seed):
    if case["call"] == "psd":
        orders, v, g = _blocks(case, seed)
        ends = np.cumsum([p * (p + 1) // 2 for p in orders])
        parts = list(zip(np.split(v, ends[:-1]), np.split(g, ends[:-1])))
        return {"out": np.concatenate([_psd_project(a) for a, _ in parts]),
                "gin": np.concatenate([_psd_project(a, b) for a, b in parts])}
    if case["call"] == "soc":
        dims, v, g = _cones(case, seed)
        v = torch.from_numpy(v).requires_grad_(True)
        first, out = np.concatenate([[0], np.cumsum(dims)[:-1]]), torch.zeros(len(g), dtype=torch.float64)
        for d in sorted(set(dims)):
            idx = torch.from_numpy(first[np.asarray(dims) == d][:, None] + np.arange(d))
            out = out.index_put((idx.reshape(-1),), _soc_project(v[idx]).reshape(-1))
        return {"out": out.detach(), "gin": torch.autograd.grad(out, v, torch.from_numpy(g))[0]}
    insts, rho, alpha = _problem(case, seed)
    S = _Stack(insts)
    n, m, K = S.q.numel(), S.b.numel(), case["K"]
    rho, alpha = torch.from_numpy(rho).to(DEV), torch.from_numpy(alpha).to(DEV)
    if case["call"] == "solve":
        with torch.no_grad():
            return _solve_exact(S, K, n, m)
    if case["call"] == "policy":
        theta = _policy_theta(case, seed).double().requires_grad_(True)
        x, s, y, rhos, alphas, loss = _policy_exact(S, theta, K, n, m)
        gtheta = torch.autograd.grad(loss.sum(), theta)[0]
        return {"x": x, "s": s, "y": y, "rho": rhos, "alpha": alphas, "loss": loss, "gtheta": gtheta}
    z0 = [torch.zeros(k, dtype=torch.float64, device=DEV) for k in (n, m, m)]
    train = case["call"] == "train"
    leaves = [t.requires_grad_(train) for t in [rho, alpha] + z0]
    x, s, y = z0
    for k in range(K):
        x, s, y, _ = S.step(x, s, y, rho[k], alpha[k])
    if not train:
        return {"x": x, "s": s, "y": y}
    rp, rd = S.residuals(x, s, y)[:2]
    loss = (rp * rp).sum() + (rd * rd).sum()
    grads = torch.autograd.grad(loss, leaves)
    return dict(zip(("x", "s", "y", "loss", "grho", "galpha", "gx0", "gs0", "gy0"), (x, s, y, loss) + grads))
