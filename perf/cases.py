"""Timed cases of the GAP regression hot path on one GPU.

The calls a program that fits and uses sparse-GPR potentials makes, over the
sizes this repository's workloads have: prediction of one small configuration
up to a 65,536-atom set, energies with gradients for training by autograd, and
least-squares fits from 1,800 to 116,667 atoms, in FP64 and with split-BF16
contractions plus FP64 refinement.

A case is a dict of plain values:
  kind     predict | screen | train | fit | stream | model
  n_cfg, lo, hi   configurations of lo .. hi atoms (uniform)
  D, M     descriptor length, number of sparse points
  nb       mean number of neighbour pairs of an atom (0: no pairs)
  dt       dtype of descriptors and Jacobians, f32 | f64
  prec     contraction arithmetic, fp64 | bf16x3

Inputs are drawn on the GPU from the seed, with the recipe of `synth`: unit-norm
Gaussian descriptors, Jacobian entries of standard deviation 0.1, neighbours
within the atom's own configuration, sparse points copied from the descriptors,
targets of a hidden model plus noise of the regularisation's size.  Neighbour
counts vary from atom to atom (2/3 nb .. 4/3 nb), as neighbour lists do.
"""
from __future__ import annotations

import torch

import paper_2310_03921_amd as gapx

DEV = "cuda"
ZETA, DELTA = 4, 1.0
JITTER, SIGMA_E, SIGMA_F, SIGMA_V, SIGMA_L = 1e-8, 1e-3, 1e-2, 1e-1, 1e-2
R_CUT, CUT_WIDTH, THETA, M_2B = 4.5, 1.0, 0.4, 10   # two-body block of `model`
REFINE = 3        # refinement steps a mixed fit may take
STREAM_STEPS = 2  # refinement passes of a streamed fit
STREAM_GROUPS = 2  # configuration groups of a streamed fit
TRAIN_DESC = 4096  # descriptors behind the variance factor of `screen`
_DTYPE = {"f32": torch.float32, "f64": torch.float64}


def _case(name, kind, n_cfg, lo, hi, D, M, nb, dt="f64", prec="fp64"):
    c = {"kind": kind, "n_cfg": n_cfg, "lo": lo, "hi": hi, "D": D, "M": M, "nb": nb, "dt": dt,
         "prec": prec}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a molecular-dynamics step of a small cell: energy and forces, one call per step
        _case("md_step_64", "predict", 1, 64, 64, 252, 2000, 30),
        # the same for a few hundred atoms in FP32, lengths that are no multiple of a tile
        _case("md_step_odd_f32", "predict", 1, 217, 217, 333, 1501, 41, dt="f32"),
        # a molecular-dynamics step of many replicas, split-BF16 contractions
        _case("md_replicas_bf16x3", "predict", 64, 96, 256, 1000, 4000, 40, dt="f32",
              prec="bf16x3"),
        # evaluation of a whole set, the 65,536-atom workload in FP64 arithmetic
        _case("predict_65k", "predict", 256, 256, 256, 1000, 4000, 40, dt="f32"),
        # active learning: energies, forces and variances of a batch of candidates
        _case("screen_40cfg", "screen", 40, 16, 216, 252, 2000, 30),
        # a training step through autograd: energies, then all three gradients
        _case("train_5k", "train", 1, 5021, 5021, 252, 500, 0),
        # the same for a large batch in FP32 with split-BF16 contractions
        _case("train_65k_bf16x3", "train", 1, 65536, 65536, 1000, 4000, 0, dt="f32",
              prec="bf16x3"),
        # the small fit of the tests and of a first trial (1,800 atoms)
        _case("fit_small", "fit", 50, 8, 64, 252, 200, 20),
        # the 116,667-atom FP64 fit
        _case("fit_116k", "fit", 1000, 16, 216, 252, 2000, 30),
        # a quarter of it with split-BF16 rows and FP64 refinement
        _case("fit_29k_mixed", "fit", 250, 16, 216, 252, 2000, 30, prec="bf16x3"),
        # long descriptors, folded by configuration groups: what does not fit whole
        _case("stream_17k_mixed", "stream", 120, 32, 256, 1500, 4000, 40, dt="f32",
              prec="bf16x3"),
        # a model of several targets and descriptors: CUR sparse points, energies, forces,
        # virials and local properties, a two-body block beside the dot-product block
        _case("model_blocks", "model", 60, 9, 70, 150, 301, 25),
    ]


def draw(rng):
    case = _draw(rng)
    # no more work than the largest listed cases
    top = 2.5e13 if case["prec"] == "bf16x3" else 1.3e13
    while (w := work(case))["flops"] > top or w["bytes"] > 3.2e10:
        case["n_cfg"] = case["n_cfg"] * 2 // 3
    if case["kind"] == "model":  # selected among the atoms, whose descriptors have full rank
        n = int(_counts(case).sum())
        case["D"], case["M"] = min(case["D"], n // 2), min(case["M"], n // 2)
    return case


def _draw(rng):
    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    kind = rng.choice(["predict", "predict", "screen", "train", "fit", "fit", "stream", "model"])
    dt = rng.choice(["f64", "f32"])
    prec = rng.choice(["fp64", "bf16x3"])
    if kind == "predict":
        hi = rng.randint(24, 256)
        return _case(None, kind, log(1, 200), rng.randint(8, hi), hi, log(24, 1000),
                     log(100, 4000), rng.randint(8, 48), dt, prec)
    if kind == "screen":
        hi = rng.randint(24, 216)
        return _case(None, kind, log(1, 120), rng.randint(8, hi), hi, log(24, 600),
                     log(100, 2500), rng.randint(8, 40), dt)
    if kind == "train":
        n = log(64, 65536)
        return _case(None, kind, 1, n, n, log(24, 1000), log(50, 4000), 0, dt, prec)
    if kind == "fit":
        hi = rng.randint(24, 216)
        return _case(None, kind, log(20, 400), rng.randint(8, hi), hi, log(24, 300),
                     log(50, 2000), rng.randint(8, 36), dt, prec)
    if kind == "stream":
        hi = rng.randint(48, 256)
        return _case(None, kind, log(16, 120), rng.randint(16, hi), hi, log(300, 1500),
                     log(300, 4000), rng.randint(16, 44), "f32", "bf16x3")
    hi = rng.randint(16, 80)
    return _case(None, kind, log(20, 120), rng.randint(6, hi), hi, log(24, 300), log(50, 500),
                 rng.randint(8, 32), dt)


# ------------------------------------------------------------------ inputs ----
def _counts(case):
    """Atoms of each configuration (from the case alone, so that sizes do not vary with the seed)."""
    g = torch.Generator().manual_seed(1000003 * case["n_cfg"] + case["hi"])
    return torch.randint(case["lo"], case["hi"] + 1, (case["n_cfg"],), generator=g)


def _pair_counts(case, n):
    g = torch.Generator().manual_seed(7919 * n + case["nb"])
    nb = case["nb"]
    return torch.randint(nb - nb // 3, nb + nb // 3 + 1, (n,), generator=g)


def _ptr(counts):
    return torch.cat([torch.zeros(1, dtype=torch.int64), counts.cumsum(0)])


def _pad4(x, D):
    """Rows zero-padded to a multiple of four entries (the library's row layout)."""
    return x if D % 4 == 0 else torch.nn.functional.pad(x, (0, 4 - D % 4))


def _inputs(case, seed):
    g = torch.Generator(DEV).manual_seed(seed)
    D, M, dt = case["D"], case["M"], _DTYPE[case["dt"]]
    counts = _counts(case)
    n = int(counts.sum())
    cfg_ptr = _ptr(counts)
    desc = torch.randn(n, D, dtype=torch.float64, device=DEV, generator=g)
    desc = (desc / desc.norm(dim=1, keepdim=True)).to(dt)
    inp = {"n": n, "cfg_ptr": cfg_ptr.to(DEV), "desc": desc}
    if case["kind"] == "model":  # its sparse points are selected in the pass
        inp["X"] = None
    elif n >= M:
        inp["X"] = desc[torch.randperm(n, device=DEV, generator=g)[:M]].double()
    else:  # a model fitted elsewhere: sparse points of the same distribution
        X = torch.randn(M, D, dtype=torch.float64, device=DEV, generator=g)
        inp["X"] = X / X.norm(dim=1, keepdim=True)
    inp["c"] = torch.randn(M, dtype=torch.float64, device=DEV, generator=g)
    if case["nb"]:
        npair = _pair_counts(case, n)
        P = int(npair.sum())
        src = torch.repeat_interleave(torch.arange(n), npair).to(DEV)
        cfg = torch.repeat_interleave(torch.arange(case["n_cfg"]), counts).to(DEV)[src]
        u = torch.rand(P, dtype=torch.float64, device=DEV, generator=g)
        cnt = counts.to(DEV)[cfg]
        j = inp["cfg_ptr"][cfg] + torch.minimum((u * cnt).long(), cnt - 1)
        jac = torch.empty(P, 3, -(-D // 4) * 4, dtype=dt, device=DEV).normal_(0.0, 0.1, generator=g)
        jac[:, :, D:] = 0
        inp |= {"pair_ptr": _ptr(npair).to(DEV), "pair_j": j.to(torch.int32), "jac": jac,
                "src": src, "cfg_of_pair": cfg}
    if case["kind"] in ("fit", "stream", "model"):
        N, nc = n, case["n_cfg"]
        sig = torch.empty(nc + 3 * N, dtype=torch.float64, device=DEV)
        sig[:nc] = SIGMA_E * counts.to(DEV).double().sqrt()
        sig[nc:] = SIGMA_F
        inp["sigma"] = sig
        noise = torch.randn(nc + 3 * N, dtype=torch.float64, device=DEV, generator=g) * sig
        X = inp["X"]
        if X is None:
            X = desc[torch.randperm(n, device=DEV, generator=g)[:M]].double()
        e, gr = _energies(desc.double(), X, inp["c"])
        inp["y"] = torch.cat([_per_cfg(inp, e), _forces(inp, gr, D).reshape(-1)]) + noise
    if case["kind"] == "model":
        r = torch.randn(inp["src"].numel(), 3, dtype=torch.float64, device=DEV, generator=g)
        rad = 5.0 * torch.rand(r.shape[0], 1, dtype=torch.float64, device=DEV, generator=g) ** (1 / 3)
        inp["pair_r"] = r / r.norm(dim=1, keepdim=True) * rad.clamp(min=0.5)
        inp["x2b"] = torch.linspace(1.0, 4.2, M_2B, dtype=torch.float64, device=DEV)
        inp["local"] = torch.arange(0, n, 3, dtype=torch.int32, device=DEV)
        nv, nl = 9 * case["n_cfg"], inp["local"].numel()
        inp["y"] = torch.cat([inp["y"],
                              SIGMA_V * torch.randn(nv, dtype=torch.float64, device=DEV, generator=g),
                              e[inp["local"].long()] +
                              SIGMA_L * torch.randn(nl, dtype=torch.float64, device=DEV, generator=g)])
        inp["sigma"] = torch.cat([inp["sigma"], torch.full((nv,), SIGMA_V, dtype=torch.float64, device=DEV),
                                  torch.full((nl,), SIGMA_L, dtype=torch.float64, device=DEV)])
    if case["kind"] == "train":
        inp["g_e"] = torch.randn(n, dtype=torch.float64, device=DEV, generator=g)
    if case["kind"] == "screen":
        t = torch.randn(TRAIN_DESC, D, dtype=torch.float64, device=DEV, generator=g)
        t = t / t.norm(dim=1, keepdim=True)
        K = _k(t, inp["X"]) / SIGMA_F
        inp["Kmm"] = _k(inp["X"], inp["X"])
        eye = torch.eye(M, dtype=torch.float64, device=DEV)
        # upper triangular R with R^T R = A^T A; held column-major, as a fit leaves it
        inp["R"] = torch.linalg.cholesky(inp["Kmm"] + JITTER * eye + K.T @ K).contiguous()
    return inp


_gap = None


def _handle():
    """The library handle a program opens once and keeps."""
    global _gap
    if _gap is None:
        _gap = gapx.Gap()
        _gap.set_fit_report(False)
    return _gap


def _atoms(inp, D):
    n = inp["n"]
    z = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    return gapx.Atoms(inp["cfg_ptr"], _pad4(inp["desc"], D), inp.get("pair_ptr", z),
                      inp.get("pair_j", torch.zeros(0, dtype=torch.int32, device=DEV)),
                      inp.get("jac"), D)


def prepare(case, seed):
    inp = _inputs(case, seed)
    D, M = case["D"], case["M"]
    gap = _handle()
    s = {"case": case, "gap": gap}
    if case["kind"] == "train":
        s |= {"desc": inp["desc"].requires_grad_(), "X": inp["X"].requires_grad_(),
              "c": inp["c"].requires_grad_(), "g_e": inp["g_e"]}
        return s
    atoms = _atoms(inp, D)
    s["atoms"] = atoms
    s["c"] = inp["c"]
    if inp["X"] is not None:
        s["sparse"] = gapx.Sparse(_pad4(inp["X"], D).contiguous(), D, ZETA, DELTA)
    for k in ("y", "sigma", "Kmm", "R", "pair_r", "local"):
        if k in inp:
            s[k] = inp[k]
    if case["kind"] == "fit":
        s["A"] = gap.design_buffer(atoms, s["sparse"])
        s["Kmm"] = torch.empty(M, M, dtype=torch.float64, device=DEV)
    elif case["kind"] == "stream":
        s["Kmm"] = torch.empty(M, M, dtype=torch.float64, device=DEV)
        s["groups"] = []
        nc = case["n_cfg"]
        cut = [nc * i // STREAM_GROUPS for i in range(STREAM_GROUPS + 1)]
        for c0, c1 in zip(cut, cut[1:]):
            a0, a1 = int(inp["cfg_ptr"][c0]), int(inp["cfg_ptr"][c1])
            rows = lambda v: torch.cat([v[c0:c1], v[nc + 3 * a0:nc + 3 * a1]])  # noqa: E731
            s["groups"].append((atoms.configs(c0, c1), rows(inp["y"]), rows(inp["sigma"])))
        s["T"] = gap.fold_buffer(M, max(a.n_rows for a, _, _ in s["groups"]))
        s["S"] = [torch.empty(a.n_atoms, -(-M // 4) * 4, dtype=torch.float64, device=DEV)
                  for a, _, _ in s["groups"]]
    elif case["kind"] == "model":
        s["k2"] = gapx.SE2b(inp["x2b"], DELTA, THETA, R_CUT, CUT_WIDTH)
        Mt = M + M_2B
        s["rows"] = inp["y"].numel()
        s["T"] = gap.fold_buffer(Mt, s["rows"])
    return s


# -------------------------------------------------------------------- pass ----
def run(s):
    case, gap = s["case"], s["gap"]
    kind, M = case["kind"], case["M"]
    if kind == "predict":
        return gap.predict(s["atoms"], s["sparse"], s["c"], case["prec"], forces=True)
    if kind == "screen":
        out = gap.predict(s["atoms"], s["sparse"], s["c"], case["prec"], forces=True)
        out["var"] = gap.predict_variance(s["atoms"], s["sparse"], s["Kmm"], JITTER, s["R"])
        return out
    if kind == "train":
        e = gapx.gap_energy(s["desc"], s["X"], s["c"], ZETA, DELTA, case["prec"])
        grads = torch.autograd.grad(e, (s["desc"], s["X"], s["c"]), s["g_e"])
        return {"e": e.detach(), "d_desc": grads[0], "d_X": grads[1], "d_c": grads[2]}
    if kind == "fit":
        a, sp, mixed = s["atoms"], s["sparse"], case["prec"] == "bf16x3"
        gap.build_kmm(sp, out=s["Kmm"])
        gap.build_knm(a, sp, case["prec"], out=s["A"])
        c, _ = gap.fit(s["A"], a.n_rows, s["Kmm"], s["y"], s["sigma"], JITTER, sp,
                       a if mixed else None, REFINE if mixed else 0)
        return {"c": c, "Kmm": s["Kmm"]}
    if kind == "stream":
        return _stream(s, gap, M, case["prec"])
    return _model(s, gap, M)


def _stream(s, gap, M, prec):
    """Configuration groups folded into one factor, then FP64 refinement by groups."""
    sp, T, Kmm = s["sparse"], s["T"], s["Kmm"]
    gap.build_kmm(sp, out=Kmm)
    gap.fold_init(T, M, Kmm, JITTER)
    for a, y, sig in s["groups"]:
        gap.build_knm_block(a, sp, T, prec)
        gap.fold_rows(T, M, a.n_rows, y, sig)
    c, _, _ = gap.fold_solve(T, M)
    for (a, _, _), S in zip(s["groups"], s["S"]):
        gap.refine_weights(a, sp, out=S)
    for _ in range(STREAM_STEPS):
        g = torch.zeros(M, dtype=torch.float64, device=DEV)
        for (a, y, sig), S in zip(s["groups"], s["S"]):
            gap.refine_rows_s(a, sp, S, c, y, sig, g)
        gap.refine_solve(T, M, Kmm, JITTER, g, c)
    return {"c": c}


def _model(s, gap, M):
    """Sparse points by CUR, then one fold of all rows of both descriptors."""
    a, k2, D, T = s["atoms"], s["k2"], s["case"]["D"], s["T"]
    idx, lev = gap.select_cur(a, M)
    sp = gapx.Sparse(a.desc[idx.long()].double(), D, ZETA, DELTA)
    Mt, n = M + M_2B, a.n_rows
    Kmm = torch.zeros(Mt, Mt, dtype=torch.float64, device=DEV)
    Kmm[:M, :M] = gap.build_kmm(sp)
    gap.build_kmm_2b(k2, out=Kmm, row0=M, col0=M)
    gap.fold_init(T, Mt, Kmm, JITTER)
    T[M:Mt, Mt + 1 + n:] = 0  # virial and local rows carry no two-body share
    gap.build_knm_block(a, sp, T, M=Mt)
    gap.build_2b_block(a, k2, s["pair_r"], T, Mt, M)
    gap.build_virial_rows(a, sp, s["pair_r"], out=T, row0=Mt + 1 + n)
    gap.build_local_rows(a, sp, s["local"], out=T, row0=Mt + 1 + n + 9 * a.n_cfg)
    gap.fold_rows(T, Mt, s["rows"], s["y"], s["sigma"])
    c, resid, _ = gap.fold_solve(T, Mt)
    out = gap.predict(a, sp, c[:M].clone(), e_cfg=True, e_atom=False, forces=True)
    two = gap.predict_2b(a, k2, s["pair_r"], c[M:].clone())
    return {"sparse": idx, "leverage": lev, "c": c, "e_cfg": out["e_cfg"] + two["e_cfg"],
            "forces": out["forces"] + two["forces"], "resid": resid}


# ------------------------------------------------------------ work and exact ----
def work(case):
    counts = _counts(case)
    N, D, M = int(counts.sum()), case["D"], case["M"]
    w = 4 if case["dt"] == "f32" else 8
    P = int(_pair_counts(case, N).sum()) if case["nb"] else 0
    R = case["n_cfg"] + 3 * N
    jac, desc, spx = 3.0 * P * D * w, float(N) * D * w, 8.0 * M * D
    dot = 2.0 * N * M * D
    kind = case["kind"]
    if kind in ("predict", "screen"):
        b = desc + spx + jac + 8.0 * (4 * N + case["n_cfg"] + M) + 4.0 * P
        f = 2 * dot + 6.0 * P * D
        if kind == "screen":
            b += 8.0 * (1.5 * M * M + N)
            f += 2.0 * N * M * M + M ** 3
        return {"bytes": b, "flops": f}
    if kind == "train":
        return {"bytes": 2 * desc + 2 * spx + 8.0 * (2 * N + 2 * M), "flops": 4 * dot}
    rows = dot + 6.0 * P * D * M + float(M) * M * D
    if kind in ("fit", "stream"):
        qr = 2.0 * M * M * (R + M - M / 3.0) + M ** 3 / 3.0
        steps = 0 if case["prec"] == "fp64" else 2
        return {"bytes": (1 + steps) * jac + desc + spx + 24.0 * R,
                "flops": rows + qr + steps * (2 * dot + 12.0 * P * D) + (dot if steps else 0.0)}
    Mt = M + M_2B
    R = R + 9 * case["n_cfg"] + (N + 2) // 3
    return {"bytes": jac + desc + spx + 16.0 * R + 24.0 * P,
            "flops": rows + 6.0 * P * D * M + 2.0 * Mt * Mt * (R + Mt) + 4.0 * N * D * D + 2 * dot}


def _k(d, X):
    return DELTA ** 2 * (d @ X.T) ** ZETA


def _energies(d, X, c):
    """Local energies and their descriptor gradients."""
    p = d @ X.T
    q = p ** (ZETA - 1)
    return DELTA ** 2 * ((q * p) @ c), DELTA ** 2 * ZETA * ((q * c) @ X)


def _per_cfg(inp, v):
    cnt = inp["cfg_ptr"].diff()
    cfg = torch.repeat_interleave(torch.arange(cnt.numel(), device=DEV), cnt)
    return torch.zeros(cnt.numel(), dtype=v.dtype, device=DEV).index_add_(0, cfg, v)


def _forces(inp, g, D, chunk=1 << 17):
    F = torch.zeros(inp["n"], 3, dtype=torch.float64, device=DEV)
    for p in range(0, inp["src"].numel(), chunk):
        J = inp["jac"][p:p + chunk, :, :D].double()
        F.index_add_(0, inp["pair_j"][p:p + chunk].long(),
                     -(J * g[inp["src"][p:p + chunk]][:, None, :]).sum(-1))
    return F


def _rows(inp, X, D, virial=False):
    """[energy rows; force rows] and, with virial, the virial rows."""
    d = inp["desc"].double()
    p = d @ X.T
    S = DELTA ** 2 * ZETA * p ** (ZETA - 1)
    nc, N, M = inp["cfg_ptr"].numel() - 1, inp["n"], X.shape[0]
    K = torch.zeros(nc + 3 * N, M, dtype=torch.float64, device=DEV)
    cnt = inp["cfg_ptr"].diff()
    K[:nc].index_add_(0, torch.repeat_interleave(torch.arange(nc, device=DEV), cnt), S * p / ZETA)
    KF = K[nc:].view(N, 3, M)
    KV = torch.zeros(nc, 9, M, dtype=torch.float64, device=DEV) if virial else None
    chunk = max(1, (1 << 27) // (3 * M))
    for q in range(0, inp["src"].numel(), chunk):
        G = inp["jac"][q:q + chunk, :, :D].reshape(-1, D).double() @ X.T
        G = -G.view(-1, 3, M) * S[inp["src"][q:q + chunk]][:, None, :]
        KF.index_add_(0, inp["pair_j"][q:q + chunk].long(), G)
        if virial:
            V = (inp["pair_r"][q:q + chunk][:, :, None, None] * G[:, None]).reshape(-1, 9, M)
            KV.index_add_(0, inp["cfg_of_pair"][q:q + chunk], V)
    return (K, KV.reshape(-1, M)) if virial else K


def _lstsq(K, Kmm, y, sigma):
    """min || [K / sigma; U] c - [y / sigma; 0] ||, by the normal equations, their
    error removed by refinement with the residual b - A c; c and the residual norm."""
    A = torch.cat([K / sigma[:, None],
                   torch.linalg.cholesky(Kmm + JITTER * torch.eye(len(Kmm), dtype=K.dtype, device=DEV)).T])
    b = torch.cat([y / sigma, torch.zeros(len(Kmm), dtype=K.dtype, device=DEV)])
    L = torch.linalg.cholesky(A.T @ A)
    c = torch.zeros(len(Kmm), dtype=K.dtype, device=DEV)
    for _ in range(4):
        c = c + torch.cholesky_solve((A.T @ (b - A @ c))[:, None], L)[:, 0]
    return c, float((b - A @ c).norm())


def _f_cut(r):
    s = torch.clamp((r - (R_CUT - CUT_WIDTH)) / CUT_WIDTH, 0.0, 1.0) * torch.pi
    f = 0.5 * (1 + torch.cos(s)) * (r < R_CUT)
    df = torch.where((s > 0) & (r < R_CUT), -0.5 * torch.pi / CUT_WIDTH * torch.sin(s), torch.zeros_like(s))
    return f, df


def _rows_2b(inp):
    x, r = inp["x2b"], inp["pair_r"].norm(dim=1)
    f, df = _f_cut(r)
    fx = _f_cut(x)[0]
    u = r[:, None] - x
    ker = DELTA ** 2 * fx * torch.exp(-u * u / (2 * THETA ** 2))
    nc, N = inp["cfg_ptr"].numel() - 1, inp["n"]
    K = torch.zeros(nc + 3 * N, x.numel(), dtype=torch.float64, device=DEV)
    K[:nc].index_add_(0, inp["cfg_of_pair"], 0.5 * f[:, None] * ker)
    dk = 0.5 * (df[:, None] - f[:, None] * u / THETA ** 2) * ker
    G = (inp["pair_r"] / r[:, None])[:, :, None] * dk[:, None, :]
    KF = K[nc:].view(N, 3, -1)
    KF.index_add_(0, inp["pair_j"].long(), -G)
    KF.index_add_(0, inp["src"], G)
    return K


def _kmm_2b(inp):
    x = inp["x2b"]
    fx = _f_cut(x)[0]
    return DELTA ** 2 * fx[:, None] * fx * torch.exp(-(x[:, None] - x) ** 2 / (2 * THETA ** 2))


def exact(case, seed):
    inp = _inputs(case, seed)
    D, M, X = case["D"], case["M"], inp["X"]
    d = inp["desc"].double()
    kind = case["kind"]
    if kind in ("predict", "screen"):
        e, g = _energies(d, X, inp["c"])
        out = {"e_atom": e, "e_cfg": _per_cfg(inp, e), "forces": _forces(inp, g, D)}
        if kind == "screen":
            k = _k(d, X)
            eye = torch.eye(M, dtype=torch.float64, device=DEV)
            L = torch.linalg.cholesky(inp["Kmm"] + JITTER * eye)
            q = torch.linalg.solve_triangular(L, k.T, upper=False)
            t = torch.linalg.solve_triangular(inp["R"], k.T, upper=False)
            out["var"] = DELTA ** 2 * (d * d).sum(1) ** ZETA - (q * q).sum(0) + (t * t).sum(0)
        return out
    if kind == "train":
        p = d @ X.T
        q = p ** (ZETA - 1)
        W = DELTA ** 2 * ZETA * inp["g_e"][:, None] * q * inp["c"]
        return {"e": DELTA ** 2 * ((q * p) @ inp["c"]), "d_desc": W @ X, "d_X": W.T @ d,
                "d_c": DELTA ** 2 * ((q * p).T @ inp["g_e"])}
    if kind in ("fit", "stream"):
        Kmm = _k(X, X)
        c, _ = _lstsq(_rows(inp, X, D), Kmm, inp["y"], inp["sigma"])
        return {"c": c, "Kmm": Kmm} if kind == "fit" else {"c": c}
    L = torch.linalg.cholesky(d.T @ d)
    lev = torch.linalg.solve_triangular(L, d.T, upper=False).square().sum(0)
    idx = torch.sort(lev, descending=True, stable=True).indices[:M]
    X = d[idx]
    K, KV = _rows(inp, X, D, virial=True)
    K2 = _rows_2b(inp)
    top = torch.cat([K, KV, _k(d, X)[inp["local"].long()]])
    right = torch.zeros(top.shape[0], M_2B, dtype=torch.float64, device=DEV)
    right[:K2.shape[0]] = K2
    c, resid = _lstsq(torch.cat([top, right], 1), torch.block_diag(_k(X, X), _kmm_2b(inp)),
                      inp["y"], inp["sigma"])
    e, g = _energies(d, X, c[:M])
    pred2 = K2 @ c[M:]
    nc = case["n_cfg"]
    return {"sparse": None, "leverage": lev, "c": c, "e_cfg": _per_cfg(inp, e) + pred2[:nc],
            "forces": _forces(inp, g, D) + pred2[nc:].view(-1, 3), "resid": resid}
