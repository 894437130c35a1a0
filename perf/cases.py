"""Performance cases of the LSQR library: what a user's program has it do.

A case is one call, or one short sequence of calls, on a seeded synthetic
system of the paper's row structure: observations grouped by star, 5
astrometric coefficients per row, 3 axes x 4 attitude columns from one random
start, 6 distinct instrumental columns, 1 global column (or a subset of these
sections). The sizes are those of the repository's workloads and tests, and
odd sizes between them.

Kinds of case ("call"):
  solve            lsqr_solve, b -> x (and the variance of x when asked for)
  refined          lsqr_solve_refined on FP32 values
  batched          lsqr_solve_batched, k noise realisations of b
  batched_refined  lsqr_solve_batched_refined on FP32 values
  gradient         r = A x - b, g = A^T r: the operators lsqr_aprod1 and
                   lsqr_aprod2 (their FP32 forms when vec is "f32"), as a
                   caller's own solver or residual check uses them
"""
import math

import torch

from paper_2308_00778_amd import LsqrSystem

DEVICE = "cuda:0"
NOISE = 1e-6  # standard deviation of the noise of b
ROW_CHUNK = 1 << 23

FULL = {"n_astro": 5, "n_axes": 3, "n_instr": 6, "n_glob": 1}


def _case(call, stars, obs, n_dfa, n_instr_cols, **kw):
    c = {"call": call, "stars": stars, "obs_lo": obs[0], "obs_hi": obs[1], "n_dfa": n_dfa,
         "n_instr_cols": n_instr_cols, "values": "f64", **FULL, "k": 1, "limit": 200,
         "tol": 1e-12, "variance": False, "constraints": 0, "astro_scale": 0.0, "vec": "f64"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: both operators on a system of a few thousand rows
        # (the smoke test's), where launches are the cost
        dict(_case("gradient", 64, (40, 90), 60, 30), name="gradient_4e3"),
        # the parity-sized workload, solved to convergence
        dict(_case("solve", 1000, (100, 100), 1000, 120), name="solve_1e5"),
        # ragged stars, odd sizes, the variance of the unknowns asked for (a
        # production run's last step); a fixed number of iterations
        dict(_case("solve", 12347, (50, 150), 10007, 1013, variance=True, limit=30),
             name="solve_1e6_variance"),
        # constraint equations below the observations
        dict(_case("solve", 10001, (60, 140), 5003, 601, constraints=300),
             name="solve_1e6_constraints"),
        # a subset of the sections: no global parameter
        dict(_case("solve", 30011, (70, 130), 20011, 2003, n_glob=0), name="solve_3e6_no_global"),
        # other section sizes: 3 astrometric, 2 instrumental, 3 global
        dict(_case("solve", 10007, (80, 120), 5009, 499, n_astro=3, n_instr=2, n_glob=3,
                   limit=25), name="solve_1e6_mixed"),
        # the single-GPU production share, 20 iterations (the benchmark's run)
        dict(_case("solve", 1000000, (100, 100), 100000, 6000, limit=20), name="solve_1e8"),
        # FP32 values, FP32 inner iterations, FP64 refinement: a quarter of the
        # rows of the mixed-precision workload at its attitude and instrumental
        # sizes, astrometric columns scaled by 10^U(-2, 2)
        dict(_case("refined", 1000000, (100, 100), 400000, 12000, values="f32", tol=1e-6,
                   astro_scale=2.0), name="refined_1e8"),
        # Monte Carlo error propagation: 16 noise realisations of b, a tenth of
        # the batched workload's rows at its attitude and instrumental sizes
        dict(_case("batched", 100000, (100, 100), 100000, 6000, k=16), name="batched_1e7_k16"),
        # the largest workload's form at a fiftieth of its rows: FP32 values,
        # ragged stars, 30,000 instrumental columns, 4 right-hand sides
        dict(_case("batched_refined", 200000, (50, 150), 200000, 30000, values="f32", k=4,
                   tol=1e-6), name="batched_refined_2e7_k4"),
        # the operators for a caller's own solver, ragged stars
        dict(_case("gradient", 150001, (50, 150), 100003, 6007), name="gradient_1.5e7"),
        # the same in FP32
        dict(_case("gradient", 50021, (50, 150), 50021, 3001, values="f32", vec="f32"),
             name="gradient_5e6_f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["solve", "solve", "solve", "refined", "batched", "batched_refined",
                       "gradient", "gradient"])
    top = {"solve": 300000, "refined": 300000, "batched": 60000, "batched_refined": 100000,
           "gradient": 500000}[call]
    stars = _log_int(rng, 100, top)
    obs = rng.choice([(100, 100), (50, 150), (30, 90), (75, 130)])
    rows = stars * (obs[0] + obs[1]) // 2
    # the attitude axis has at most a column per 50 rows and axis, the
    # instrumental section one per 200
    n_dfa = _log_int(rng, 20, max(21, min(400000, rows // 50)))
    n_instr_cols = _log_int(rng, 12, max(13, min(30000, rows // 200)))
    kw = {}
    if call == "solve":
        kw["limit"] = rng.choice([20, 30, 200])
        kw["variance"] = kw["limit"] < 200 and rng.random() < 0.3
        kw["values"] = rng.choice(["f64", "f64", "f64", "f32"])
        part = rng.random()
        if part < 0.25:
            kw.update(rng.choice([{"n_glob": 0}, {"n_astro": 3, "n_instr": 2, "n_glob": 3},
                                  {"n_axes": 0, "n_glob": 5}, {"n_astro": 4, "n_instr": 5},
                                  {"n_astro": 5, "n_instr": 0, "n_glob": 0}]))
        elif part < 0.4:
            kw["constraints"] = _log_int(rng, 5, 500)
    elif call == "refined":
        kw.update(values="f32", tol=1e-6, astro_scale=rng.choice([0.0, 2.0]))
    elif call == "batched":
        kw["k"] = rng.choice([2, 4, 5, 8, 16])
    elif call == "batched_refined":
        kw.update(values="f32", tol=1e-6, k=rng.choice([2, 4]))
    else:
        kw["values"] = rng.choice(["f64", "f64", "f32"])
        if kw["values"] == "f32":
            kw["vec"] = rng.choice(["f64", "f32"])
    return _case(call, stars, obs, n_dfa, n_instr_cols, **kw)


# ------------------------------------------------------------------- inputs
def _sizes(case):
    na, nx, ni, ng = case["n_astro"], case["n_axes"], case["n_instr"], case["n_glob"]
    att0 = na * case["stars"]
    ins0 = att0 + nx * case["n_dfa"]
    glob0 = ins0 + case["n_instr_cols"]
    return na, 4 * nx, ni, ng, att0, ins0, glob0, glob0 + ng


def _system(case, seed):
    """The matrix of a case on the GPU (values, index arrays, constraint rows)."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(1000003 * int(seed) + 17)
    na, natt, ni, ng, _, _, _, n = _sizes(case)
    stars = case["stars"]
    # observations per star: a property of the case, so that every seed's row
    # vectors have one length
    shape = torch.Generator(device=DEVICE)
    shape.manual_seed(20230801 + stars)
    counts = torch.randint(case["obs_lo"], case["obs_hi"] + 1, (stars,), device=DEVICE,
                           generator=shape)
    star = torch.repeat_interleave(torch.arange(stars, device=DEVICE), counts)
    m = star.numel()
    vdt = torch.float64 if case["values"] == "f64" else torch.float32
    values = torch.empty((na + natt + ni + ng, m), dtype=vdt, device=DEVICE)
    for c in range(values.shape[0]):
        torch.randn(m, generator=gen, device=DEVICE, dtype=vdt, out=values[c])
    if case["astro_scale"] > 0.0:  # astrometric columns of different scales
        e = case["astro_scale"] * (2.0 * torch.rand((na, stars), generator=gen, device=DEVICE)
                                   - 1.0)
        for j in range(na):
            values[j] *= torch.repeat_interleave((10.0 ** e[j]).to(vdt), counts)
    att = torch.randint(0, max(1, case["n_dfa"] - 3), (m,), device=DEVICE, generator=gen)
    # six distinct ascending columns: sorted draws from [0, n - 5), plus 0..5
    draws = [torch.randint(0, case["n_instr_cols"] - max(0, ni - 1), (m,), device=DEVICE,
                           generator=gen, dtype=torch.int32) for _ in range(ni)]
    for hi in range(ni - 1, 0, -1):
        for j in range(hi):
            a, b = draws[j], draws[j + 1]
            draws[j], draws[j + 1] = torch.minimum(a, b), torch.maximum(a, b)
    instr = torch.empty((ni, m), dtype=torch.int32, device=DEVICE)
    for j in range(ni):
        torch.add(draws[j], j, out=instr[j])
    del draws
    s = {"values": values, "star": star, "att": att, "instr": instr, "m": m, "n": n,
         "counts": counts, "con": None}
    if case["constraints"] > 0:  # long sparse rows, weighed like an observation
        nc = case["constraints"]
        lens = torch.randint(50, 501, (nc,), device=DEVICE, generator=gen).clamp(max=n)
        rowptr = torch.zeros(nc + 1, dtype=torch.int64, device=DEVICE)
        torch.cumsum(lens, 0, out=rowptr[1:])
        nnz = int(rowptr[-1])
        row = torch.repeat_interleave(torch.arange(nc, device=DEVICE), lens)
        # distinct columns of a row: a random start and equal steps
        start = torch.randint(0, n, (nc,), device=DEVICE, generator=gen)
        k = torch.arange(nnz, device=DEVICE) - rowptr[row]
        col = (start[row] + k * (n // lens)[row]) % n
        val = torch.randn(nnz, generator=gen, device=DEVICE, dtype=torch.float64)
        val *= math.sqrt(values.shape[0]) / torch.sqrt(lens.double())[row]
        s["con"] = {"rowptr": rowptr, "col": col, "val": val, "row": row, "n": nc}
    s["gen"] = gen
    return s


def _columns(case, s, lo, hi):
    """(columns, coefficient) of rows [lo, hi), one pair per coefficient."""
    na, natt, ni, ng, att0, ins0, glob0, _ = _sizes(case)
    star, att = s["star"][lo:hi], s["att"][lo:hi]
    c = 0
    for j in range(na):
        yield na * star + j, s["values"][c, lo:hi]
        c += 1
    for a in range(case["n_axes"]):
        for q in range(4):
            yield att0 + a * case["n_dfa"] + q + att, s["values"][c, lo:hi]
            c += 1
    for j in range(ni):
        yield ins0 + s["instr"][j, lo:hi].long(), s["values"][c, lo:hi]
        c += 1
    for g in range(ng):
        yield glob0 + g, s["values"][c, lo:hi]
        c += 1


def _apply(case, s, x):
    """A x in 64 bits (x: [n])."""
    y = torch.zeros(s["m"] + (s["con"]["n"] if s["con"] else 0), dtype=torch.float64,
                    device=DEVICE)
    for lo in range(0, s["m"], ROW_CHUNK):
        hi = min(s["m"], lo + ROW_CHUNK)
        for col, a in _columns(case, s, lo, hi):
            y[lo:hi] += a.double() * x[col]
    if s["con"]:
        con = s["con"]
        y[s["m"]:].index_add_(0, con["row"], con["val"] * x[con["col"]])
    return y


def _apply_t(case, s, y, square=False):
    """A^T y in 64 bits (square: the sums of squared coefficients)."""
    na, natt, ni, _, att0, ins0, glob0, n = _sizes(case)
    x = torch.zeros(n, dtype=torch.float64, device=DEVICE)
    # (first column, columns) of the section of each coefficient; a section is
    # summed in `copies` parts, so that few columns do not share one address
    sections = [(0, att0)] * na + [(att0, ins0 - att0)] * natt + [(ins0, glob0 - ins0)] * ni
    for lo in range(0, s["m"], ROW_CHUNK):
        hi = min(s["m"], lo + ROW_CHUNK)
        i = torch.arange(hi - lo, device=DEVICE)
        for c, (col, a) in enumerate(_columns(case, s, lo, hi)):
            v = a.double() * (a.double() if square else y[lo:hi])
            if isinstance(col, int):
                x[col] += v.sum()
                continue
            first, width = sections[c]
            copies = max(1, min(1024, (1 << 22) // width))
            part = torch.zeros(width * copies, dtype=torch.float64, device=DEVICE)
            part.index_add_(0, (col - first) * copies + i % copies, v)
            x[first:first + width] += part.view(width, copies).sum(1)
    if s["con"]:
        con = s["con"]
        v = con["val"] * (con["val"] if square else y[s["m"]:][con["row"]])
        x.index_add_(0, con["col"], v)
    return x


def _rhs(case, s):
    """k right-hand sides A x_true + noise, [rows, k]."""
    xt = torch.randn(s["n"], generator=s["gen"], device=DEVICE, dtype=torch.float64)
    b = _apply(case, s, xt)
    if case["k"] == 1:
        b += NOISE * torch.randn(b.numel(), generator=s["gen"], device=DEVICE,
                                 dtype=torch.float64)
        return b
    B = torch.empty((b.numel(), case["k"]), dtype=torch.float64, device=DEVICE)
    for j in range(case["k"]):
        B[:, j] = b + NOISE * torch.randn(b.numel(), generator=s["gen"], device=DEVICE,
                                          dtype=torch.float64)
    return B


def _inputs(case, seed):
    s = _system(case, seed)
    if case["call"] == "gradient":
        vdt = torch.float64 if case["vec"] == "f64" else torch.float32
        s["x"] = torch.randn(s["n"], generator=s["gen"], device=DEVICE, dtype=vdt)
        s["b"] = torch.randn(s["m"], generator=s["gen"], device=DEVICE, dtype=vdt)
    else:
        s["b"] = _rhs(case, s)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    con = s["con"] or {}
    h = LsqrSystem(s["values"], s["star"], s["att"], s["instr"], n_stars=case["stars"],
                   n_dfa=case["n_dfa"], n_instr_cols=case["n_instr_cols"],
                   n_astro=case["n_astro"], n_axes=case["n_axes"], n_instr=case["n_instr"],
                   n_glob=case["n_glob"], con_rowptr=con.get("rowptr"), con_col=con.get("col"),
                   con_val=con.get("val"))
    if case["variance"]:
        h.set_option("variance", 1)
    if case["call"] == "batched":
        h.set_option("att_rhs", 4)
    state = {"case": case, "handle": h, "b": s["b"]}
    if case["call"] == "gradient":
        state.update(x=s["x"], r=torch.empty_like(s["b"]), g=torch.empty_like(s["x"]))
    return state


def run(state):
    case, h = state["case"], state["handle"]
    call = case["call"]
    if call == "solve":
        x, _ = h.solve(state["b"], case["limit"], case["tol"], case["tol"])
        return {"x": x, "var": h.variance()} if case["variance"] else {"x": x}
    if call == "refined":
        return {"x": h.solve_refined(state["b"], case["limit"], case["tol"], case["tol"])[0]}
    if call == "batched":
        return {"x": h.solve_batched(state["b"], case["limit"], case["tol"], case["tol"])[0]}
    if call == "batched_refined":
        return {"x": h.solve_batched_refined(state["b"], case["limit"], case["tol"],
                                             case["tol"])[0]}
    r, g = state["r"], state["g"]
    torch.neg(state["b"], out=r)
    g.zero_()
    if case["vec"] == "f64":
        h.aprod1(state["x"], r)
        h.aprod2(g, r)
    else:
        h.aprod1_f32(state["x"], r)
        h.aprod2_f32(g, r)
    return {"r": r, "g": g}


# Iterations a solve to convergence takes on these systems (the scaled matrix
# has a condition number of 3 to 5 whatever its size), and the inner
# iterations of a refined solve
SOLVE_ITERATIONS, REFINED_ITERATIONS = 36, 42


def work(case):
    """Each LSQR iteration has to read the matrix (values and indices) once for
    A v and, as every entry of A^T u needs the whole of u first, read and
    write the row vector; k right-hand sides share the reads of the matrix."""
    m = case["stars"] * (case["obs_lo"] + case["obs_hi"]) / 2
    na, natt, ni, ng, _, _, _, n = _sizes(case)
    vb = 8 if case["values"] == "f64" else 4
    row = (na + natt + ni + ng) * vb + 8 * (na > 0) + 8 * (natt > 0) + 4 * ni
    flops = 4.0 * m * (na + natt + ni + ng)
    if case["call"] == "gradient":
        ub = 8 if case["vec"] == "f64" else 4
        return {"bytes": m * (row + 2 * ub) + 3 * n * ub, "flops": flops}
    refined = case["call"] in ("refined", "batched_refined")
    itn = REFINED_ITERATIONS if refined else min(case["limit"], SOLVE_ITERATIONS)
    ub, k = (4 if refined else 8), case["k"]
    # column vectors per iteration: v, w, y read and written
    return {"bytes": itn * (m * (row + 2 * ub * k) + 48 * n * k), "flops": itn * k * flops}


# ------------------------------------------------------- the same in 64 bits
def _lsqr(case, s, b, limit):
    """Paige and Saunders' LSQR on the column-scaled system, plain torch in 64
    bits: the iterate after `limit` iterations, or where ||A^T r|| no longer
    matters, and the sums of (w / rho)^2, both unscaled."""
    ssq = _apply_t(case, s, None, square=True)
    p = torch.where(ssq > 0, 1.0 / torch.sqrt(ssq.clamp(min=1e-300)), torch.ones_like(ssq))
    u = b.clone()
    beta = float(u.norm())
    u /= beta
    v = p * _apply_t(case, s, u)
    alpha = float(v.norm())
    v /= alpha
    w, y, var = v.clone(), torch.zeros_like(v), torch.zeros_like(v)
    phibar, rhobar, start = beta, alpha, alpha * beta
    for _ in range(limit):
        u = _apply(case, s, p * v) - alpha * u
        beta = float(u.norm())
        u /= beta
        v = p * _apply_t(case, s, u) - beta * v
        alpha = float(v.norm())
        v /= alpha
        rho = math.hypot(rhobar, beta)
        c, sn = rhobar / rho, beta / rho
        theta, rhobar = sn * alpha, -c * alpha
        phi, phibar = c * phibar, sn * phibar
        var += (w / rho) ** 2
        y += (phi / rho) * w
        w = v - (theta / rho) * w
        if alpha * abs(c) * phibar <= 1e-15 * start:
            break
    return p * y, p * p * var


def exact(case, seed):
    m = case["stars"] * (case["obs_lo"] + case["obs_hi"]) / 2
    limit = case["limit"] if case["call"] == "solve" else 200
    passes = 1 if case["call"] == "gradient" else 2 * min(limit, 40) * case["k"]
    if m * passes > 1.5e10:  # over about 20 seconds
        return None
    s = _inputs(case, seed)
    if case["call"] == "gradient":
        x, b = s["x"].double(), s["b"].double()
        r = _apply(case, s, x) - b
        return {"r": r, "g": _apply_t(case, s, r)}
    if case["k"] == 1:
        x, var = _lsqr(case, s, s["b"], limit)
        return {"x": x, "var": var} if case["variance"] else {"x": x}
    return {"x": torch.stack([_lsqr(case, s, s["b"][:, j].contiguous(), limit)[0]
                              for j in range(case["k"])], dim=1)}
