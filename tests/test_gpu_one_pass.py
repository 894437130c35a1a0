"""GPU parity of the one-pass row form (attitude and instrumental histograms
both in LDS, one sweep over A): Eq. (3) element by element and fixed-iteration
solves against the oracle, at the edges of its LDS plan, where it gives way to
the bucket order, and on general layouts. Tolerances as in the full-layout
parity tests: c eps sum |terms| for the operator, 1e-10 for the iterates.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps

# 19,456 FP64 columns fit in the histograms (3 n_dfa + n_instr_cols)
SPECS = {
    # everything of the vector in LDS too; fewer rows than one wave
    "tiny": dict(n_stars=2, obs=(10, 20), n_dfa=5, n_instr_cols=7),
    "small": dict(n_stars=400, obs=(10, 70), n_dfa=60, n_instr_cols=30),
    # the vector's instrumental slice beside the histograms, not its attitude
    "instr_slice": dict(n_stars=400, obs=(40, 90), n_dfa=3500, n_instr_cols=500),
    # neither
    "no_slice": dict(n_stars=400, obs=(40, 90), n_dfa=3000, n_instr_cols=10000),
    # exactly full, and one attitude start more (bucket order, two buckets)
    "full": dict(n_stars=400, obs=(40, 90), n_dfa=6000, n_instr_cols=1456),
    "past_full": dict(n_stars=400, obs=(40, 90), n_dfa=6499, n_instr_cols=1456),
    "no_slice_f32": dict(n_stars=400, obs=(40, 90), n_dfa=3000, n_instr_cols=10000,
                         value_dtype="f32"),
    "small_f32": dict(n_stars=400, obs=(10, 70), n_dfa=60, n_instr_cols=30, value_dtype="f32"),
    # general layouts: no attitude, no global, several globals, one section
    "no_att": dict(n_stars=300, obs=(10, 70), n_axes=0, n_glob=5),
    "no_glob": dict(n_stars=300, obs=(10, 70), n_dfa=120, n_instr_cols=23, n_glob=0),
    "mixed": dict(n_stars=300, obs=(10, 70), n_dfa=120, n_instr_cols=23, n_astro=3, n_instr=2,
                  n_glob=3),
    "mixed_f32": dict(n_stars=300, obs=(10, 70), n_dfa=120, n_instr_cols=23, n_astro=4, n_instr=5,
                      n_glob=1, value_dtype="f32"),
    "astro_only": dict(n_stars=300, obs=(10, 70), n_axes=0, n_instr=0, n_glob=0),
    "att_only": dict(n_stars=300, obs=(10, 70), n_dfa=4000, n_astro=0, n_instr=0, n_glob=0),
    # general layout in bucket order (four buckets)
    "no_glob_buckets": dict(n_stars=900, obs=(60, 90), n_dfa=20011, n_instr_cols=203, n_glob=0),
    "mixed_buckets": dict(n_stars=900, obs=(60, 90), n_dfa=7001, n_instr_cols=203, n_astro=3,
                          n_instr=2, n_glob=3),
}

_SYS = {}


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def system(name):
    if name not in _SYS:
        S = synth.make_system(synth.tiny(seed=81 + list(SPECS).index(name), **SPECS[name]))
        _SYS[name] = (S, oracle.OracleSystem.from_synth(S))
    return _SYS[name]


def abs_system(S):
    sp = S.spec
    return oracle.OracleSystem(np.abs(S.values.astype(np.float64)), S.star_of_row, S.att_start,
                               S.instr_idx, n_stars=sp.n_stars, n_dfa=sp.n_dfa,
                               n_instr_cols=sp.n_instr_cols, n_astro=sp.n_astro,
                               n_axes=sp.n_axes, n_par_axis=sp.n_par_axis, n_instr=sp.n_instr,
                               n_glob=sp.n_glob)


def gpu_system(S):
    from paper_2308_00778_amd import LsqrSystem

    return LsqrSystem.from_host(S, "cuda:0")


def rel_inf(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("name", list(SPECS))
def test_one_pass_operators(torch_cuda, name):
    torch = torch_cuda
    S, o = system(name)
    say(f"one-pass operators: {name} m={S.m} n={o.n}")
    rng = np.random.default_rng(16)
    y, x0 = rng.standard_normal(o.m), rng.standard_normal(o.n)
    x, y0 = rng.standard_normal(o.n), rng.standard_normal(o.m)
    ab = abs_system(S)
    g = gpu_system(S)
    yd, xd = torch.from_numpy(y0).cuda(), torch.from_numpy(x0).cuda()
    g.aprod1(torch.from_numpy(x).cuda(), yd)
    g.aprod2(xd, torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    got1, got2 = yd.cpu().numpy(), xd.cpu().numpy()
    g.close()
    c = 2.0 * np.sqrt(S.m) + 32
    assert np.all(np.abs(got1 - o.aprod1(x, y0))
                  <= 32 * EPS * ab.aprod1(np.abs(x), np.abs(y0)) + 1e-300)
    assert np.all(np.abs(got2 - o.aprod2(y, x0))
                  <= c * EPS * ab.aprod2(np.abs(y), np.abs(x0)) + 1e-300)


# 10 iterations: below the unknown count of every system; graph launches of 4
# (an iteration's stopping tests inside the next one, and after the last), and
# single launches
@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("name", list(SPECS))
def test_one_pass_solve(torch_cuda, name, graph):
    torch = torch_cuda
    S, o = system(name)
    itn = 10
    b = o.aprod1(synth.x_true(S.spec), synth.noise(S.spec, S.m))
    x_ref, i_ref = o.lsqr(b, itn, atol=0.0, btol=0.0, conlim=0.0, tests=False)
    say(f"one-pass solve: {name} m={S.m} n={o.n} graph={graph}")
    g = gpu_system(S)
    g.set_option("tests", 0)
    g.set_option("graph", graph)
    g.set_option("chunk", 4)
    bd = torch.from_numpy(b).cuda()
    xs = []
    for _ in range(2):  # a second solve on the handle's state
        x, info = g.solve(bd, itn, atol=0.0, btol=0.0)
        xs.append(x.cpu().numpy())
        assert info.itn == i_ref.itn == itn and info.istop == 7
        for k in ("rnorm", "anorm", "acond", "xnorm", "bnorm"):
            a, r = getattr(info, k), getattr(i_ref, k)
            assert abs(a - r) <= 1e-8 * abs(r), (k, a, r)
    g.close()
    for x in xs:
        assert rel_inf(x, x_ref) <= 1e-10


# A right-hand side that the first iteration solves exactly (one column of ones:
# every quantity is a power of two), so that beta is exactly 0 and the next
# iteration starts from u = 0: the solution stays, in one pass and in bucket
# order.
@pytest.mark.parametrize("buckets", [0, 1])
def test_zero_residual_keeps_solution(torch_cuda, buckets):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    say(f"zero residual: att_buckets={buckets}")
    m = 4
    values = torch.zeros((12, m), dtype=torch.float64, device="cuda")
    values[0] = 1.0
    zero = torch.zeros(m, dtype=torch.int64, device="cuda")
    g = LsqrSystem(values, zero, zero.clone(), torch.zeros((0, m), dtype=torch.int32, device="cuda"),
                   n_stars=1, n_dfa=4, n_instr_cols=0, n_astro=0, n_instr=0, n_glob=0)
    g.set_option("tests", 0)
    if buckets:
        g.set_option("att_buckets", buckets)
    x, info = g.solve(torch.full((m,), 2.0, dtype=torch.float64, device="cuda"), 2, atol=0.0,
                      btol=0.0)
    got = x.cpu().numpy()
    g.close()
    assert info.itn == 2 and info.rnorm == 0.0
    assert got[0] == 2.0 and np.all(got[1:] == 0.0)


# Beyond 32 buckets, from 64 steps of 64 rows a wave (4,194,304 x 4 rows with 256
# CUs), the star-order pass deals its rows in pieces; with 32 buckets it does not.
# The two solves differ in the order of sums only: 1e-10 as against the oracle.
def test_pieces_agree_with_ranges(torch_cuda):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    spec = synth.tiny(seed=23, n_stars=175003, obs=(50, 150), n_dfa=20011, n_instr_cols=203)
    arrays, first = synth.device_system(spec, "cuda:0")
    m = int(first[-1])
    say(f"pieces: m={m}")
    assert m > 64 * 64 * 16 * torch.cuda.get_device_properties(0).multi_processor_count
    b = synth.device_noise(spec, m, 0, "cuda:0")
    xs = []
    for buckets in (33, 62, 32):
        g = LsqrSystem(**arrays, n_stars=spec.n_stars, n_dfa=spec.n_dfa,
                       n_instr_cols=spec.n_instr_cols)
        g.set_option("tests", 0)
        g.set_option("att_buckets", buckets)
        x, info = g.solve(b, 6, atol=0.0, btol=0.0)
        assert info.itn == 6
        xs.append(x.cpu().numpy())
        g.close()
    assert rel_inf(xs[0], xs[2]) <= 1e-10
    assert rel_inf(xs[1], xs[2]) <= 1e-10


# k-tiles of a matrix past the last-level cache's size (nontemporal loads; small
# systems load plain): the solutions of the single solves, to 1e-10 at equal
# iteration counts.
@pytest.mark.parametrize("k", [2, 4])
@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
def test_tiles_past_the_cache(torch_cuda, f32, k):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    # 224 and 128 bytes a row: more than 320 MB
    spec = synth.tiny(seed=29, n_stars=30011 if f32 else 17011, obs=(50, 150), n_dfa=9001,
                      n_instr_cols=203, value_dtype="f32" if f32 else "f64")
    arrays, first = synth.device_system(spec, "cuda:0")
    m = int(first[-1])
    say(f"tiles past the cache: m={m} k={k} f32={f32}")
    assert m * (128 if f32 else 224) > 320 << 20
    g = LsqrSystem(**arrays, n_stars=spec.n_stars, n_dfa=spec.n_dfa,
                   n_instr_cols=spec.n_instr_cols)
    g.set_option("tests", 0)
    g.set_option("ktile", k)
    B = torch.stack([synth.device_noise(spec, m, r, "cuda:0") for r in range(k)], 1).contiguous()
    X, infos = g.solve_batched(B, 6, 0.0, 0.0)
    X = X.cpu().numpy()
    for r in range(k):
        x, info = g.solve(B[:, r].contiguous(), 6, atol=0.0, btol=0.0)
        assert info.itn == 6 and infos[r].itn == 6
        assert rel_inf(X[:, r], x.cpu().numpy()) <= 1e-10
    g.close()


# The instrumental tail with and without the compact copy of the indices: columns
# past one histogram, against the oracle.
@pytest.mark.parametrize("compact", [1, 0])
@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
def test_instr_tail_indices(torch_cuda, f32, compact):
    torch = torch_cuda
    S = synth.make_system(synth.tiny(seed=31, n_stars=300, obs=(10, 70), n_dfa=120,
                                     n_instr_cols=25001, value_dtype="f32" if f32 else "f64"))
    o = oracle.OracleSystem.from_synth(S)
    say(f"instrumental tail: m={S.m} f32={f32} compact={compact}")
    b = np.stack([o.aprod1(synth.x_true(S.spec), synth.noise(S.spec, S.m, r)) for r in range(4)], 1)
    g = gpu_system(S)
    g.set_option("tests", 0)
    g.set_option("compact_index", compact)
    g.set_option("ktile", 4)
    x, _ = g.solve(torch.from_numpy(b[:, 0].copy()).cuda(), 6, atol=0.0, btol=0.0)
    X, _ = g.solve_batched(torch.from_numpy(b).cuda(), 6, 0.0, 0.0)
    x, X = x.cpu().numpy(), X.cpu().numpy()
    g.close()
    for r in range(4):
        want = o.lsqr(b[:, r].copy(), 6, atol=0.0, btol=0.0, conlim=0.0, tests=False)[0]
        assert rel_inf(X[:, r], want) <= 1e-10
        if r == 0:
            assert rel_inf(x, want) <= 1e-10


# Eq. (3) in FP32: the attitude columns are sums of FP64 products in both forms,
# rounded to FP32 once. So each is within half an ulp of the exact sum, and the
# rounding of a sum of that many terms in FP64.
@pytest.mark.parametrize("buckets", [0, 3])
@pytest.mark.parametrize("name", ["small_f32", "no_slice_f32", "mixed_f32"])
def test_f32_attitude_products_in_fp64(torch_cuda, name, buckets):
    torch = torch_cuda
    S, o = system(name)
    sp = S.spec
    say(f"FP64 products of FP32 values: {name} m={S.m} buckets={buckets}")
    y = np.random.default_rng(17).standard_normal(S.m).astype(np.float32)
    yl = y.astype(np.longdouble)
    exact, mag, terms = (np.zeros(3 * sp.n_dfa, dtype=np.longdouble) for _ in range(3))
    for ax in range(3):
        for q in range(4):
            p = S.values[sp.n_astro + 4 * ax + q].astype(np.longdouble) * yl  # 48 of 64 bits
            c = ax * sp.n_dfa + q + S.att_start
            np.add.at(exact, c, p)
            np.add.at(mag, c, np.abs(p))
            np.add.at(terms, c, 1)
    g = gpu_system(S)
    if buckets:
        g.set_option("att_buckets", buckets)
    x = torch.zeros(o.n, dtype=torch.float32, device="cuda")
    g.aprod2_f32(x, torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    a0 = sp.n_astro * sp.n_stars
    got = x.cpu().numpy()[a0:a0 + 3 * sp.n_dfa].astype(np.longdouble)
    g.close()
    bound = 2.0 ** -24 * np.abs(exact) + 2.0 * terms * EPS * mag + 1e-45
    assert np.all(np.abs(got - exact) <= bound)


# LSQR_OPT_ASTRO_SCAN at one-pass sizes: the scan runs (one writer per column, a
# fixed order), so the astrometric columns have the bits they have beside a
# bucket count, which rules the one pass out.
def test_astro_scan_is_honoured(torch_cuda):
    torch = torch_cuda
    S, o = system("small")
    sp = S.spec
    say(f"segmented scan at one-pass sizes: m={S.m}")
    y = np.random.default_rng(19).standard_normal(S.m)
    got = []
    for buckets in (0, 1):
        g = gpu_system(S)
        g.set_option("astro_scan", 1)
        if buckets:
            g.set_option("att_buckets", buckets)
        x = torch.zeros(o.n, dtype=torch.float64, device="cuda")
        g.aprod2(x, torch.from_numpy(y).cuda())
        torch.cuda.synchronize()
        got.append(x.cpu().numpy()[:sp.n_astro * sp.n_stars])
        g.close()
    assert np.array_equal(got[0], got[1])
    want = o.aprod2(y, np.zeros(o.n))[:sp.n_astro * sp.n_stars]
    assert rel_inf(got[0], want) <= 1e-12


# Systems whose histograms fit in LDS but nothing of the vector beside them, with
# the matrix past the last-level cache: the bucket order is quicker for FP64
# vectors (attitude pre-pass: a window of its own in the profile), the sweep for
# the refined solve's FP32 vectors, whose instrumental slice fits. Either way the
# iterates of the other fused mode, to 1e-10, and A^T y adjoint to A x.
@pytest.mark.parametrize("f32", [False, True], ids=["f64", "f32"])
def test_large_systems_without_windows(torch_cuda, f32):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    spec = synth.tiny(seed=37, n_stars=28001 if f32 else 16001, obs=(75, 125), n_dfa=4000,
                      n_instr_cols=4500, value_dtype="f32" if f32 else "f64")
    arrays, first = synth.device_system(spec, "cuda:0")
    m = int(first[-1])
    say(f"no windows: m={m} f32={f32}")
    assert m * (128 if f32 else 224) > 320 << 20
    kw = dict(n_stars=spec.n_stars, n_dfa=spec.n_dfa, n_instr_cols=spec.n_instr_cols)
    b = synth.device_noise(spec, m, 0, "cuda:0")
    xs = []
    for fused in (2, 1):
        g = LsqrSystem(**arrays, **kw)
        g.set_option("tests", 0)
        g.set_option("fused", fused)
        g.set_option("profile", 1)
        x, info = g.solve(b, 6, atol=0.0, btol=0.0)
        assert info.itn == 6
        pre, n = g.pass_times()["pre"]
        say(f"  fused={fused}: pre-pass window {1e3 * pre / n:.1f} us")
        assert (pre / n > 0.015) == (fused == 2)
        xs.append(x.cpu().numpy())
        if f32 and fused == 2:
            xr, _ = g.solve_refined(b, 6, 0.0, 0.0, 1)
            pre, n = g.pass_times()["pre"]
            say(f"  refined: pre-pass window {1e3 * pre / n:.1f} us")
            assert pre / n < 0.015
            assert rel_inf(xr.cpu().numpy(), xs[0]) <= 1e-3  # one FP32 inner solve
        if fused == 2:
            gen = torch.Generator(device="cuda").manual_seed(3)
            u = torch.randn(g.n, generator=gen, device="cuda", dtype=torch.float64)
            w = torch.randn(m, generator=gen, device="cuda", dtype=torch.float64)
            au = g.aprod1(u, torch.zeros(m, dtype=torch.float64, device="cuda"))
            aw = g.aprod2(torch.zeros(g.n, dtype=torch.float64, device="cuda"), w)
            torch.cuda.synchronize()
            lhs, rhs = float(au @ w), float(u @ aw)
            assert abs(lhs - rhs) <= 1e-12 * float(au.norm() * w.norm())
        g.close()
    assert rel_inf(xs[0], xs[1]) <= 1e-10
