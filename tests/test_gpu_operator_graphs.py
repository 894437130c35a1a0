"""The operators recorded in a caller's HIP graph: what a recorded call reads
lives as long as the handle, whatever is done with the handle between the
replays, and every replay gives the result of the eager call. Tolerances as in
the parity tests: c eps sum |terms|.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps

SPECS = {
    # one pass over the rows
    "one_pass": dict(n_stars=400, obs=(10, 70), n_dfa=600, n_instr_cols=130),
    # bucket order, and instrumental columns past one histogram
    "tail": dict(n_stars=400, obs=(10, 70), n_dfa=700, n_instr_cols=25000),
    "tail_f32": dict(n_stars=400, obs=(10, 70), n_dfa=700, n_instr_cols=25000, value_dtype="f32"),
    # bucket order, and rows enough (2^19) for A x to take its attitude part from it
    "long": dict(n_stars=6000, obs=(60, 130), n_dfa=7000, n_instr_cols=600),
    "long_f32": dict(n_stars=6000, obs=(60, 130), n_dfa=7000, n_instr_cols=600, value_dtype="f32"),
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
        S = synth.make_system(synth.tiny(seed=121 + list(SPECS).index(name), **SPECS[name]))
        sp = S.spec
        ab = oracle.OracleSystem(np.abs(S.values.astype(np.float64)), S.star_of_row, S.att_start,
                                 S.instr_idx, n_stars=sp.n_stars, n_dfa=sp.n_dfa,
                                 n_instr_cols=sp.n_instr_cols)
        _SYS[name] = (S, oracle.OracleSystem.from_synth(S), ab)
    return _SYS[name]


def gpu_system(torch, S, stream):
    from paper_2308_00778_amd import LsqrSystem

    sp = S.spec
    t = dict(values=torch.from_numpy(S.values).cuda(),
             star_of_row=torch.from_numpy(S.star_of_row).cuda(),
             att_start=torch.from_numpy(S.att_start).cuda(),
             instr_idx=torch.from_numpy(S.instr_idx).cuda())
    torch.cuda.synchronize()
    return LsqrSystem(**t, n_stars=sp.n_stars, n_dfa=sp.n_dfa, n_instr_cols=sp.n_instr_cols,
                      stream=stream)


def close2(got, want, bound, m):
    c = 2.0 * np.sqrt(m) + 32
    assert np.all(np.abs(got - want) <= c * EPS * bound + 1e-300)


# A recorded A^T y after a solve has built the compact index copies: the copies
# are freed (and their memory given other contents) before the replays.
@pytest.mark.parametrize("name", ["one_pass", "tail", "tail_f32"])
def test_recorded_aprod2_outlives_the_compact_copies(torch_cuda, name):
    torch = torch_cuda
    S, o, ab = system(name)
    say(f"recorded aprod2, compact copies freed: {name} m={S.m} n={o.n}")
    rng = np.random.default_rng(7)
    b, x0 = rng.standard_normal(S.m), rng.standard_normal(o.n)
    st = torch.cuda.Stream()
    g = gpu_system(torch, S, st)
    g.solve(torch.from_numpy(b).cuda(), 3, atol=0.0, btol=0.0)
    assert g.pass_times()["compact"] == 1
    y = torch.from_numpy(b).cuda()
    x = torch.zeros(o.n, dtype=torch.float64, device="cuda")
    g.aprod2(x, y)  # everything allocated
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        g.aprod2(x, y)
    g.set_option("compact_index", 0)
    fill = [torch.full((S.m,), -1, dtype=torch.int32, device="cuda") for _ in range(8)]
    for k in range(3):
        yk = rng.standard_normal(S.m)
        y.copy_(torch.from_numpy(yk))
        x.copy_(torch.from_numpy(x0))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        close2(x.cpu().numpy(), o.aprod2(yk, x0), ab.aprod2(np.abs(yk), np.abs(x0)), S.m)
    del graph, fill
    g.close()


# A x recorded as the first call of a handle whose attitude section the rows'
# workgroups cannot stage themselves: nothing is allocated inside the capture.
@pytest.mark.parametrize("name", ["tail", "tail_f32"])
def test_first_aprod1_can_be_recorded(torch_cuda, name):
    torch = torch_cuda
    S, o, ab = system(name)
    say(f"recorded aprod1, first call: {name} m={S.m} n={o.n}")
    rng = np.random.default_rng(8)
    st = torch.cuda.Stream()
    g = gpu_system(torch, S, st)
    x = torch.zeros(o.n, dtype=torch.float64, device="cuda")
    y = torch.zeros(S.m, dtype=torch.float64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        g.aprod1(x, y)
    for k in range(3):
        xk, y0 = rng.standard_normal(o.n), rng.standard_normal(S.m)
        want, bound = o.aprod1(xk, y0), ab.aprod1(np.abs(xk), np.abs(y0))
        for call in (graph.replay, lambda: g.aprod1(x, y)):
            x.copy_(torch.from_numpy(xk))
            y.copy_(torch.from_numpy(y0))
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            assert np.all(np.abs(y.cpu().numpy() - want) <= 32 * EPS * bound + 1e-300)
    del graph
    g.close()


# A x recorded before and after the bucket order and the scratch of its pre-pass
# exist: the recorded call never uses that scratch (a solve short of memory frees
# it), so both graphs hold the same kernels and give the same bits. Nor does an
# eager call on fewer than 2^19 rows, where gathering is quicker.
@pytest.mark.parametrize("name,buckets,vec", [("tail", 0, "f64"), ("tail_f32", 0, "f64"),
                                              ("tail_f32", 0, "f32"), ("one_pass", 3, "f64"),
                                              ("long", 0, "f64"), ("long_f32", 0, "f64"),
                                              ("long_f32", 0, "f32")])
def test_recorded_aprod1_holds_no_scratch_of_the_order(torch_cuda, name, buckets, vec):
    torch = torch_cuda
    S, o, ab = system(name)
    say(f"recorded aprod1, bucket order: {name} m={S.m} n={o.n} vec={vec}")
    dt, eps = (torch.float64, EPS) if vec == "f64" else (torch.float32, 2.0 ** -23)
    rng = np.random.default_rng(9)
    st = torch.cuda.Stream()
    g = gpu_system(torch, S, st)
    if buckets:
        g.set_option("att_buckets", buckets)
    ax, aty = (g.aprod1, g.aprod2) if vec == "f64" else (g.aprod1_f32, g.aprod2_f32)
    x = torch.zeros(o.n, dtype=dt, device="cuda")
    y = torch.zeros(S.m, dtype=dt, device="cuda")
    ax(x, y)
    torch.cuda.synchronize()
    graphs = [torch.cuda.CUDAGraph() for _ in range(2)]
    with torch.cuda.graph(graphs[0], stream=st):
        ax(x, y)
    aty(x, y)  # builds the bucket order
    ax(x, y)   # allocates the scratch of the pre-pass
    torch.cuda.synchronize()
    with torch.cuda.graph(graphs[1], stream=st):
        ax(x, y)
    for k in range(3):
        xk = torch.from_numpy(rng.standard_normal(o.n)).to(dt)
        y0 = torch.from_numpy(rng.standard_normal(S.m)).to(dt)
        got = []
        for call in (graphs[0].replay, graphs[1].replay, lambda: ax(x, y)):
            x.copy_(xk)
            y.copy_(y0)
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            got.append(y.cpu())
        assert torch.equal(got[0], got[1])
        assert torch.equal(got[0], got[2]) == (S.m < 2 ** 19)  # eager: the pre-pass
        xn, yn = xk.double().numpy(), y0.double().numpy()
        want, bound = o.aprod1(xn, yn), ab.aprod1(np.abs(xn), np.abs(yn))
        for v in got:
            assert np.all(np.abs(v.double().numpy() - want) <= 32 * eps * bound + 1e-30)
    del graphs
    g.close()


# The first A^T y of a handle, recorded: the call needs no more than what an
# earlier call of another kind has left (or nothing, without attitude), whichever
# form the options and the system's size ask for.
@pytest.mark.parametrize("before", ["batched", "fused1", "fused2"])
def test_first_aprod2_recorded_after_other_calls(torch_cuda, before):
    torch = torch_cuda
    S, o, ab = system("one_pass")
    say(f"recorded aprod2, first call after {before}: m={S.m} n={o.n}")
    rng = np.random.default_rng(10)
    st = torch.cuda.Stream()
    g = gpu_system(torch, S, st)
    b = torch.from_numpy(rng.standard_normal((S.m, 2))).cuda()
    if before == "batched":  # the bucket order only, and the recorded call asks for one pass
        g.set_option("ktile", 2)
        g.solve_batched(b, 2, 0.0, 0.0)
    else:
        g.set_option("fused", int(before[-1]))
        g.solve(b[:, 0].contiguous(), 2, atol=0.0, btol=0.0)
        g.set_option("fused", 3 - int(before[-1]))
    _record_aprod2(torch, g, st, S.m, o, ab, rng)


def test_first_aprod2_recorded_without_attitude(torch_cuda):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    spec = synth.tiny(seed=131, n_stars=300, obs=(10, 70), n_axes=0, n_glob=2)
    S = synth.make_system(spec)
    o = oracle.OracleSystem.from_synth(S)
    ab = oracle.OracleSystem(np.abs(S.values), S.star_of_row, S.att_start, S.instr_idx,
                             n_stars=spec.n_stars, n_dfa=spec.n_dfa,
                             n_instr_cols=spec.n_instr_cols, n_axes=0, n_glob=2)
    say(f"recorded aprod2, first call, no attitude section: m={S.m} n={o.n}")
    st = torch.cuda.Stream()
    t = dict(values=torch.from_numpy(S.values).cuda(),
             star_of_row=torch.from_numpy(S.star_of_row).cuda(),
             att_start=torch.from_numpy(S.att_start).cuda(),
             instr_idx=torch.from_numpy(S.instr_idx).cuda())
    torch.cuda.synchronize()
    g = LsqrSystem(**t, n_stars=spec.n_stars, n_dfa=spec.n_dfa, n_instr_cols=spec.n_instr_cols,
                   n_axes=0, n_glob=2, stream=st)
    _record_aprod2(torch, g, st, S.m, o, ab, np.random.default_rng(11))


def _record_aprod2(torch, g, st, m, o, ab, rng):
    x = torch.zeros(o.n, dtype=torch.float64, device="cuda")
    y = torch.zeros(m, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        g.aprod2(x, y)
    for k in range(3):
        yk, x0 = rng.standard_normal(m), rng.standard_normal(o.n)
        want, bound = o.aprod2(yk, x0), ab.aprod2(np.abs(yk), np.abs(x0))
        for call in (graph.replay, lambda: g.aprod2(x, y)):
            y.copy_(torch.from_numpy(yk))
            x.copy_(torch.from_numpy(x0))
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            close2(x.cpu().numpy(), want, bound, m)
    del graph
    g.close()
