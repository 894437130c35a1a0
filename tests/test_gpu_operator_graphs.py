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
@pytest.mark.parametrize("name", list(SPECS))
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
