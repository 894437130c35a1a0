"""A x of a system with more than 2^31 attitude columns per axis: attitude starts
need all 64 bits. The column vectors of the handle take 206 GB (258 GB while it
is created), so the module runs on its own and only where that much is free.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -23
N_DFA = 2 ** 31 + 1000
STARTS = [0, 1, 2 ** 31 - 5, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 500, N_DFA - 4]


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# FP32 vectors (half the memory), the windows read from x and from its
# interleaved copy
def test_starts_beyond_32_bits(torch_cuda):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    torch.cuda.empty_cache()
    n = 5 + 3 * N_DFA + 6 + 1
    need = 5 * 8 * n + (4 << 30)
    free = torch.cuda.mem_get_info()[0]
    say(f"wide attitude: n={n}, {need / 1e9:.0f} GB needed, {free / 1e9:.0f} GB free")
    if free < need:
        pytest.skip("not enough device memory")
    rng = np.random.default_rng(41)
    m = len(STARTS)
    values = rng.standard_normal((24, m)).astype(np.float32)
    t = np.array(STARTS, dtype=np.int64)
    instr = np.repeat(np.arange(6, dtype=np.int32)[:, None], m, axis=1)
    g = LsqrSystem(torch.from_numpy(values).cuda(), torch.zeros(m, dtype=torch.int64, device="cuda"),
                   torch.from_numpy(t).cuda(), torch.from_numpy(instr).cuda(), n_stars=1,
                   n_dfa=N_DFA, n_instr_cols=6)
    try:
        x = torch.zeros(n, dtype=torch.float32, device="cuda")
        for lo, hi in ((0, 5), (n - 7, n)):
            x[lo:hi] = torch.from_numpy(rng.standard_normal(hi - lo).astype(np.float32)).cuda()
        for ax in range(3):
            for s in STARTS:
                c = 5 + ax * N_DFA + s
                x[c:c + 4] = torch.from_numpy(rng.standard_normal(4).astype(np.float32)).cuda()
        cols = [np.arange(5)[:, None] + np.zeros(m, dtype=np.int64)]
        cols += [(5 + ax * N_DFA + q + t)[None, :] for ax in range(3) for q in range(4)]
        cols += [np.arange(n - 7, n)[:, None] + np.zeros(m, dtype=np.int64)]
        cols = np.concatenate(cols, 0)
        xs = np.array([x[c].item() for c in cols.ravel().tolist()]).reshape(cols.shape)
        v = values.astype(np.float64)
        want, bound = (v * xs).sum(0), np.abs(v * xs).sum(0)
        for interleave in (0, 1):
            say(f"wide attitude: aprod1_f32 interleave={interleave}")
            g.set_option("att_interleave", interleave)
            y = torch.zeros(m, dtype=torch.float32, device="cuda")
            g.aprod1_f32(x, y)
            torch.cuda.synchronize()
            got = y.cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - want) <= 32 * EPS32 * bound)
    finally:
        g.close()
        x = None
        torch.cuda.empty_cache()
