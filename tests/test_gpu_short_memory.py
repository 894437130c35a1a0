"""A solve where device memory is short: the scratch that an earlier A x keeps in
the handle is given up for it (1e8 rows, FP32 values: 800 MB of scratch; all but
about 500 MB of the rest of the memory is taken).
"""
import contextlib

import pytest

import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_solve_takes_the_operators_scratch(torch_cuda):
    torch = torch_cuda
    from paper_2308_00778_amd import LsqrSystem

    torch.cuda.empty_cache()
    spec = synth.tiny(seed=141, n_stars=1000000, obs=(100, 100), n_dfa=100000, n_instr_cols=6000,
                      value_dtype="f32")
    arrays, first = synth.device_system(spec, "cuda:0")
    m = int(first[-1])
    say(f"short memory: m={m}")
    g = LsqrSystem(**arrays, n_stars=spec.n_stars, n_dfa=spec.n_dfa,
                   n_instr_cols=spec.n_instr_cols)
    b = synth.device_noise(spec, m, 0, "cuda:0")
    hogs = []
    try:
        g.set_option("tests", 0)
        want, _ = g.solve(b, 3, atol=0.0, btol=0.0)  # the solver's own vectors
        y = torch.zeros(m, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free0 = torch.cuda.mem_get_info()[0]
        g.aprod1(want, y)
        torch.cuda.synchronize()
        assert free0 - torch.cuda.mem_get_info()[0] >= 8 * m  # the scratch
        # all of the memory in blocks, then four of 128 MB given back
        for size in (8 << 30, 1 << 30, 128 << 20):
            if size == 128 << 20:
                del hogs[-1]
                torch.cuda.empty_cache()
            with contextlib.suppress(torch.cuda.OutOfMemoryError):
                while True:
                    hogs.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert hogs[-4].numel() == 128 << 20
        del hogs[-4:]
        torch.cuda.empty_cache()
        say(f"  {torch.cuda.mem_get_info()[0] / 1e6:.0f} MB reported free")
        with pytest.raises(torch.cuda.OutOfMemoryError):
            torch.empty(m, dtype=torch.float64, device="cuda")
        # row-order u~: a vector of m values more
        g.set_option("fused", 3)
        x = torch.empty_like(want)
        g.solve(b, 3, atol=0.0, btol=0.0, x=x)
        hogs.clear()
        torch.cuda.synchronize()
        err = float((x - want).abs().max() / want.abs().max())
        say(f"  rel_inf {err:.2e}")
        assert err <= 1e-10
    finally:
        hogs.clear()
        g.close()
        torch.cuda.empty_cache()
