"""GPU tests of the two-pass (plane) sweep of grid sides up to 128: its joined
launches against the same sweeps one call at a time."""
import numpy as np
import pytest

from paper_1402_1763_amd import binding, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()
    torch.cuda.set_device(0)


def _samplers(n, precision, chains, count):
    ws = [workloads.small_workload(n, 9, precision=precision, seed=41 + c, rng_seed=43)
          for c in range(chains)]
    pbs = [workloads.make_problem(w) for w in ws]
    out = []
    for _ in range(count):
        smp = binding.Sampler([p["data"] for p in pbs], [p["noise_var"] for p in pbs],
                              [p["pk_init"] for p in pbs], 9, ws[0].box, seed=43,
                              precision=precision)
        smp.set_diagnostics(start=2, thin=7, trace_cap=6, moments=True)
        out.append(smp)
    return out


# a few planes, and more planes than CUs (other workgroups at 80 and 128)
@pytest.mark.parametrize("n,precision,chains", [(8, "fp64", 2), (16, "fp64", 1), (48, "fp32", 3),
                                                (80, "fp32", 4), (80, "fp64", 1), (80, "fp64", 4),
                                                (96, "fp32", 1), (96, "fp32", 3),
                                                (128, "fp32", 3), (128, "fp64", 1)])
def test_a_run_of_sweeps_equals_single_sweeps(n, precision, chains):
    """35 sweeps (the P draws' gamma variates are computed 32 sweeps ahead) in
    one call, one by one and by graph replays, recording every 7th: states,
    traces and moments bitwise equal; the four kernels one by one, too."""
    run, single, graph, timed = _samplers(n, precision, chains, 4)
    run.sweep(35)
    for _ in range(35):
        single.sweep(1)
    g = binding.SweepGraph([graph])
    g.launch(34)
    g.launch(1)
    g.close()
    timed.sweep_timed(35)
    for c in range(chains):
        s, p, done = run.state(c)
        mean, var = run.moments(c)
        assert done == 35 and np.isfinite(s).all()
        for other in (single, graph, timed):
            s2, p2, done2 = other.state(c)
            assert done2 == 35 and np.array_equal(s, s2) and np.array_equal(p, p2)
            assert np.array_equal(run.trace(c).cpu().numpy(), other.trace(c).cpu().numpy())
            m2, v2 = other.moments(c)
            assert bool((mean == m2).all()) and bool((var == v2).all())
