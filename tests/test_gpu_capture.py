"""GPU tests of sweeps captured by the caller's own graph: replays follow the
sweep index on the device."""
import numpy as np
import pytest

from paper_1402_1763_amd import binding, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision,chains", [(32, "fp64", 1), (64, "fp32", 1), (64, "fp32", 5),
                                                (256, "fp32", 1)])
def test_replays_of_captured_sweeps_record_by_the_device_index(n, precision, chains):
    """Four captured sweeps replayed five times, recording every third sample:
    state, trace and moments bitwise those of 20 eager sweeps."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    ws = [workloads.small_workload(n, 9, precision=precision, seed=51 + c, rng_seed=53)
          for c in range(chains)]
    pbs = [workloads.make_problem(w) for w in ws]
    side = torch.cuda.Stream()
    out = []
    with torch.cuda.stream(side):
        for _ in range(2):
            smp = binding.Sampler([p["data"] for p in pbs], [p["noise_var"] for p in pbs],
                                  [p["pk_init"] for p in pbs], 9, ws[0].box, seed=53,
                                  precision=precision)
            smp.set_diagnostics(start=2, thin=3, trace_cap=8, moments=True)
            out.append(smp)
    eager, smp = out
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        smp.sweep(4)
    for _ in range(5):
        with torch.cuda.stream(side):
            graph.replay()
        torch.cuda.synchronize()
    eager.sweep(20)
    for c in range(chains):
        smp.set_state(c, None, None, 20)     # the host's count: what the replays did
    assert smp.recorded() == eager.recorded() == 6
    for c in range(chains):
        s, p, done = eager.state(c)
        s2, p2, done2 = smp.state(c)
        assert done == done2 == 20 and np.array_equal(s, s2) and np.array_equal(p, p2)
        assert torch.equal(smp.trace(c), eager.trace(c))
        maps = smp.moments(c) + eager.moments(c)
        torch.cuda.synchronize()             # written on the samplers' stream
        assert torch.equal(maps[0], maps[2]) and torch.equal(maps[1], maps[3])
    for x in out:
        x.close()
