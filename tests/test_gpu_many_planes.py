"""GPU tests of what runs where planes queue (more of them than the 256 CUs) or
where the library keeps the four-pass schedule: the Wiener filter, the
log-determinant, sweeps and mixing sweeps against the oracle."""
import numpy as np
import pytest

from oracle import adjoint, logdet, mixing, sampler
from paper_1402_1763_amd import binding, workloads
from tests.gpu_util import TOL, errors, gpu_sampler, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.load()
    torch.cuda.set_device(0)


def _rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def _problems(n, precision, chains, nb=8):
    ws = [workloads.small_workload(n, nb, precision=precision, seed=140 + c, rng_seed=37,
                                   mask_frac=0.1 + 0.05 * c, sigma2=0.5 + 0.5 * c) for c in range(chains)]
    pbs = [workloads.make_problem(w) for w in ws]
    smp = binding.Sampler([p["data"] for p in pbs], [p["noise_var"] for p in pbs],
                          [p["pk_init"] for p in pbs], nb, ws[0].box, seed=37, precision=precision)
    return ws, pbs, smp


# FP64 96^3 x 3 keeps four passes; the others are planes in queues
@pytest.mark.parametrize("precision,n,chains", [("fp64", 96, 3), ("fp32", 80, 4), ("fp32", 128, 3),
                                                ("fp64", 64, 5)])
def test_wiener_gradient_and_logdet_match_oracle(precision, n, chains):
    import torch
    k, every = 5, 2
    ws, pbs, smp = _problems(n, precision, chains)
    pk = np.stack([(0.4 + 0.1 * c) * workloads.power_spectrum(workloads.bin_centres(w), w)
                   for c, w in enumerate(ws)])
    d = torch.from_numpy(np.stack([p["data"] for p in pbs])).cuda()
    pk_t = torch.from_numpy(pk).cuda()
    wf = binding.WienerFilter(smp, k, every, chain=None)
    chi2, _ = wf.forward(d, pk_t)
    gd, gp = wf.backward(d)
    tr = wf.logdet_trace(pk_t, 1, probe0=3)
    for c in (0, chains - 1):
        one = binding.WienerFilter(smp, k, every, chain=c)       # few planes
        c1, _ = one.forward(d[c].contiguous(), pk_t[c].contiguous())
        gd1, gp1 = one.backward(d[c].contiguous())
        assert float(c1) == float(chi2[c])
        assert torch.equal(gd1, gd[c]) and torch.equal(gp1, gp[c])
        assert torch.equal(one.logdet_trace(pk_t[c].contiguous(), 1, probe0=3), tr[c])
        prob = oracle_problem(ws[c], pbs[c], chain=c)
        vc = ws[c].cell_volume
        loss, gp_ref, gd_ref = adjoint.wf_gradient(prob, pk[c] / vc, k)
        errs = (abs(float(chi2[c]) - loss) / abs(loss), _rel(gd[c].cpu().numpy(), gd_ref),
                _rel(gp[c].cpu().numpy(), gp_ref / vc),
                _rel(tr[c].cpu().numpy(), logdet.trace_probe(prob, pk[c] / vc, k, 3) / vc))
        print(f"{n}^3 {precision} x {chains}, chain {c}: chi2 %.1e grad_d %.1e grad_P %.1e trace %.1e" % errs,
              flush=True)
        assert max(errs) < TOL[precision]
    smp.close()


@pytest.mark.timeout(300)
def test_wiener_gradient_at_256_matches_oracle():
    """The four-pass iteration in FP32, two iterations with a checkpoint each."""
    import torch
    ws, pbs, smp = _problems(256, "fp32", 1, nb=16)
    w, pb = ws[0], pbs[0]
    pk = 0.5 * workloads.power_spectrum(workloads.bin_centres(w), w)
    d = torch.from_numpy(pb["data"]).cuda()
    wf = binding.WienerFilter(smp, 2, 1)
    chi2, _ = wf.forward(d, torch.from_numpy(pk).cuda())
    gd, gp = wf.backward(d)
    torch.cuda.synchronize()
    print("256^3: oracle", flush=True)
    loss, gp_ref, gd_ref = adjoint.wf_gradient(oracle_problem(w, pb), pk / w.cell_volume, 2)
    errs = (abs(float(chi2) - loss) / abs(loss), _rel(gd.cpu().numpy(), gd_ref),
            _rel(gp.cpu().numpy(), gp_ref / w.cell_volume))
    print("  chi2 %.1e grad_d %.1e grad_P %.1e" % errs, flush=True)
    assert max(errs) < TOL["fp32"]
    smp.close()


# two histogram sets of 8 copies per wave up to 96 bins, of 2 beyond
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nb", [96, 97, 300])
def test_mixing_sweeps_of_many_bins_match_oracle(precision, nb):
    w = workloads.small_workload(32, nb, precision=precision, seed=87, rng_seed=88)
    pb = workloads.make_problem(w)
    smp = gpu_sampler(w, pb)
    smp.sweep(1)
    smp.mixing_sweep(2)
    s_gpu, p_gpu, done = smp.state()
    smp.close()
    prob = oracle_problem(w, pb)
    st = sampler.State(s=np.zeros((w.n,) * 3), p_grid=pb["pk_init"] / w.cell_volume)
    st = sampler.sweep(prob, st)
    for _ in range(2):
        st = mixing.mixing_sweep(prob, st)
    err_s, err_p = errors(s_gpu, p_gpu, st.s, st.p_grid * w.cell_volume)
    print(f"mixing {nb} bins {precision}: err_s={err_s:.1e} err_P={err_p:.1e}", flush=True)
    assert done == 3 and err_s < TOL[precision] and err_p < TOL[precision]


# FP64 96^3 x 3 and 128^3 x 3: four passes by default, planes in queues when chosen
@pytest.mark.parametrize("path", [None, "whole"])
@pytest.mark.parametrize("precision,n,chains", [("fp64", 96, 3), ("fp64", 128, 3), ("fp32", 96, 4)])
def test_runs_equal_single_sweeps_and_match_oracle(precision, n, chains, path):
    ws, pbs, run = _problems(n, precision, chains)
    _, _, single = _problems(n, precision, chains)
    for smp in (run, single):
        if path:
            smp.set_x_path(path)
        smp.set_diagnostics(start=1, thin=1, trace_cap=4, moments=True)
    run.sweep(3)
    for _ in range(3):
        single.sweep(1)
    for c in range(chains):
        s, p, _ = run.state(c)
        s1, p1, _ = single.state(c)
        assert np.array_equal(s, s1) and np.array_equal(p, p1)
        for a, b in zip(run.moments(c), single.moments(c)):
            assert bool((a == b).all())
    c = chains - 1
    prob = oracle_problem(ws[c], pbs[c], chain=c)
    st = sampler.State(s=np.zeros((n,) * 3), p_grid=pbs[c]["pk_init"] / ws[c].cell_volume)
    st = sampler.run_chain(prob, st, 3)
    err_s, err_p = errors(s, p, st.s, st.p_grid * ws[c].cell_volume)
    print(f"{n}^3 {precision} x {chains} {path}: err_s={err_s:.1e} err_P={err_p:.1e}", flush=True)
    assert err_s < TOL[precision] and err_p < TOL[precision]
    run.close()
    single.close()
