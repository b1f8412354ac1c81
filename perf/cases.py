"""The work that a user of this framework has it do, as cases to be timed and checked.

Kinds of case, each through the public entry points of paper_1402_1763_amd:
  gibbs    k Gibbs sweeps of one problem (1 or more chains) that records the P(k) trace and the
           running posterior moments, then the moments' maps (Sampler.sweep, Sampler.moments)
  batch    k replays of one graph over problems of several grid sides, with the same records
  mixing   k mixing sweeps (joint update of signal and spectrum), with the same records
  wiener   chi2 of the messenger Wiener filter and its gradients by the spectrum and the data
           (autograd.wiener_chi2, forward and backward)
  logdet   the log-determinant term of the spectrum gradient (WienerFilter.logdet_trace)
  acf      autocorrelation and correlation lengths of a recorded P(k) trace (binding.acf)
  session  a whole short run on host data: set up a Sampler, sweep, read the state back

Results of FP32 problems come back from the library as float64 arrays that hold FP32 precision;
a program keeps those in float32, and so does run().
"""
import math

import numpy as np
import torch

from paper_1402_1763_amd import autograd, binding

SIDES = (8, 16, 32, 48, 64, 80, 96, 128, 256)      # 512 is left out: its set-up alone takes many seconds
BATCH = ((64, 32), (48, 8), (80, 8), (96, 8))      # (grid side, chains) of the batched workload


def listed():
    return [
        # the smallest problems: a sweep is a handful of launches, so latency counts
        dict(name="gibbs-16-fp64", kind="gibbs", n=16, bins=8, prec="fp64", mask="none", sweeps=50),
        # the small FP64 configuration: 20% of the voxels unobserved at random
        dict(name="gibbs-32-fp64", kind="gibbs", n=32, bins=16, prec="fp64", mask="random", sweeps=50),
        # an odd side (radix 5) in FP64, with a per-voxel response and a proper prior on P(k)
        dict(name="gibbs-80-fp64-response", kind="gibbs", n=80, bins=16, prec="fp64", mask="random",
             sweeps=25, response=True, prior_b0=50.0),
        # the 128^3 survey configuration: sphere minus a wedge, FP32 fields
        dict(name="gibbs-128-fp32-survey", kind="gibbs", n=128, bins=32, prec="fp32", mask="survey",
             sweeps=25),
        # the 256^3 survey configuration, which the headline benchmark runs
        dict(name="gibbs-256-fp32-survey", kind="gibbs", n=256, bins=64, prec="fp32", mask="survey",
             sweeps=20),
        # many independent mocks of several sides in one graph
        dict(name="batch-48-96-fp32", kind="batch", bins=16, prec="fp32", sweeps=25),
        # mixing sweeps at the size of the headline benchmark
        dict(name="mixing-256-fp32-survey", kind="mixing", n=256, bins=64, prec="fp32",
             mask="survey", sweeps=10),
        # gradient-based inference on one data set, and on eight data sets in one launch each
        dict(name="wiener-128-fp32", kind="wiener", n=128, bins=32, prec="fp32", mask="survey",
             iters=50, every=10, chains=1),
        dict(name="wiener-128-fp32-x8", kind="wiener", n=128, bins=32, prec="fp32", mask="survey",
             iters=50, every=10, chains=8),
        # the same gradient's log-determinant term, by random probes
        dict(name="logdet-96-fp32", kind="logdet", n=96, bins=16, prec="fp32", mask="random",
             iters=30, probes=4, chains=1),
        # statistical efficiency of a recorded chain: 8000 samples of 32 bins, lags to 400
        dict(name="acf-8000x32", kind="acf", t=8000, bins=32, lag=400),
        # a new data set from host arrays to a sample in host memory
        dict(name="session-128-fp32", kind="session", n=128, bins=32, prec="fp32", mask="survey",
             sweeps=100),
    ]


def draw(rng):
    kind = rng.choice(["gibbs", "gibbs", "gibbs", "batch", "mixing", "wiener", "logdet", "acf",
                       "session"])
    if kind == "acf":
        t = int(math.exp(rng.uniform(math.log(50), math.log(20000))))
        bins = int(math.exp(rng.uniform(0, math.log(200))))
        return dict(kind=kind, t=t, bins=bins, lag=rng.randint(1, min(t - 1, 600)))
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "batch":
        return dict(kind=kind, bins=rng.randint(4, 40), prec="fp32", sweeps=rng.randint(5, 25))
    n = rng.choice(SIDES[2:] if kind in ("mixing", "wiener", "logdet") else SIDES)
    if kind in ("wiener", "logdet", "session"):
        n = min(n, 128)
    cap = (256 if prec == "fp32" else 200) ** 3 if kind in ("gibbs", "mixing") else 2 * 128 ** 3
    chains = max(1, min(40, cap // n ** 3))
    case = dict(kind=kind, n=n, bins=rng.randint(3, max(4, min(300, n))), prec=prec,
                mask=rng.choice(["random", "survey", "none"]),
                chains=rng.randint(1, chains) if kind != "session" else 1,
                response=rng.random() < 0.25)
    if kind in ("gibbs", "mixing", "session"):
        case["sweeps"] = rng.randint(3, 15)
        case["prior_b0"] = rng.choice([0.0, 50.0])
    else:
        case["iters"] = rng.randint(3, 25)
        case["every"] = rng.randint(1, case["iters"])
        case["probes"] = rng.randint(1, 4)
    return case


# ---------------------------------------------------------------- inputs
def spectrum(k):
    """P(k) of the mocks, in volume units; 0 at k = 0."""
    k = np.asarray(k, dtype=np.float64)
    kk = np.where(k > 0, k, 1.0)
    return np.where(k > 0, 1.0e4 * kk ** -1.5 * np.exp(-(kk / 0.3) ** 2), 0.0)


def box_of(n):
    return 500.0 if n == 32 else 7.8125 * n


def bin_spectrum(n, bins):
    dk = math.sqrt(3.0) * math.pi * n / box_of(n) / bins
    return spectrum((np.arange(bins) + 0.5) * dk)


def mock(n, mask, response, seed):
    """A mock survey (data, noise variance, response or None) as float64 arrays on the GPU: a
    Gaussian field of the mocks' spectrum, seen with noise on the observed voxels."""
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    box = box_of(n)
    vcell = (box / n) ** 3
    m = torch.fft.fftfreq(n, d=1.0 / n, dtype=torch.float64, device=dev)
    mz = torch.arange(n // 2 + 1, dtype=torch.float64, device=dev)
    k = 2 * math.pi / box * (m[:, None, None] ** 2 + m[None, :, None] ** 2 + mz ** 2).sqrt()
    kk = k.clamp_min(1e-30)
    amp = torch.where(k > 0, 1.0e4 * kk ** -1.5 * torch.exp(-(kk / 0.3) ** 2) / vcell, 0.0).sqrt()
    white = torch.randn((n, n, n), dtype=torch.float64, device=dev, generator=gen)
    s = torch.fft.irfftn(torch.fft.rfftn(white) * amp, s=(n, n, n))
    u = torch.rand((n, n, n), dtype=torch.float64, device=dev, generator=gen)
    if mask == "survey":
        c = (torch.arange(n, dtype=torch.float64, device=dev) + 0.5) * (box / n) - 0.5 * box
        x, y, z = c[:, None, None], c[None, :, None], c[None, None, :]
        r2 = x * x + y * y + z * z
        phi0 = float(torch.rand(1, dtype=torch.float64, device=dev, generator=gen)) * 360.0
        phi = torch.rad2deg(torch.atan2(y, x)) % 360.0
        seen = (r2 < (0.45 * box) ** 2) & ((phi - phi0) % 360.0 >= 30.0)
        noise = 1.0 / (3.0e-4 * torch.exp(-r2 / 400.0 ** 2) * vcell)
    else:
        seen = torch.rand((n, n, n), device=dev, generator=gen) >= (0.2 if mask == "random" else -1.0)
        noise = 0.5 + 1.5 * u
    resp = None
    if response:
        resp = 0.5 + torch.rand((n, n, n), dtype=torch.float64, device=dev, generator=gen)
    eps = torch.randn((n, n, n), dtype=torch.float64, device=dev, generator=gen)
    d = (s if resp is None else resp * s) + noise.sqrt() * eps
    return (torch.where(seen, d, 0.0).contiguous(),
            torch.where(seen, noise, math.inf).contiguous(), resp)


def mocks(case, seed):
    """The case's problems: a list of (grid side, [mock of every chain])."""
    if case["kind"] == "batch":
        sizes, mask = BATCH, "random"
    else:
        sizes, mask = ((case["n"], case.get("chains", 1)),), case["mask"]
    return [(n, [mock(n, mask, case.get("response", False), seed * 1000 + 100 * i + c)
                 for c in range(chains)]) for i, (n, chains) in enumerate(sizes)]


def sampler(case, n, chains, seed, sample_pk=True):
    host = [[None if a is None else a.cpu().numpy() for a in one] for one in chains]
    pk = 0.1 * bin_spectrum(n, case["bins"])
    return binding.Sampler([h[0] for h in host], [h[1] for h in host], [pk] * len(host),
                           case["bins"], box_of(n), seed=seed, precision=case["prec"],
                           sample_pk=sample_pk,
                           response=[h[2] for h in host] if case.get("response") else None,
                           pk_prior=(0.0, case.get("prior_b0", 0.0)))


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "acf":
        rng = np.random.default_rng(seed)
        phi = rng.uniform(0.3, 0.999, case["bins"])
        x = np.empty((case["t"], case["bins"]))
        e = rng.standard_normal(x.shape) * np.sqrt(1 - phi * phi)
        x[0] = rng.standard_normal(case["bins"])
        for i in range(1, case["t"]):
            x[i] = phi * x[i - 1] + e[i]
        state["trace"] = torch.from_numpy(np.exp(0.3 * x)).cuda()
        return state
    problems = mocks(case, seed)
    if kind == "session":
        n, chains = problems[0]
        state["host"] = [None if a is None else a.cpu().numpy() for a in chains[0]]
        state["seed"] = seed
        return state
    state["samplers"] = [sampler(case, n, chains, seed + i, sample_pk=kind not in ("wiener", "logdet"))
                         for i, (n, chains) in enumerate(problems)]
    if kind in ("gibbs", "batch", "mixing"):
        # one sample a pass: P(k) of the first 8, and the running moments of the signal
        for smp in state["samplers"]:
            smp.set_diagnostics(start=case["sweeps"] - 1, thin=case["sweeps"], trace_cap=8,
                                moments=True)
        if kind == "batch":
            state["graph"] = binding.SweepGraph(state["samplers"])
        return state
    n, chains = problems[0]
    smp = state["samplers"][0]
    one = len(chains) == 1
    pk = torch.from_numpy(np.stack([bin_spectrum(n, case["bins"])] * len(chains))).cuda()
    state["wf"] = binding.WienerFilter(smp, case["iters"], case.get("every", case["iters"]),
                                       chain=0 if one else None)
    state["pk"] = pk[0].clone() if one else pk
    if kind == "wiener":
        d = torch.stack([c[0] for c in chains])
        state["d"] = d[0].clone() if one else d
    return state


# ---------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "acf":
        return binding.acf(state["trace"], case["lag"])
    keep = (lambda t: t.float()) if case["prec"] == "fp32" else (lambda t: t)
    if kind == "session":
        data, noise, resp = state["host"]
        smp = binding.Sampler(data, noise, 0.1 * bin_spectrum(case["n"], case["bins"]),
                              case["bins"], box_of(case["n"]), seed=state["seed"],
                              precision=case["prec"], response=resp,
                              pk_prior=(0.0, case.get("prior_b0", 0.0)))
        smp.sweep(case["sweeps"])
        s, pk, _ = smp.state()
        smp.close()
        to = np.float32 if case["prec"] == "fp32" else np.float64
        return s.astype(to, copy=False), pk.astype(to, copy=False)
    if kind == "wiener":
        pk, d = state["pk"].requires_grad_(), state["d"].requires_grad_()
        chi2 = autograd.wiener_chi2(pk, d, state["wf"])
        grad_pk, grad_d = torch.autograd.grad(chi2.sum(), (pk, d))
        return keep(chi2.detach()), keep(grad_pk), keep(grad_d)
    if kind == "logdet":
        return keep(state["wf"].logdet_trace(state["pk"], case["probes"]))
    if kind == "batch":
        state["graph"].launch(case["sweeps"])
    elif kind == "mixing":
        state["samplers"][0].mixing_sweep(case["sweeps"])
    else:
        state["samplers"][0].sweep(case["sweeps"])
    out = []
    for smp in state["samplers"]:
        maps = [smp.moments(c) for c in range(smp.n_chains)]
        rows = min(smp.recorded(), 8)
        out.append((keep(smp.trace_buf[:, :rows]),
                    [keep(torch.stack([m[i] for m in maps])) if len(maps) > 1 else keep(maps[0][i])
                     for i in (0, 1)]))
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def sweep_work(n, real, seen):
    """Bytes and operations of one sweep: the field and the observed voxels' two coefficients
    read, the field written; a real 3D transform each way and about 60 operations a voxel for
    the two draws."""
    m = n ** 3
    return (2 + 2 * seen) * m * real, 5 * m * math.log2(m) + 60 * m


def work(case):
    kind = case["kind"]
    if kind == "acf":
        t, b, lag = case["t"], case["bins"], case["lag"]
        return {"bytes": 8 * b * (t + lag + 1), "flops": 2.0 * b * sum(t - i for i in range(lag + 1))}
    real = 4 if case["prec"] == "fp32" else 8
    seen = {"survey": 0.35, "random": 0.8, "none": 1.0}[case.get("mask", "random")]
    byts = flops = 0.0
    for n, chains in (BATCH if kind == "batch" else ((case["n"], case.get("chains", 1)),)):
        m = n ** 3
        b, f = sweep_work(n, real, seen)
        if kind in ("gibbs", "batch", "mixing"):
            # the sweeps, one update of the running moments, and their two maps
            b, f = case["sweeps"] * b + m * (4 * 8 + 2 * 8 + 2 * real), case["sweeps"] * f + 10 * m
        elif kind == "session":
            # data and noise in, the sample out
            b, f = case["sweeps"] * b + 3 * 8 * m, case["sweeps"] * f + 10 * m
        elif kind == "wiener":
            # a forward and an adjoint iteration each, the latter with the stored iterate
            b, f = case["iters"] * (2 * b + m * real) + 3 * 8 * m, 2 * case["iters"] * (f - 50 * m)
        else:
            b, f = case["probes"] * case["iters"] * b, case["probes"] * case["iters"] * (f - 50 * m)
        byts, flops = byts + chains * b, flops + chains * f
    return {"bytes": byts, "flops": flops}


# ---------------------------------------------------------------- the same in 64 bits
# Plain torch in float64 from the model's equations; the random numbers follow the library's
# documented contract (Philox4x32-10 counters and Box-Muller, include/mf.h).
M32 = 0xFFFFFFFF


def mul_hi_lo(const, x):
    """High and low 32 bits of const * x, for int64 tensors (or arrays) of 32-bit values."""
    lo = const * (x & 0xFFFF)
    hi = const * (x >> 16) + (lo >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def philox(c0, c1, c2, c3, seed):
    """Four words of counter (c0, c1, c2, c3), int64 tensors or arrays that broadcast."""
    k0, k1 = seed & M32, (seed >> 32) & M32
    c1, c2, c3 = c0 * 0 + c1, c0 * 0 + c2, c0 * 0 + c3
    for _ in range(10):
        h0, l0 = mul_hi_lo(0xD2511F53, c0)
        h1, l1 = mul_hi_lo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def uniform(x):
    x = x >> 9
    return ((x.double() if isinstance(x, torch.Tensor) else x) + 0.5) * 2.0 ** -23


def normals(xa, xb):
    lib = torch if isinstance(xa, torch.Tensor) else np
    r, a = lib.sqrt(-2.0 * lib.log(uniform(xa))), 2.0 * math.pi * uniform(xb)
    return r * lib.cos(a), r * lib.sin(a)


class Exact:
    """The chains of one problem in 64 bits, all at once (leading axis: the chain)."""

    def __init__(self, case, n, chains, seed):
        dev = "cuda"
        self.n, self.nb, self.seed, self.m = n, case["bins"], seed, n ** 3
        self.chains = len(chains)
        self.vcell = (box_of(n) / n) ** 3
        self.b0 = case.get("prior_b0", 0.0) / self.vcell
        d = torch.stack([c[0] for c in chains])
        nv = torch.stack([c[1] for c in chains])
        r = torch.stack([c[2] for c in chains]) if case.get("response") else torch.ones_like(d)
        self.seen = torch.isfinite(nv) & (r != 0)
        self.d, self.nv, self.r = d, nv, torch.where(self.seen, r, 0.0)
        ratio = torch.where(self.seen, nv / torch.where(self.seen, r * r, 1.0), math.inf)
        self.tau = ratio.amin(dim=(1, 2, 3))
        tau = self.tau[:, None, None, None]
        self.omw = torch.where(self.seen, (tau * r * r / nv).clamp(max=1.0), 0.0)
        self.beta = torch.where(self.seen, tau * r * d / nv, 0.0)
        i = torch.arange(n, device=dev)
        k = torch.where(i <= n // 2, i, i - n)
        kz = torch.arange(n // 2 + 1, device=dev)
        q = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz ** 2
        thr = [-((-3 * b * b * n * n) // (4 * self.nb ** 2)) for b in range(1, self.nb)]
        edge = torch.tensor(thr, dtype=torch.int64, device=dev)
        self.bin = torch.bucketize(q, edge, right=True)
        self.live = q > 0
        w = torch.full((n // 2 + 1,), 2.0, dtype=torch.float64, device=dev)
        w[0] = w[-1] = 1.0
        self.w = torch.where(self.live, w, 0.0)
        self.count = torch.bincount(self.bin.flatten(), self.w.flatten(), self.nb).cpu().numpy()

    def fft(self, x):
        return torch.fft.rfftn(x, dim=(1, 2, 3))

    def ifft(self, x):
        return torch.fft.irfftn(x, s=(self.n,) * 3, dim=(1, 2, 3))

    def per_mode(self, v):
        """[chain, bin] values at every mode, 0 at k = 0."""
        return torch.where(self.live, v[:, self.bin], 0.0)

    def per_bin(self, x):
        """Full-grid sums of x over every bin: [chain, bin]."""
        return torch.stack([torch.bincount(self.bin.flatten(), (x[c] * self.w).flatten(), self.nb)
                            for c in range(self.chains)])

    def each(self, f):
        return torch.stack([f(c) for c in range(self.chains)])

    def messenger_normals(self, sweep):
        n = self.n
        c0 = torch.arange(n * n * (n // 4), device="cuda").view(n, n, n // 4)

        def one(c):
            x = philox(c0, sweep, 0, c, self.seed)
            return torch.cat(normals(x[0], x[1]) + normals(x[2], x[3]), dim=2)
        return self.each(one)

    def signal_normals(self, sweep):
        """Complex normals of every mode, Hermitian on the planes kz = 0 and N/2: a
        self-conjugate mode is real with the full variance, and of a conjugate pair the member
        with the larger ix N + iy takes its partner's normals conjugated."""
        n, h = self.n, self.n // 2
        ix = torch.arange(h, device="cuda")[:, None, None]
        iy = torch.arange(n, device="cuda")[None, :, None]
        kz = torch.arange(h + 1, device="cuda")[None, None, :]
        c0 = (kz * n + iy) * h + ix
        i = torch.arange(n, device="cuda")
        j = (n - i) % n
        lin = i[:, None] * n + i[None, :]
        par = j[:, None] * n + j[None, :]

        def one(c):
            x = philox(c0, sweep, 1, c, self.seed)
            ga, gb = normals(x[0], x[1]), normals(x[2], x[3])
            g = torch.cat([torch.complex(*ga), torch.complex(*gb)], dim=0)
            for z in (0, h):
                p = g[:, :, z]
                p = torch.where(par < lin, p[j][:, j].conj(), p)
                g[:, :, z] = torch.where(par == lin, math.sqrt(2.0) * p.real + 0j, p)
            return g
        return self.each(one)

    def messenger(self, s, sweep):
        tau = self.tau[:, None, None, None]
        a = 1.0 - self.omw
        return a * s + self.beta + (tau * a).sqrt() * self.messenger_normals(sweep)

    def signal(self, th, p, sweep):
        f = p / (p + self.tau[:, None])
        v = self.m * self.tau[:, None] * f
        return self.per_mode(f) * th + self.per_mode((0.5 * v).sqrt()) * self.signal_normals(sweep)

    def gibbs(self, s, p, sweep):
        sh = self.signal(self.fft(self.messenger(s, sweep)), p, sweep)
        sigma = self.per_bin(sh.real ** 2 + sh.imag ** 2).cpu().numpy()
        new = p.cpu().numpy().copy()
        ok = self.count > 0
        for c in range(self.chains):
            g = np.array([gamma(0.5 * k, b, c, sweep, self.seed)
                          for b, k in enumerate(self.count) if k > 0])
            new[c, ok] = (sigma[c, ok] + 2 * self.m * self.b0) / (2 * self.m * g)
        return self.ifft(sh), torch.from_numpy(new).cuda()

    def mixing(self, s, p, sweep):
        th = self.fft(self.messenger(s, sweep))
        sh = self.signal(th, p, sweep)
        root = (self.m * p).sqrt()
        h1 = self.per_bin(sh.real ** 2 + sh.imag ** 2) / root ** 2
        h2 = self.per_bin(sh.real * th.real + sh.imag * th.imag) / root
        h1, h2, u, new = (v.cpu().numpy().copy() for v in (h1, h2, root, p))
        ratio = np.ones_like(new)
        tau = self.tau.cpu().numpy()
        for c in range(self.chains):
            for b in range(self.nb):
                if not (self.count[b] > 0 and h1[c, b] > 0):
                    continue
                mean, sd = h2[c, b] / h1[c, b], math.sqrt(self.m * tau[c] / h1[c, b])
                un, um = truncated(mean, sd, b, c, sweep, self.seed)
                if un is None:
                    continue
                lr = math.log(u[c, b] / un) + self.m * self.b0 * (u[c, b] ** -2 - un ** -2)
                if math.log(um) <= lr:
                    new[c, b], ratio[c, b] = un * un / self.m, un / u[c, b]
        sh = sh * self.per_mode(torch.from_numpy(ratio).cuda())
        return self.ifft(sh), torch.from_numpy(new).cuda()

    def start(self):
        p = np.stack([0.1 * bin_spectrum(self.n, self.nb) / self.vcell] * self.chains)
        return torch.zeros_like(self.d), torch.from_numpy(p).cuda()


def gamma(a, b, chain, sweep, seed):
    """Marsaglia and Tsang's Gamma(a, 1) of bin b."""
    d = (a + 1.0 if a < 1.0 else a) - 1.0 / 3.0
    boost = 1.0
    for j in range(1 << 16):
        w = [int(v) for v in philox(np.int64(b * 65536 + j), sweep, 2, chain, seed)]
        if j == 0 and a < 1.0:
            boost = uniform(w[3]) ** (1.0 / a)
        z = normals(np.int64(w[0]), np.int64(w[1]))[0]
        v = (1.0 + z / math.sqrt(9.0 * d)) ** 3
        if v > 0 and math.log(uniform(w[2])) < 0.5 * z * z + d - d * v + d * math.log(v):
            return d * v * boost
    return -1.0


def truncated(mean, sd, b, chain, sweep, seed):
    """(a draw of N(mean, sd^2) given > 0, or None; the acceptance uniform)."""
    a = -mean / sd
    r = 0.5 * (a + math.sqrt(a * a + 4.0))
    um = 1.0
    for j in range(64):
        w = [int(v) for v in philox(np.int64(b * 65536 + j), sweep, 3, chain, seed)]
        if j == 0:
            um = uniform(w[3])
        if a <= 0.5:
            z = float(normals(np.int64(w[0]), np.int64(w[1]))[0])
            ok = z > a
        else:
            z = a - math.log(uniform(w[0])) / r
            ok = uniform(w[1]) <= math.exp(-0.5 * (z - r) ** 2)
        if ok:
            return mean + sd * z, um
    return None, um


def exact(case, seed):
    kind = case["kind"]
    if kind == "acf":
        x = prepare(case, seed)["trace"]
        t = case["t"]
        x = x - x.mean(dim=0)
        f = torch.fft.rfft(x, n=2 * t, dim=0)
        c = torch.fft.irfft(f.real ** 2 + f.imag ** 2, n=2 * t, dim=0)[:case["lag"] + 1]
        pairs = t - torch.arange(case["lag"] + 1, device="cuda", dtype=torch.float64)
        return c / pairs[:, None] / (x * x).mean(dim=0), None
    problems = mocks(case, seed)
    if kind == "session":
        n, chains = problems[0]
        e = Exact(case, n, chains, seed)
        s, p = e.start()
        for i in range(case["sweeps"]):
            s, p = e.gibbs(s, p, i)
        return s[0], p[0] * e.vcell
    if kind in ("wiener", "logdet"):
        n, chains = problems[0]
        e = Exact(case, n, chains, seed)
        squeeze = (lambda v: v[0]) if len(chains) == 1 else (lambda v: v)
        pk = torch.from_numpy(np.stack([bin_spectrum(n, case["bins"])] * len(chains))).cuda()
        iters = case["iters"]
        safe = torch.where(e.seen, e.nv, 1.0)
        tau = e.tau[:, None, None, None]

        def filtered(pk, beta):
            f = e.per_mode((pk / e.vcell) / (pk / e.vcell + e.tau[:, None]))
            s = torch.zeros_like(beta)
            for _ in range(iters):
                s = e.ifft(f * e.fft((1.0 - e.omw) * s + beta))
            return s
        if kind == "wiener":
            pk.requires_grad_()
            d = e.d.clone().requires_grad_()
            s = filtered(pk, torch.where(e.seen, tau * e.r * d / safe, 0.0))
            chi2 = torch.where(e.seen, d * (d - e.r * s) / safe, 0.0).sum(dim=(1, 2, 3))
            gp, gd = torch.autograd.grad(chi2.sum(), (pk, d))
            return squeeze(chi2.detach()), squeeze(gp), squeeze(gd)
        total = 0.0
        c0 = torch.arange(n ** 3 // 4, device="cuda")
        for j in range(case["probes"]):
            xi = e.each(lambda c: (1.0 - 2.0 * (torch.stack(philox(c0, j, 4, c, seed), 1) >> 31))
                        .double().view(n, n, n))
            z = torch.where(e.seen, torch.sign(e.r) * safe.sqrt() * xi, 0.0)
            s = filtered(pk, torch.where(e.seen, tau * e.r * z / safe, 0.0))
            a = e.fft(torch.where(e.seen, e.r * (z - e.r * s) / safe, 0.0))
            b = e.fft(torch.where(e.seen, e.r * z / safe, 0.0))
            total = total + e.per_bin((a.real * b.real + a.imag * b.imag) / e.m)
        return squeeze(total / case["probes"] / e.vcell)
    out = []
    for i, (n, chains) in enumerate(problems):
        e = Exact(case, n, chains, seed + i)
        s, p = e.start()
        for k in range(case["sweeps"]):
            if k == case["sweeps"] - 1:
                trace, mean = (p * e.vcell)[:, None], s
            s, p = (e.mixing if kind == "mixing" else e.gibbs)(s, p, k)
        one = (lambda v: v[0]) if len(chains) == 1 else (lambda v: v)
        out.append((trace, [one(mean), one(torch.zeros_like(mean))]))
    return out
