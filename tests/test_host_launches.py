"""CPU tests of which kernels the library launches: tests/hip_stub.cpp stands in
for the HIP runtime in a child process, so no device is needed and no kernel
runs."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, os
import numpy as np
from paper_1402_1763_amd import binding
lib = binding.load()
stub = ctypes.CDLL(os.environ["HIP_STUB"])
stub.stub_log.restype = ctypes.c_char_p

def log():
    out = stub.stub_log().decode().splitlines()
    stub.stub_reset()
    return out

def problem(n, precision="fp32", chains=1, nb=8, sample_pk=True):
    desc = binding.make_desc(n, nb, 10.0 * n, 1, precision, sample_pk=sample_pk, n_chains=chains)
    size = binding.mf_workspace_bytes(desc)
    ws = np.zeros(size + 256, dtype=np.uint8)
    ptr = (ws.ctypes.data + 255) // 256 * 256
    one = np.ones((n, n, n))
    h = binding.mf_init_problem(desc, [one] * chains, [one] * chains, [np.ones(nb)] * chains, None, ptr, size, 0)
    problem.keep.append(ws)
    stub.stub_reset()
    return h
problem.keep = []

def names(lines):
    return [l.split(" grid ")[0] for l in lines]

def sweep(h, n, stream=0):
    return lib.mf_gibbs_sweep(ctypes.c_void_p(h), n, ctypes.c_void_p(stream))

def state(h):
    return lib.mf_get_chain_state(ctypes.c_void_p(h), 0, binding._dptr(np.zeros(1 << 22)), None, None, None)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    stub = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", stub], check=True)

    def go(body):
        env = dict(os.environ, LD_PRELOAD=stub, HIP_STUB=stub, PYTHONPATH=ROOT)
        res = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body)], cwd=ROOT, env=env,
                             capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-3000:]
        return res.stdout
    return go


@pytest.mark.parametrize("n,precision,nth", [(n, p, k) for n, p in ((16, "fp64"), (64, "fp32"), (96, "fp32"))
                                             for k in range(7)])
def test_a_run_cut_short_is_completed_by_the_next_call(run, n, precision, nth):
    """Launch `nth` of the 7 of a three-sweep run fails: the state call that
    follows launches what the field is owed (the column of the sweep it was in,
    the run's end) before it reads the field, once."""
    out = run(f"""
        h = problem({n}, "{precision}")
        sweep(h, 3)
        whole = names(log())
        assert len(whole) == 7 and [k.split("_")[0] for k in whole] == ["plane", "column"] * 3 + ["plane"]
        end = whole[-1]
        h = problem({n}, "{precision}")
        stub.stub_fail_launch({nth})
        assert sweep(h, 3) == binding.MF_E_DEVICE
        assert names(log()) == whole[:{nth}]
        # the first retry fails, too, unless nothing is owed: reported, and owed still
        if {nth} > 0:
            stub.stub_fail_launch(0)
            assert state(h) == binding.MF_E_DEVICE and log() == []
        assert state(h) == 0
        got = names(log())
        column = got[0] if {nth} % 2 == 1 and {nth} < 6 else None
        want = ([column] if column else []) + ([end] if {nth} > 0 else [])
        assert got[:-1] == want and got[-1].startswith("zpass_kernel"), (got, want)
        assert column is None or column.startswith("column_kernel")
        assert state(h) == 0 and len(log()) == 1       # nothing owed any more
        _, _, done = binding.mf_get_chain_state(h, 0, {n}, 8, 0, True)
        assert done == ({nth} + 1) // 2, done
    """)
    print(out)


def test_every_call_on_the_field_completes_a_run_first(run):
    """Sweeps, mixing sweeps, checkpoints and new states of one chain of several
    do so; a checkpoint into the only chain replaces the field instead."""
    run("""
        def broken(chains=1):
            h = problem(64, chains=chains)
            stub.stub_fail_launch(2)
            assert sweep(h, 3) == binding.MF_E_DEVICE
            log()
            return h
        end = "plane_kernel<float, 64, true, -1, false"
        h = broken(); sweep(h, 1); assert log()[0].startswith(end)
        h = broken(); assert lib.mf_mixing_sweep(ctypes.c_void_p(h), 1, None) == 0; assert log()[0].startswith(end)
        h = broken(); binding.mf_gibbs_sweep_timed(h, 1, 0); assert log()[0].startswith(end)
        h = broken(); blob = binding.mf_save_checkpoint(h, 0, 0); assert log()[0].startswith(end)
        h = broken(2); binding.mf_load_checkpoint(h, 1, blob, 0); assert log()[0].startswith(end)
        h = broken(1); binding.mf_load_checkpoint(h, 0, blob, 0); assert not any(l.startswith(end) for l in log())
        assert state(h) == 0 and len(log()) == 1
        h = broken(); binding.mf_set_chain_state(h, 0, None, np.ones(8), 5, 0); assert log()[0].startswith(end)
        h = broken(); binding.mf_debug_spectrum(h, 0, 64, stream=0); assert log()[0].startswith(end)
        h = broken(); g = binding.mf_graph_create([h], 0); log()
        binding.mf_graph_launch(g, 1, 0); assert log()[0].startswith(end)
        # not inside a capture, where every replay would repeat it
        h = broken(); stub.stub_caller_captures(1)
        assert sweep(h, 1, stream=8) == binding.MF_E_STATE and log() == []
    """)


def test_calls_on_the_scratch_and_the_records_complete_a_run_first(run):
    """The Wiener filter and the log-determinant use the P draw's partials as
    scratch, and new diagnostics would take an old sweep's records."""
    run("""
        end = "plane_kernel<float, 64, true, -1, false"
        def broken():
            h = problem(64)
            stub.stub_fail_launch(2)
            assert sweep(h, 3) == binding.MF_E_DEVICE
            log()
            return h
        def device(doubles):
            problem.keep.append(np.zeros(doubles + 64))
            return (problem.keep[-1].ctypes.data + 255) // 256 * 256
        field, bins = device(64 ** 3), device(8)
        h = broken()
        size = binding.mf_wiener_workspace_bytes(h, 0, 2, 1)
        ws = device(size // 8 + 1)
        binding.mf_wiener_forward(h, 0, field, bins, 2, 1, ws, size, bins, None, 0); first = log()[0]
        assert first.startswith(end), first
        stub.stub_fail_launch(2); assert sweep(h, 3) == binding.MF_E_DEVICE; log()
        binding.mf_wiener_backward(h, 0, field, ws, size, field, bins, 0); assert log()[0].startswith(end)
        h = broken()
        out = ctypes.c_size_t(0)
        assert lib.mf_wiener_logdet_workspace_bytes(ctypes.c_void_p(h), 0, ctypes.byref(out)) == 0
        ws = device(out.value // 8 + 1)
        assert lib.mf_wiener_logdet_trace(ctypes.c_void_p(h), 0, ctypes.c_void_p(bins), 2, 1, 0, ctypes.c_void_p(ws),
                                          out.value, ctypes.c_void_p(bins), None) == 0
        assert log()[0].startswith(end)
        h = broken()
        assert lib.mf_set_diagnostics(ctypes.c_void_p(h), ctypes.c_uint64(0), 1, ctypes.c_void_p(device(64)), 4, None, None) == 0
        assert log()[0].startswith(end)
    """)


def test_a_graph_launch_that_fails_counts_and_completes_its_sweeps(run):
    """The failing step of a launch of 10 sweeps: the first sweep's launches,
    replays of four, the sweep left over or the end."""
    run("""
        end = "plane_kernel<float, 64, true, -1, false"
        for nth in range(7):
            h = problem(64)
            g = binding.mf_graph_create([h], 0)
            log()
            stub.stub_fail_launch(nth)
            assert lib.mf_graph_launch(ctypes.c_void_p(g), 10, None) == binding.MF_E_DEVICE
            ran = sum("column" in l for l in log())
            assert ran == (0, 0, 1, 5, 9, 9, 10)[nth]
            assert state(h) == 0
            owed = names(log())[:-1]
            half = nth in (1, 5)                     # a column owed
            assert [k.startswith(end) for k in owed] == [False] * half + [True] * (nth > 0), (nth, owed)
            assert binding.mf_get_chain_state(h, 0, 64, 8, 0, False)[2] == ran + half
    """)


def test_what_a_graph_launch_replays_and_launches(run):
    """Several problems: pieces of a run are replayed, up to four further sweeps
    each, and sweeps that renew the gamma variates launched.  A single problem:
    four further sweeps are replayed, the others launched.  Every sweep is there
    once, on the path of the graph's making."""
    run("""
        def launch(g, n, of):
            binding.mf_graph_launch(g, n, 0)
            lines = log()
            assert sum("column" in l for l in lines) == of * n, (n, lines)
            assert sum(", true, -1, false" in l for l in lines) == of, (n, lines)       # the end
            assert sum("plane_kernel" in l and ", false, 0, true" in l for l in lines) == of    # the first sweep
            return "".join("g" if l == "graph" else l[0] for l in lines if l[0] != " ")
        a, b = problem(64), problem(48, chains=2)
        g = binding.mf_graph_create([a, b], 0)
        assert log() == []
        both = "pcpc"                                      # a sweep of both
        for n, want in ((1, "g"), (2, "g"), (4, "g"), (5, "gg"), (6, "gg"), (25, "g" * 7), (32, "g" * 8),
                        (33, "g" * 8 + both + "pp"), (40, "g" * 8 + both + "gg"), (1, "g")):
            assert launch(g, n, 2) == want, n
        assert lib.mf_set_x_path(ctypes.c_void_p(a), 0) == 0
        assert launch(g, 1, 2) == "g" and launch(g, 33, 2) == "g" * 8 + both + "pp"
        path = ctypes.c_int32(-1)
        lib.mf_get_x_path(ctypes.c_void_p(a), ctypes.byref(path))
        assert path.value == 0
        stub.stub_caller_captures(1)
        assert lib.mf_graph_launch(ctypes.c_void_p(g), 1, ctypes.c_void_p(8)) == binding.MF_E_DEVICE and log() == []
        stub.stub_caller_captures(0)
        h = problem(64)
        g = binding.mf_graph_create([h], 0)
        for n, want in ((1, "pcp"), (4, "pc" * 4 + "p"), (5, "pcgp"), (10, "pcggpcp"),
                        (40, "pc" + "g" * 7 + "pc" * 4 + "g" + "pc" * 3 + "p")):
            assert launch(g, n, 1) == want, n
        # moments of every fifth sweep: launched
        mom = np.zeros(2 * 64 ** 3)
        h, other = problem(64), problem(64)
        assert lib.mf_set_diagnostics(ctypes.c_void_p(h), ctypes.c_uint64(0), 5, None, 0,
                                      ctypes.c_void_p(mom.ctypes.data), None) == 0
        log()
        g = binding.mf_graph_create([h, other], 0)
        assert launch(g, 11, 2) == "gg" + both + "g" + both + "pp"
        # without the two-pass sweep there is no first sweep and no end
        h, other = problem(96, "fp64", 3), problem(64)
        assert lib.mf_set_x_path(ctypes.c_void_p(other), 0) == 0
        g = binding.mf_graph_create([h, other], 0)
        for n, graphs in ((1, 1), (4, 1), (7, 2), (40, 10)):
            binding.mf_graph_launch(g, n, 0)
            lines = log()
            assert lines.count("graph") == graphs and len(lines) == graphs + 8 * n
    """)


def test_a_path_chosen_is_the_path_run_timed_and_reported(run):
    """The default up to 128^3 is the two-pass sweep, reported as the whole path;
    the split path with its default tiles can be chosen, is reported with its
    geometry and is what the autotuner times against the whole path.  Setting
    what is reported changes nothing."""
    run("""
        def tuning(h):
            t = binding.mf_tuning()
            assert lib.mf_get_tuning(ctypes.c_void_p(h), ctypes.byref(t)) == 0
            path = ctypes.c_int32(-1)
            assert lib.mf_get_x_path(ctypes.c_void_p(h), ctypes.byref(path)) == 0
            assert path.value == t.x_path
            return t
        def choose(h, t):
            assert lib.mf_set_tuning(ctypes.c_void_p(h), ctypes.byref(t)) == 0
        def kinds(h):
            stub.stub_reset()
            assert sweep(h, 2) == 0
            return [k.split("_")[0] for k in names(log())]
        planes = ["plane", "column", "plane", "column", "plane"]
        split = ["zpass", "ysplit", "xsplit", "ysplit"] * 2
        for n, precision, chains, default in ((64, "fp32", 1, planes), (128, "fp32", 1, planes), (96, "fp64", 2, planes),
                                              (96, "fp64", 3, split), (16, "fp32", 1, planes)):
            h = problem(n, precision, chains)
            assert kinds(h) == default, (n, precision, chains)
            t = tuning(h)
            assert t.x_path == (0 if default is split else 1)
            assert (t.x_cols > 0) == (t.y_units > 0) == (default is split)
            choose(h, t)
            assert kinds(h) == default
            if n == 16:
                continue
            choose(h, binding.mf_tuning(x_path=0))
            t = tuning(h)
            assert t.x_path == 0 and t.x_cols > 0 and t.x_k1 > 0 and t.x_hist == 8 and t.y_units > 0
            assert kinds(h) == split
            choose(h, binding.mf_tuning(x_path=1))
            assert tuning(h).x_path == 1 and tuning(h).x_cols == 0 and kinds(h) == planes
        # four kernels one by one, in the split form, for a problem without a choice
        h = problem(64)
        for k in range(4):
            binding.mf_debug_run_kernel(h, k, 0, 0)
        assert [k.split("_")[0] for k in names(log())] == split[:4]
        # every x tile is timed on the split path, and planes for the whole path only
        h = problem(64)
        ms = (ctypes.c_double * 10)()
        assert lib.mf_autotune(ctypes.c_void_p(h), 5, None, ms, None) == 0
        runs = names(log())
        for v in range(3):
            assert sum(k == f"xsplit_kernel<float, 64, 0, {v}>" for k in runs) >= 18, v
        assert sum(k.startswith("column") for k in runs) == 3 * 6
    """)


def test_gamma_variates_are_computed_for_the_sweeps_that_use_them(run):
    """The workgroups of a run's first launch: the planes and as many more as the
    gamma variates of the run's sweeps take, at most 32 of them; recorded sweeps
    compute none, and every 32nd sweep those of the next.  The workgroups ahead of
    the planes (these, and one per bin of the P draw) come in eights."""
    run("""
        bins, nt = 300, 256                  # threads of a 64^3 FP32 plane
        wgs = lambda sweeps: -(-sweeps * bins // (8 * nt)) * 8
        nb = 304
        def first(h, n):
            sweep(h, n)
            return [int(l.split(" grid ")[1].split()[0]) for l in log() if l.startswith("plane")]
        h = problem(64, nb=bins)
        for n in (1, 3, 32, 33, 40):
            assert first(h, n)[0] == 64 + wgs(min(n, 32)), n
        grids = first(h, 70)
        assert grids[32] == 64 + nb + wgs(32) and grids[64] == 64 + nb + wgs(6)
        assert set(grids[1:32] + grids[33:64] + grids[65:]) == {64 + nb}
        mom = np.zeros(2 * 64 ** 3)
        assert lib.mf_set_diagnostics(ctypes.c_void_p(h), ctypes.c_uint64(0), 1, None, 0,
                                      ctypes.c_void_p(mom.ctypes.data), None) == 0
        log()
        assert first(h, 20)[1:] == [64 + nb] * 20
        assert first(problem(64, nb=bins, sample_pk=False), 3) == [64, 64 + nb, 64 + nb, 64 + nb]
    """)


def test_every_chain_starts_on_the_same_xcd(run):
    """Workgroups of the passes over planes come in eights per chain."""
    run("""
        for n, precision, nb in ((48, "fp32", 5), (80, "fp64", 9), (96, "fp64", 16), (128, "fp32", 33)):
            h = problem(n, precision, 3, nb)
            assert lib.mf_set_tuning(ctypes.c_void_p(h), ctypes.byref(binding.mf_tuning(x_path=0))) == 0
            sweep(h, 1)
            assert lib.mf_mixing_sweep(ctypes.c_void_p(h), 1, None) == 0
            assert lib.mf_set_tuning(ctypes.c_void_p(h), ctypes.byref(binding.mf_tuning(x_path=1))) == 0
            sweep(h, 3)
            for line in log():
                kernel, grid = line.split(" grid ")
                if kernel.startswith(("ysplit", "xsplit", "xmixinv", "plane")):
                    assert int(grid.split()[0]) % 8 == 0, line
    """)


def test_sweep_bytes_count_the_normals_drawn_ahead(run):
    """FP64 problems of at most 128 planes write and read one real per voxel more
    on the two-pass sweep, and only there."""
    run("""
        def nbytes(h):
            out = (ctypes.c_size_t * binding.MF_NUM_KERNELS)()
            assert lib.mf_sweep_bytes(ctypes.c_void_p(h), out) == 0
            return list(out)
        for n, precision, chains in ((32, "fp64", 1), (32, "fp64", 4), (32, "fp64", 5), (64, "fp32", 1), (64, "fp64", 2)):
            h = problem(n, precision, chains)
            rs, m = (8 if precision == "fp64" else 4), n ** 3
            spec = (n // 2 + 1) * n * n * 2 * rs
            two = nbytes(h)
            assert lib.mf_set_x_path(ctypes.c_void_p(h), 0) == 0
            four = nbytes(h)
            ahead = chains * m * rs if precision == "fp64" and n * chains <= 128 else 0
            assert two[0] - four[0] == ahead
            assert two[1] == 0 and four[1] == 2 * spec * chains
            # every launch that the bytes describe is there: a column kernel that draws ahead
            assert lib.mf_set_x_path(ctypes.c_void_p(h), 1) == 0
            log(); sweep(h, 2)
            assert any("column_kernel" in k and k.endswith("true>") for k in names(log())) == (ahead > 0)
    """)
