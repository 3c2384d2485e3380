"""The library's host code on a stand-in for the HIP runtime
(hip_host_model.cpp): which device its launches go to, what its pinned
staging holds while other work is on its way, and the shapes it launches.
No GPU: each scenario runs in a process of its own, in which the stand-in's
symbols come before the real runtime's."""
import ctypes as C
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    from paper_2103_09642_amd import edupic
    if not os.path.exists(edupic.LIB_PATH):
        from paper_2103_09642_amd import build
        build.build()
    so = str(tmp_path_factory.mktemp("model") / "model.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_2103_09642_amd", "csrc"), os.path.join(HERE, "hip_host_model.cpp"),
                    "-o", so], check=True)
    return so


def _scenario(model, name, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), model, name, *map(str, args)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


# ---------------------------------------------------------------------------
# In the scenarios' process
# ---------------------------------------------------------------------------
class Lib:
    """The library on the stand-in, without torch: contexts and cases by their handles."""

    def __init__(self, model):
        self.m = C.CDLL(model, mode=C.RTLD_GLOBAL)
        self.m.model_log.restype = C.c_char_p
        self.m.model_volt.restype = C.POINTER(C.c_double)
        self.m.model_step.restype = C.c_int64
        sys.modules["torch"] = None  # the binding then loads the library alone
        from paper_2103_09642_amd import edupic, workloads
        self.e, self.w, self.L = edupic, workloads, edupic.load()
        self.keep = []

    def ok(self, code):
        assert code == 0, (code, self.L.edp_last_error())

    def context(self, device=0, stream=None):
        h = C.c_void_p()
        self.ok(self.L.edp_create(C.byref(h), device, stream))
        ctx = self.e.Context.__new__(self.e.Context)
        ctx.h = h
        ctx.set_xsec(self.w.synthetic_xsec())
        self.keep.append(ctx)
        return ctx

    def stream(self):
        s = C.c_void_p()
        assert self.m.hipStreamCreateWithFlags(C.byref(s), 0) == 0
        return s

    def case(self, ctx, **kw):
        kw = dict(dict(n_init_e=500, n_init_i=500, n_grid=50, weight=10.0, cap_e=5000, cap_i=5000, pressure_pa=5.0,
                       flags=["allow_unstable"]), **kw)
        d = self.w.base_case(**kw)
        nbytes = ctx.case_bytes(d)
        arena = np.zeros(nbytes + 256, dtype=np.uint8)
        at = (arena.ctypes.data + 255) // 256 * 256
        i = C.c_int64()
        desc = self.e.make_desc(d)
        self.ok(self.L.edp_case_create(ctx.h, C.byref(desc), at, nbytes, C.byref(i)))
        c = self.e.Case.__new__(self.e.Case)
        c.ctx, c.case, c.ng, c.id, c.arena, c.at = ctx, d, d["n_grid"], i.value, arena, at
        self.keep.append(c)
        return c

    def advance(self, ctx, cases, steps):
        n = len(cases)
        return self.L.edp_advance_steps(ctx.h, (C.c_int64 * n)(*[c.id for c in cases]), n, (C.c_int64 * n)(*steps))

    def launches(self, name=""):
        out = []
        for line in self.m.model_log().decode().splitlines():
            f = line.split()
            if f[0] == "launch" and name in f[1]:
                out.append(dict([("name", f[1])] + [(k, int(v)) for k, v in (q.split("=") for q in f[2:])]))
        return out

    def volts(self, case, steps):
        """V(t_s) of steps 0 .. steps - 1 as the case's device memory holds it, and as it should be."""
        d = case.case
        want = np.zeros(steps)
        t = np.arange(steps) * d["dt_e"]
        for v, f, ph in d["harmonics"]:
            want += v * np.sin(2 * np.pi * f * t + ph)
        return np.ctypeslib.as_array(self.m.model_volt(C.c_void_p(case.at)), (steps,)), want

    def particles(self, case, sp, n):
        """The first n slots of a species' first buffer set."""
        at = (C.c_void_p * 6)()
        self.m.model_arrays(C.c_void_p(case.at), sp, at)
        out = {k: np.ctypeslib.as_array(C.cast(at[i], C.POINTER(C.c_double)), (n,)) for i, k in enumerate(("x", "vx", "vy", "vz"))}
        out["uid"] = np.ctypeslib.as_array(C.cast(at[4], C.POINTER(C.c_uint64)), (n,))
        if sp == 0:
            out["vp2"] = np.ctypeslib.as_array(C.cast(at[5], C.POINTER(C.c_float)), (n,)).astype(np.float64)
        return out


def scenario_device(lib):
    """A context on device 1 whose stream is the default one, called from a thread whose device is 0."""
    ctx = lib.context(device=1)
    g = lib.case(ctx, flags=["allow_unstable", "density", "eepf", "current", "meane", "xt", "ifed"])
    st = lib.w.random_state(300, 300, g.case["gap_m"], seed=1)
    calls = {"counts": g.counts, "deposit": g.deposit, "fields": g.fields, "density": lambda: g.density(reset=True),
             "eepf": g.eepf, "currents": g.currents, "mean_energy": g.mean_energy, "xt": lambda: g.xt("ne"),
             "ifed": g.ifed, "info": g.info, "reset_diag": g.reset_diag, "get_state": lambda: g.get_state(0),
             "set_state": lambda: g.set_state(0, st["e"], 5)}
    for name, call in calls.items():
        lib.m.hipSetDevice(0)
        lib.m.model_clear()
        call()
        assert all(q["dev"] == 1 for q in lib.launches()), (name, lib.launches())
        assert lib.m.model_device() == 0, f"{name} left another device current"
    # the default stream whose work ends before the memory is given back is device 1's
    lib.ok(lib.advance(ctx, [g], [7]))
    lib.m.hipSetDevice(0)
    lib.m.model_clear()
    ctx.close()
    waits = [line.split()[-1] for line in lib.m.model_log().decode().splitlines() if line.startswith("wait stream=0 ")]
    assert waits and set(waits) == {"dev=1"} and lib.m.model_device() == 0, waits


def scenario_small_failure(lib):
    """The second window of the persistent small cases cannot be launched."""
    ctx = lib.context(stream=lib.stream())
    ctx.set_option(lib.e.OPT_SMALL_MAX, 1 << 20)
    cases = [lib.case(ctx, seed=k) for k in range(2)]
    lib.m.model_fail(b"7k_small", 2)
    assert lib.advance(ctx, cases, [10_000] * 2) == lib.e.EDP_EHIP
    for g in cases:
        g.counts()
    lib.m.model_finish()
    for g in cases:
        got, want = lib.volts(g, 4096)
        assert np.allclose(got, want, rtol=1e-9, atol=1e-9)
    # and the context goes on
    lib.ok(lib.advance(ctx, cases, [50] * 2))


def scenario_read_beside_advance(lib, n_cases, small):
    """Another thread reads while the voltages of an advance are on their way to the device."""
    ctx = lib.context(stream=lib.stream())
    ctx.set_option(lib.e.OPT_SMALL_MAX, small)
    cases = [lib.case(ctx, seed=k) for k in range(n_cases)]
    readers = []

    def read():
        for g in cases:
            g.counts()
            g.deposit()
            g.get_state(0)

    @C.CFUNCTYPE(None)
    def hook():
        readers.append(threading.Thread(target=read))
        readers[0].start()
        readers[0].join(0.3)  # it may have to wait for this thread

    # an upload (the first copy is that of the workgroups' roles); small cases' by one launch
    lib.m.model_hook(b"k_small_volt" if small else b"copy from pinned", 1 if small else n_cases + 1, hook)
    lib.ok(lib.advance(ctx, cases, [6000] * n_cases))
    readers[0].join()
    lib.m.model_finish()
    for g in cases:
        got, want = lib.volts(g, 6000)
        assert np.allclose(got, want, rtol=1e-9, atol=1e-9)


def scenario_workgroups_per_cu(lib):
    """Threads of a full chip's launches (8 CUs, each with room for 1024 particle threads) by the option."""
    lib.m.model_cus(8)
    ctx = lib.context(stream=lib.stream())
    g = lib.case(ctx, n_init_e=30_000, n_init_i=30_000, cap_e=40_000, cap_i=40_000)
    for k in (0, 1, 2, 3, 4, 5, 7, 64):
        ctx.set_option(lib.e.OPT_PART_WG_PER_CU, k)
        lib.m.model_clear()
        lib.ok(lib.advance(ctx, [g], [1]))
        for q in lib.launches("11k_particles"):
            assert q["grid"] * q["block"] == 8 * 256 * (min(k, 4) or 4), (k, q)
        lib.m.model_finish()


def scenario_large_state(lib, n):
    """Waits for the stream in a state load of n particles; they arrive whole and in order."""
    ctx = lib.context(stream=lib.stream())
    g = lib.case(ctx, n_init_e=0, n_init_i=0, cap_e=n + 10, cap_i=n + 10)
    st = lib.w.random_state(n, n, g.case["gap_m"], seed=1)
    for sp, key in ((0, "e"), (1, "i")):
        lib.m.model_clear()
        g.set_state(sp, st[key], 5)
        assert lib.m.model_log().count(b"wait") <= 12, lib.m.model_log()
        have = lib.particles(g, sp, n)
        for k in ("x", "vx", "vy", "vz", "uid"):
            assert np.array_equal(have[k], st[key][k]), k
        if sp == 0:
            v2 = st[key]["vy"] ** 2 + st[key]["vz"] ** 2
            assert np.all(have["vp2"] >= v2) and np.all(have["vp2"] <= v2 * (1 + 2.0 ** -22))


def scenario_side_by_side(lib, n_cases, steps, own_stream, most):
    """The waits between streams of a call, and that the caller's stream is behind all of its work."""
    stream = lib.stream() if own_stream else None
    ctx = lib.context(stream=stream)
    cases = [lib.case(ctx, seed=k) for k in range(n_cases)]
    for call in (1, 2):
        lib.m.model_clear()
        lib.ok(lib.advance(ctx, cases, [steps + k // 2 for k in range(n_cases)]))
        log = lib.m.model_log()
        assert log.count(b"order") <= most, log.decode()
        assert len({q["stream"] for q in lib.launches("11k_particlesILi0")}) >= 2
        # the runtime was asked for the groups' occupancies in the first call
        assert call == 1 or b"occupancy" not in log, log.decode()
        # the first group's steps do not wait for the second's voltages
        assert log.index(b"k_particles") < log.rindex(b"upload")
        assert lib.m.hipStreamSynchronize(stream) == 0
        for k, g in enumerate(cases):
            assert lib.m.model_step(C.c_void_p(g.at)) == call * (steps + k // 2)


def scenario_distinct_schedules(lib):
    """Launch shapes of two cases that fill the chip under each candidate of the benchmark's tuner."""
    from paper_2103_09642_amd import tune
    lib.m.model_cus(8)
    ctx = lib.context(stream=lib.stream())
    cases = [lib.case(ctx, n_init_e=30_000, n_init_i=30_000, cap_e=40_000, cap_i=40_000, seed=k) for k in range(2)]

    def shapes(wg, groups):
        ctx.set_option(lib.e.OPT_PART_WG_PER_CU, wg)
        ctx.set_option(lib.e.OPT_GROUPS, groups)
        lib.m.model_clear()
        lib.ok(lib.advance(ctx, cases, [1, 1]))
        lib.m.model_finish()
        return tuple(sorted((q["grid"], q["block"]) for q in lib.launches("11k_particlesILi0")))

    every = [(w, g) for w in tune.DISTINCT_WG_CANDIDATES for g in tune.DISTINCT_GROUP_CANDIDATES]
    assert len({shapes(w, g) for w, g in every}) == len(every)
    for w in range(1, 9):  # and nothing but the single workgroup is left out
        assert w == 1 or any(shapes(w, 2) == shapes(v, 2) for v in tune.DISTINCT_WG_CANDIDATES)
    for g in range(1, 5):
        assert any(shapes(0, g) == shapes(0, h) for h in tune.DISTINCT_GROUP_CANDIDATES)


def scenario_wide_workgroups(lib):
    """Threads of the launches of the cases that the GPU tests of wide workgroups advance, on a chip of 256 CUs."""
    import test_gpu_edges as t
    lib.m.model_cus(256)
    ctx = lib.context(stream=lib.stream())
    n = 300_001
    for flags in (t.MEASURE, ["null_collision"], t.MEASURE + ["null_collision"]):
        g = lib.case(ctx, n_init_e=n, n_init_i=n, n_grid=200, cap_e=n + 20_000, cap_i=n + 20_000, ion_subcycle=5,
                     flags=["allow_unstable"] + flags, **t.SURFACES)
        for wg, threads in ((0, 512), (1, 256)):
            ctx.set_option(lib.e.OPT_PART_WG_PER_CU, wg)
            lib.m.model_clear()
            lib.ok(lib.advance(ctx, [g], [5]))
            lib.m.model_finish()
            assert {q["block"] for q in lib.launches("11k_particles")} == {threads}


def scenario_measurement_limits(lib):
    """The largest measurement histograms a case may ask for beside 1000 nodes."""
    ctx = lib.context(stream=lib.stream())

    def accepts(**kw):
        try:
            return ctx.case_bytes(lib.w.base_case(n_grid=1000, **kw)) > 0
        except lib.e.EdpError as err:
            assert err.code == lib.e.EDP_EINVAL
            return False

    # electrons: 48 bytes a node with the xt arrays and 4 a bin, 51200 in all
    for n, ok in ((800, True), (801, False), (1056, False), (1057, False)):
        assert accepts(flags=["eepf", "xt"], n_eepf=n) == ok, n
    # ions: 40 bytes a node and 8 a pair of bins, 57344 in all
    for n, ok in ((2167, True), (2168, False), (2423, False), (2424, False)):
        assert accepts(flags=["ifed"], n_ifed=n) == ok, n


def scenario_small_case_limit(lib):
    """The path of a small case with every measurement by its grid (2000 EEPF bins: 48 bytes a node and 8000 of 40960),
    and the threads of its workgroup."""
    ctx = lib.context(stream=lib.stream())
    ctx.set_option(lib.e.OPT_SMALL_MAX, 1 << 20)
    for ng, small in ((400, 512), (543, 512), (544, 256), (686, 256), (687, 0), (793, 0), (1000, 0)):
        g = lib.case(ctx, n_grid=ng, n_eepf=2000 if ng < 800 else 100,
                     flags=["allow_unstable", "density", "eepf", "current", "meane", "xt", "ifed"])
        lib.m.model_clear()
        lib.ok(lib.advance(ctx, [g], [3]))
        lib.m.model_finish()
        assert [q["block"] for q in lib.launches("7k_small")] == [small] * bool(small), ng
        assert bool(lib.launches("11k_particles")) != bool(small), ng


def scenario_lds_granules(lib):
    """Workgroups of 256 per CU of electron launches with 48 bytes a node, 8000 of the EEPF and the kernel's 12360."""
    lib.m.model_cus(8)
    ctx = lib.context(stream=lib.stream())
    # three of 42 granules of 1280 bytes fit 160 KiB, three of 43 do not
    for ng, per_cu in ((690, 3), (695, 3), (696, 2), (713, 2), (714, 2), (740, 2)):
        g = lib.case(ctx, n_init_e=30_000, n_init_i=30_000, cap_e=40_000, cap_i=40_000, n_grid=ng,
                     flags=["allow_unstable", "density", "eepf", "current", "meane", "xt", "ifed"])
        lib.m.model_clear()
        lib.ok(lib.advance(ctx, [g], [1]))
        lib.m.model_finish()
        assert [(q["grid"], q["block"]) for q in lib.launches("11k_particlesILi0")] == [(8 * per_cu, 256)], ng


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    the_lib = Lib(sys.argv[1])
    globals()["scenario_" + sys.argv[2]](the_lib, *map(int, sys.argv[3:]))
    os._exit(0)  # contexts and arenas go with the process, in no order


# ---------------------------------------------------------------------------
# The tests
# ---------------------------------------------------------------------------
def test_reads_and_transfers_launch_on_the_contexts_device(model):
    """Reads and state transfers launch on their context's device, whichever
    is current in the calling thread, and leave that one current; closing the
    context waits for its own device."""
    _scenario(model, "device")


def test_a_failed_small_case_window_leaves_nothing_under_way(model):
    """An advance of small cases that fails between its windows has ended what
    it had launched: a read after it does not get into their voltages."""
    _scenario(model, "small_failure")


@pytest.mark.parametrize("n_cases,small", [(1, 0), (3, 0), (3, 1 << 20)], ids=["one", "side-by-side", "small"])
def test_a_read_beside_an_advance_leaves_its_voltages_alone(model, n_cases, small):
    """Reads and transfers use the memory the voltages are uploaded from: one
    from another thread waits for the upload."""
    _scenario(model, "read_beside_advance", n_cases, small)


def test_the_workgroup_option_gives_its_share_of_the_wave_slots(model):
    """EDP_OPT_PART_WG_PER_CU = k: k workgroups of 256 threads per CU, or as
    many threads in larger ones."""
    _scenario(model, "workgroups_per_cu")


@pytest.mark.parametrize("n", [10_240, 61_440, 61_441, 300_001])
def test_a_state_load_does_not_wait_chunk_by_chunk(model, n):
    """A load goes through the pinned staging in chunks, a wait each, only
    while that is the faster way."""
    _scenario(model, "large_state", n)


@pytest.mark.parametrize("n_cases,steps,own_stream,most", [(2, 5, 1, 2), (2, 3000, 1, 4), (4, 3000, 1, 8), (2, 5, 0, 4)])
def test_groups_side_by_side_wait_once_a_window(model, n_cases, steps, own_stream, most):
    """Two groups side by side wait for the caller's stream and it for them
    once a window, in a call of a few steps without a stream for each, and the
    first is under way before the second is prepared."""
    _scenario(model, "side_by_side", n_cases, steps, own_stream, most)


def test_the_benchmarks_tuner_tries_schedules_that_differ(model):
    """No two of the candidates that bench.py tunes over launch the same."""
    _scenario(model, "distinct_schedules")
    bench = open(os.path.join(ROOT, "bench.py")).read()
    assert "tune.DISTINCT_WG_CANDIDATES" in bench and "tune.DISTINCT_GROUP_CANDIDATES" in bench


def test_the_gpu_tests_of_wide_workgroups_launch_them(model):
    """Measurements, null collisions and surfaces run in workgroups of 512
    threads at the sizes of their tests, and of 256 by option."""
    _scenario(model, "wide_workgroups")


def test_the_limits_of_measurement_histograms_stand(model):
    """What a case may measure is a limit of the interface, not of how much
    LDS the kernels leave free."""
    _scenario(model, "measurement_limits")


def test_which_small_cases_run_in_one_workgroup(model):
    """Cases whose measurements leave the persistent kernel little LDS stay on
    the lockstep path, which is the faster one for them."""
    _scenario(model, "small_case_limit")


def test_a_launch_has_no_more_workgroups_than_the_lds_granules_hold(model):
    """LDS is given out in granules, which the runtime's occupancy does not
    count: a workgroup beyond what fits waits for a whole one to end."""
    _scenario(model, "lds_granules")
