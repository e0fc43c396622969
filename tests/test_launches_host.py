"""What the library's host code launches, on a machine without a GPU: libfr.so
runs against a stand-in for the HIP runtime (hip_stand_in.cpp) that logs the
kernels and gives each a time by its name.  Each scenario is a program of its
own, so that the stand-in never meets a real runtime."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = textwrap.dedent(r"""
    import ctypes, os, re, sys
    import numpy as np
    S = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    S.stand_in_log.restype = ctypes.c_char_p
    S.stand_in_cost.argtypes = S.stand_in_cold.argtypes = [ctypes.c_char_p, ctypes.c_double]
    from paper_1409_0405_amd import frlib, inputs

    INTERP = r"opmul\w*kernelIf?Li[0-9]+E(Lb[01]E)?Li(0|4|8)E"    # products of tag 4 * type + operator
    DIV = r"opmul\w*kernelIf?Li[0-9]+E(Lb[01]E)?Li(3|7|11)E"

    def costs(us={}, **more):
        # one microsecond per launch and these on top, by a part of the name
        S.stand_in_clear()
        for name, t in dict(us, **more).items():
            S.stand_in_cost(name.encode(), t)

    def log():
        # [(device, blocks, kernel)] since the last costs()
        rows = [l.split(" ", 2) for l in S.stand_in_log().decode().splitlines()]
        return [(int(a), int(b), c) for a, b, c in rows]

    def mixed(n=3):
        return inputs.small_mixed_box(nxy=n, n_pri_layers=3, n_tet_layers=3, jitter=0.1, seed=2)

    def buffers(m):
        # 64-byte aligned host arrays as the states of every type
        keep, out = [], []
        for t in range(3):
            q = m.query(t)
            n = q["nupts"] * 5 * q["ld"] if q["nelem"] else 0
            a = np.zeros(n + 16)
            keep.append(a)
            out.append((a.ctypes.data + 63) // 64 * 64 if n else 0)
        return keep, out

    def rhs(m):
        (k1, u), (k2, r) = buffers(m), buffers(m)
        m.rhs(u, r)
""")


@pytest.fixture(scope="session")
def stand_in(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("hip") / "hip_stand_in.so")
    subprocess.run([cxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_stand_in.cpp"), "-o", out],
                   check=True)
    return out


def _run(stand_in, body):
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), stand_in], env=env,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


@pytest.mark.parametrize("prec", ("split_bf16", "split_fp16"))
def test_separate_gradient_kernels_run_stage_by_stage(stand_in, prec):
    """The gradient products of every type come before the first point-wise
    kernel: they share what the common solution just wrote in the caches."""
    _run(stand_in, f"""
        m = frlib.Mesh(mixed(), 4, system="ns", precision="{prec}", mu=0.02)
        costs()
        rhs(m)
        kinds = []
        for _, _, k in log():
            tag = re.search(r"opmul_split\\w*kernelILi\\d+ELb[01]ELi(\\d+)E", k)
            if tag and int(tag[1]) % 4 == 1:
                kinds.append("gradient")
            elif "upts_kernel" in k:
                kinds.append("upts")
        assert kinds == ["gradient", "gradient", "upts", "upts"], kinds
    """)


TUNED = """
    def chosen(report, kind):
        return re.search(kind + r" stage: [^;]*, (\\w+);", report)[1]

    def step(m):
        # the kernels of one step, after the first stage's interpolation
        (k, u) = buffers(m)
        for t in range(3):
            if m.query(t)["nelem"]:
                m.set_solution(t, u[t])
        S.stand_in_clear()
        m.rk_step(frlib.FR_RK45_2RP, 1e-3, 1)
        return [k for _, _, k in log()]
"""


def test_autotuner_times_the_fused_gradient_stage_with_the_divergence_product(stand_in):
    """Fused gradient stage without the volume part, divergence as a product:
    the fastest form of large tetrahedral meshes at order 4."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent("""
        m = frlib.Mesh(mixed(), 4, system="ns", precision="fp32", mu=0.02)
        costs(gradflux_small=50.0, gradflux_stream=50.0)
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "fused", report
        ks = step(m)
        assert any("gradflux_kernel" in k for k in ks) and not any("divtile" in k for k in ks), ks
    """))


@pytest.mark.parametrize("system", ("ns", "euler"))
def test_tuning_again_compares_everything_again(stand_in, system):
    """A form that lost, or was switched off by a forced product, is back in
    the next comparison."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent(f"""
        m = frlib.Mesh(mixed(), 3, system="{system}", precision="fp32", mu=0.02)

        def tiles():
            ks = step(m)
            return [any("divtile" in k for k in ks), sum("interptile" in k or bool(re.search(INTERP, k)) for k in ks)]

        costs(divtile=50.0)
        assert chosen(m.autotune(), "tet") != "tiles" and not tiles()[0]
        costs()
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "tiles", report
        want = tiles()
        assert want[0]
        for op in (0, 3):
            for t in (0, 1):
                m.set_blocking(t, op, 2, 0)
        assert not tiles()[0]
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "tiles", report
        assert tiles() == want, (tiles(), want)
    """))


def test_forms_are_timed_with_the_interpolation_that_runs(stand_in):
    """The forms without the divergence stage on tiles interpolate every
    stage's input: on tiles where that was found faster."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent("""
        m = frlib.Mesh(mixed(), 3, system="ns", precision="fp32", mu=0.02)
        costs({INTERP: 100.0}, divtile=20.0)
        report = m.autotune()
        for kind in ("tet", "pri"):
            assert re.search(kind + r" interp: [^;]*, tile;", report), report
            assert chosen(report, kind) == "fused", report
        assert not any(re.search(INTERP, k) for k in step(m))
    """))


def test_forms_are_timed_with_the_attached_closure(stand_in):
    """With the closure the divergence product is followed by the update
    kernel; the divergence stage on tiles applies the correction itself."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent("""
        m = frlib.Mesh(mixed(), 1, system="ns", precision="fp32", mu=0.02)
        net = frlib.MLP(0)
        stats = np.ones(280, np.float32)
        m.closure_attach(net, stats.ctypes.data)
        costs(negdivconf=100.0, divtile=20.0)
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "tiles", report
        m.closure_attach(None)
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "fused", report
    """))


def test_tuning_stays_out_of_the_per_kernel_timing(stand_in):
    _run(stand_in, """
        m = frlib.Mesh(mixed(), 2, system="ns", precision="fp32", mu=0.02)
        m.profile(True)
        rhs(m)
        m.autotune()
        counts = {k: n for k, (_, n) in m.profile_read().items() if n}
        assert counts["common_flux"] == counts["gradflux_tet"] == counts["div_pri"] == 1, counts
    """)


def test_small_meshes_are_tuned_as_they_run(stand_in):
    """The tiles of every type share a launch on a small mesh: cheaper than
    the sum of the types alone, and than their fastest forms alone."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent("""
        m = frlib.Mesh(mixed(), 3, system="ns", precision="fp32", mu=0.02)
        # a type alone: tiles 6 + 2, fused 1 + 1 + 3 (+ the interpolation's 1);
        # both types: tiles 6 + 2 in all, fused twice 6
        costs({DIV: 2.0}, gradflux_small=5.0, gradflux_stream=50.0, divtile=1.0)
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "tiles", report
        ks = step(m)
        assert any("divtile_small" in k for k in ks) and not any(re.search(DIV, k) for k in ks), ks
        # and not where it costs more
        costs({DIV: 2.0}, gradflux_small=20.0, gradflux_stream=50.0, divtile=1.0)
        report = m.autotune()
        assert chosen(report, "tet") == chosen(report, "pri") == "fused", report
    """))


@pytest.mark.parametrize("box,order,system,prec", [("mixed(3)", 4, "ns", "fp32"), ("mixed(3)", 4, "ns", "fp64"),
                                                   ("mixed(16)", 4, "ns", "fp32"), ("inputs.hex_box(4)", 4, "euler", "fp32"),
                                                   ("inputs.hex_box(4)", 4, "ns", "fp64"),
                                                   ("inputs.hex_box(17)", 4, "ns", "fp32"),
                                                   ("inputs.hex_box(17)", 3, "euler", "fp64")])
def test_every_device_of_a_process_gets_the_lds_limit(stand_in, box, order, system, prec):
    """A kernel's limit on dynamic LDS belongs to the device that it was
    raised on: meshes on two devices, in turn."""
    _run(stand_in, f"""
        box = {box}
        for device in (0, 1, 0, 2):
            S.stand_in_device(device)
            m = frlib.Mesh(box, {order}, system="{system}", precision="{prec}", mu=0.02)
            costs()
            rhs(m)
            assert {{d for d, _, _ in log()}} == {{device}}
            if "{system}" == "ns" and "{prec}" == "fp32" and m.query(0)["nelem"]:
                for t in (0, 1):
                    m.set_gradient_form(t, 2)
                rhs(m)
            m.close()
    """)


def test_products_that_tie_alone_are_decided_by_the_stage(stand_in):
    """A variant that is a little slower on its own, where its input is in the
    caches, and faster behind the kernels of a stage."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent("""
        m = frlib.Mesh(mixed(), 4, system="ns", precision="split_bf16", mu=0.02)
        costs({r"opmul_split_kernel": 0.05, r"opmul_split_lds_kernel": 0.0})
        S.stand_in_cold(DIV.replace("w*", "w*lds_").encode(), 3.0)
        report = m.autotune()
        for kind in ("tet", "pri"):
            assert re.search(kind + r" op3 cap \\d stage 0", report), report
            assert re.search(kind + r" op1 cap \\d stage 1", report), report
        ks = [k for k in step(m) if re.search(DIV, k)]
        assert ks and not any("lds" in k for k in ks), ks
    """))


@pytest.mark.parametrize("us", (-3.0, -1.0))
def test_tuning_survives_times_that_are_not_positive(stand_in, us):
    """Two event times of different clock corrections can lie a few
    microseconds the wrong way round; so can every time of a variant."""
    _run(stand_in, textwrap.dedent(TUNED) + textwrap.dedent(f"""
        for prec in ("fp32", "fp64", "split_bf16"):
            m = frlib.Mesh(mixed(), 2, system="euler", precision=prec)
            costs({{"opmul": {us}}})
            report = m.autotune()
            assert re.search(r"pri op3 cap \\d stage \\d", report), report
            rhs(m)
            m.close()
    """))


@pytest.mark.parametrize("scheme", ("FR_RK45_2RP", "FR_RK4", "FR_FWD_EULER"))
def test_batches_launch_every_step(stand_in, scheme):
    """No step is replayed from an earlier call, and the groups take turns
    step by step; side by side or one after the other, a step is the same
    launches."""
    _run(stand_in, f"""
        B = frlib.Batch([(mixed(), 2), (mixed(), 4), (mixed(2), 2)], system="euler", precision="fp32")
        def step(n):
            S.stand_in_clear()
            B.rk_step(frlib.{scheme}, n)
            return [k for _, _, k in log()]
        costs()
        want = step(1)
        assert want and step(1) == want and step(3) == 3 * want
        B.set_graph(False)
        assert step(1) == want
        B.set_graph(True)
        assert step(2) == 2 * want
        B.close()
    """)
