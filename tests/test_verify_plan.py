"""Verify attention's launch plan, run without a GPU over its sizes, against
what the built kernels reserve (not gpu)."""
import os
import re
import subprocess

import pytest

import code_objects

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAVE_REGISTERS = 512   # vector registers of a SIMD lane, shared by its waves
SIMDS = 4
LDS = 160 * 1024


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "verify_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2603_19610_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan", "verify_plan_check.cpp"), "-o", exe], check=True)

    def run(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout
    return run


def _part_kernels():
    """(type, D, row tiles, registers, fixed LDS, is the mass kernel)."""
    out = []
    for name, (regs, lds) in code_objects.kernels().items():
        m = re.search(r"verify_(part|mass)_kernelINS\w_\d(Bf16|F32)ILi(\d+)EEELi(\d+)E", name)
        if m:
            out.append((m[2], int(m[3]), int(m[4]), regs, lds, m[1] == "mass"))
    return out


def _resident(D, rt, regs, lds, mass):
    """Workgroups of a compute unit that registers and LDS admit."""
    waves = rt * (2 if rt <= 2 else 1) + 2
    most = WAVE_REGISTERS // regs * SIMDS // waves
    ring = 4 * 2 * 64 * D * 2 // (2 if mass else 1)  # (fp32: half as many tokens of twice the bytes)
    return min(most, LDS // (ring + lds))


def test_plan_counts_on_resident_workgroups_only(check):
    """The registers that the waves-per-SIMD attribute makes a kernel reserve
    count, not those it uses: a plan that took two D = 64 workgroups per
    compute unit where one fits would let a captured call wait for workgroups
    that cannot start."""
    kernels = _part_kernels()
    assert len(kernels) > 100 and {k[2] for k in kernels} == set(range(1, 10))
    fit = {k: _resident(*k[1:]) for k in kernels}
    assert min(fit.values()) >= 1, [k for k, v in fit.items() if v < 1]
    check("resident", min(fit.values()))


def test_plan_runs_in_one_round(check):
    """Chunks are as long as it takes for every group's chunks to fit the
    device together: one workgroup too many doubles the launch's time."""
    check("round")


def test_plan_fits_its_workspace(check):
    check("areas")


def test_finish_grid_stays_within_a_launch(check):
    check("finish")


def test_workspace_size_holds_under_every_budget(check):
    """pvlm_verify_attn_workspace_size knows no stream: its answer has to do on
    streams with any compute-unit budget."""
    check("sized")


def test_bench_names_the_plan_the_library_picks(check):
    import sys
    sys.path.insert(0, ROOT)
    import bench
    import workloads as W
    for name, w in W.WORKLOADS.items():
        got = check("show", int(w.dtype == "bf16"), w.batch, w.T, w.hq, w.hkv, w.head_dim, w.n_cap(),
                    int(w.lengths().max()))
        assert tuple(map(int, got.split())) == bench.verify_plan(w)[:4], name
    assert bench.verify_kernel_label(W.WORKLOADS["llava72b"]) == \
        "verify_part_kernel<Bf16<128>,5,7> + verify_finish_kernel<Bf16<128>>"
