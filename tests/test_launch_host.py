"""Workspaces, memory accounting and launch shapes, checked on the host: a C++
program runs the library over a stand-in for the HIP runtime (host_runtime.cpp)
that records allocations and looks at every launch instead of running it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2609_16408_amd")
FP64, FP32 = 0, 1


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(PKG, "librpa_mi355x.so")):
        pytest.skip("needs a C++ compiler and the built library")
    exe = str(tmp_path_factory.mktemp("host") / "host_runtime")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "host_runtime.cpp"), "-L", PKG, "-lrpa_mi355x",
           "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib", "-rdynamic", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(*args):
        p = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert p.returncode == 0, (p.returncode, p.stdout, p.stderr)
        return p.stdout

    return run


# one and two systems, where a single FP64 slot may be longer than the FP32 slots
# together, and many; grids the marching solver takes (whole planes and 12-row tiles)
@pytest.mark.parametrize("n_occ,nvec", [(1, 1), (1, 2), (2, 1), (3, 20)])
@pytest.mark.parametrize("precond", [False, True])
@pytest.mark.parametrize("precision", [FP64, FP32])
@pytest.mark.parametrize("n", [(26, 27, 28), (13, 24, 48)])
def test_sternheimer_workspaces_lie_inside_their_allocation(host, n, precision, precond, n_occ, nvec):
    host("slots", *n, n_occ, nvec, precision, int(precond))


# one system, fewer systems than workgroups, and more
@pytest.mark.parametrize("n_occ,n_pts", [(1, 1), (2, 9), (16, 40)])
@pytest.mark.parametrize("window", [False, True])
@pytest.mark.parametrize("precision", [FP64, FP32])
def test_counted_workspace_is_what_a_job_allocates(host, precision, window, n_occ, n_pts):
    host("workspace", 24, 24, 20, n_occ, n_pts, 3, precision, int(window))


# grids on and off the padding of the transform matrices, and one beyond them
@pytest.mark.parametrize("precond,n_proj", [(False, 0), (True, 0), (False, 6)])
@pytest.mark.parametrize("n", [(16, 16, 16), (24, 17, 18), (130, 8, 9)])
def test_server_counts_what_a_worker_keeps(host, n, precond, n_proj):
    if precond and max(n) > 64:
        pytest.skip("the preconditioner needs dimensions of at most 64")
    host("resident", *n, 3, int(precond), n_proj)


# launches of one range; ranges of points (many start vectors of one orbital, a
# long grid) and of start vectors
@pytest.mark.parametrize("N,n_occ,ng,B", [(343, 1, 1, 1), (110592, 128, 512, 64), (110592, 1, 1, 39000), (110592, 33, 40, 50000),
                                          ((1 << 32) + 77, 1, 3, 2), (343, 1, 1, 1 << 25), (520, 17, 17, 1 << 25)])
def test_expansion_launches_stay_within_the_grid_limit(host, N, n_occ, ng, B):
    host("expand", N, n_occ, ng, B)


@pytest.fixture(scope="module")
def fixed_lds(tmp_path_factory):
    """Fixed LDS of every kernel of the built library, from its metadata."""
    tools = [os.path.join("/opt/rocm/llvm/bin", t) for t in ("llvm-objdump", "llvm-readelf")]
    if not all(map(os.path.exists, tools)):
        pytest.skip("needs the LLVM tools of ROCm")
    at = tmp_path_factory.mktemp("objects")
    shutil.copy(os.path.join(PKG, "librpa_mi355x.so"), at)
    subprocess.run([tools[0], "--offloading", "librpa_mi355x.so"], cwd=at, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(at)):
        if "gfx950" in f:
            notes = subprocess.run([tools[1], "--notes", f], cwd=at, check=True, capture_output=True, text=True).stdout
            for size, name in re.findall(r"\.group_segment_fixed_size: (\d+).*?\n    \.name: +(\S+)", notes, re.S):
                out[name] = int(size)
    return out


# whole planes and tiles on each LDS pitch, with the most projectors that setup accepts
@pytest.mark.parametrize("precond,window", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("precision", [FP64, FP32])
@pytest.mark.parametrize("n", [(7, 14, 53), (13, 27, 28), (9, 28, 48), (12, 28, 50)])
def test_accepted_problems_fit_the_local_memory(host, fixed_lds, n, precision, precond, window):
    fixed = max(v for k, v in fixed_lds.items() if "6k_cocgI" in k)
    lds = int(host("lds", *n, precision, int(precond), int(window)).split("lds ")[1].split()[0])
    assert lds + fixed <= 160 * 1024, (lds, fixed)


@pytest.mark.parametrize("precision", [FP64, FP32])
@pytest.mark.parametrize("n", [(24, 24, 24), (48, 48, 48), (17, 36, 20)])
def test_plain_stencil_launches_the_same_on_a_preconditioned_handle(host, n, precision):
    assert host("stencil", *n, precision, 1, 3) == host("stencil", *n, precision, 0, 3)


# few and many vectors of grids with small, large and several tiles
@pytest.mark.parametrize("precision,waves_per_cu", [(FP64, 16), (FP32, 24)])
@pytest.mark.parametrize("n,nvec", [((48, 48, 48), 65), ((48, 48, 48), 512), ((24, 24, 24), 65), ((128, 8, 8), 300), ((12, 12, 12), 64),
                                    ((9, 24, 72), 5), ((72, 72, 72), 31), ((7, 7, 7), 1), ((60, 30, 40), 65), ((60, 30, 40), 200)])
def test_stencil_split_takes_the_fewest_plane_steps(host, n, nvec, precision, waves_per_cu):
    """A march split along x repeats 12 halo planes per segment: the launch takes
    the fewest steps of rounds times planes among the splits of up to two rounds."""
    f = host("stencil", *n, precision, 0, nvec).split()
    x, y, z, block, lds = int(f[1]), int(f[2]), int(f[3]), int(f[5]), int(f[7])
    fit = 256 * max(1, min(waves_per_cu // (block // 64), 160 * 1024 // lds))

    def steps(k):
        return -(-x * y * k // fit) * (-(-n[0] // k) + 12)

    allowed = [k for k in range(1, n[0] + 1) if k == 1 or x * y * k <= 2 * fit]
    assert z in allowed and steps(z) == min(map(steps, allowed))
