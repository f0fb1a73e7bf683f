"""The library's host code end to end on the CPU, under AddressSanitizer and
UndefinedBehaviorSanitizer: every host source linked against stand-ins of the
HIP calls and kernel launchers (tests/sanitize/hip_standin.cpp), which check
the lifetime of each stream, event, graph and allocation and run queued work
in any order that the waits between streams allow.  The cases are in
tests/sanitize/standin_check.cpp; products are the oracle's within 1e-12 * B
(FP64) or 2e-5 * B (FP32), B the oracle's product in absolute values."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import h2gen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2109_05451_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "sanitize")
HOST = ["h2_api.cpp", "h2_batch.cpp", "h2_compress.cpp", "h2_parse.cpp", "h2_plan.cpp", "h2_server.cpp",
        "h2_noalloc.hip"]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("standin")
    gxx, gcc = shutil.which("g++"), shutil.which("gcc")
    if gxx is None or gcc is None:
        pytest.skip("g++ or gcc not found")
    san = ["-O1", "-g", "-fPIC", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-fno-omit-frame-pointer"]
    cxx = [gxx, "-std=c++17", *san, "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
           "-DHIP_SYMBOL(x)=x", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-x", "c++"]
    jobs = [cxx + ["-c", os.path.join(CSRC, f), "-o", str(tmp / (f + ".o"))] for f in HOST]
    jobs += [cxx + ["-c", os.path.join(HERE, f), "-o", str(tmp / (f + ".o"))]
             for f in ("hip_standin.cpp", "standin_check.cpp")]
    jobs.append([gcc, "-std=c99", *san, "-c", os.path.join(ROOT, "oracle", "h2_oracle.c"), "-o",
                 str(tmp / "h2_oracle.o")])
    with ThreadPoolExecutor(4) as pool:
        done = list(pool.map(lambda c: subprocess.run(c, capture_output=True, text=True), jobs))
    for r in done:
        if r.returncode != 0:
            assert "hip_runtime.h: No such file" in r.stderr or "cannot find" in r.stderr, r.stderr[-2000:]
            pytest.skip("sanitized host build unavailable")
    out = str(tmp / "standin_check")
    r = subprocess.run([gxx, *san, *sorted(str(p) for p in tmp.glob("*.o")), "-o", out, "-lpthread", "-lm"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out


def run(exe, tmp_path, case, reps):
    files = []
    for i, b in enumerate(reps):
        path = tmp_path / f"{i}.h2"
        np.asarray(b).tofile(path)
        files.append(str(path))
    r = subprocess.run([exe, case, *files], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith(case + " ok"), (r.stdout + r.stderr)[-3000:]


def reps(seeds=range(8)):
    """Small operators of any shape (ranks, arity, depth, empty leaves, one or
    two bases), a built one and one with rows of more than 64 outputs."""
    out = [h2gen.random_rep(100 + i, q=1 + i % 6, max_children=1 + i % 3, max_leaf=2 + i % 9, max_rank=1 + i % 5,
                            separate=bool(i % 2), integer=False) for i in seeds]
    out.append(np.array(h2gen.build(h2gen.points(300, 2, 5), 8, 2, 0.7, "exp", 0.1).array, copy=True))
    out.append(h2gen.random_rep(124, q=2, max_children=2, max_leaf=70, ranks=([66] * 3, [66] * 3), p_adm=0.3,
                                integer=False, allow_empty=False))
    return out


def test_products(exe, tmp_path):
    run(exe, tmp_path, "products", reps())


def test_graph_replays(exe, tmp_path):
    run(exe, tmp_path, "graphs", reps(range(1, 8, 3)))


def test_growing_workspace_drops_graphs(exe, tmp_path):
    run(exe, tmp_path, "growth", reps(range(2, 5)))


def test_graphs_of_a_destroyed_stream(exe, tmp_path):
    run(exe, tmp_path, "streams", reps(range(2, 3)))


def test_batch_tuned_while_a_replay_is_queued(exe, tmp_path):
    run(exe, tmp_path, "batch", reps()[:-1])


def test_fp32_input_copy_only_where_read(exe, tmp_path):
    run(exe, tmp_path, "fp32", reps()[:-1])


def test_load_where_memory_is_short(exe, tmp_path):
    run(exe, tmp_path, "memory", [h2gen.random_rep(5, q=5, max_children=2, max_leaf=6, max_rank=5, p_adm=0.3,
                                                   separate=s, integer=False) for s in (False, True)])


def test_recompression_where_memory_is_short(exe, tmp_path):
    # mostly dense blocks: the new handle is larger than the scratch
    run(exe, tmp_path, "compress_memory", [h2gen.random_rep(3, q=1, max_children=40, max_leaf=255, max_rank=2,
                                                            p_adm=0.02, integer=False, allow_empty=False)])


def test_composed_stages_fit_a_launch(exe, tmp_path):
    run(exe, tmp_path, "split_rows", reps(range(1)))


def test_profiled_products_run_the_same_launches(exe, tmp_path):
    run(exe, tmp_path, "profile", reps())
