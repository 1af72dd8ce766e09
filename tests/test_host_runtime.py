"""The stage runtime's host logic on the CPU (no GPU): the message admission of Alg. 2's receive loop, the stash
slots under pipeline_limit (Sec. 3.3), duplicate / surplus messages, the per-wait time limit, the weight-gradient
groups, the optimizer's bucket plan (Sec. 5.2) and the chunk -> lowest-layer gate of the overlapped step (Sec. 5.3).
tests/host/host_logic_test.cpp drives paper_2110_13005_amd/csrc/host_logic.h (the header stage.cpp takes these
decisions from) with a simulated event layer; it is built and run twice: with the address + undefined-behaviour
sanitizers and with the thread sanitizer."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "host", "host_logic_test.cpp")


def _build_and_run(tmp_path, name, flags):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path / name)
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", "-Werror", *flags, SRC, "-o", exe, "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1",
               TSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert "all checks passed" in r.stdout
    assert "runtime error" not in r.stderr and "Sanitizer" not in r.stderr, r.stderr[-3000:]


def test_host_logic_address_and_undefined_behaviour_sanitizers(tmp_path):
    _build_and_run(tmp_path, "hl_asan", ["-fsanitize=address,undefined", "-fno-sanitize-recover=all"])


def test_host_logic_thread_sanitizer(tmp_path):
    _build_and_run(tmp_path, "hl_tsan", ["-fsanitize=thread"])


def test_stage_runtime_takes_its_decisions_from_the_tested_header():
    """stage.cpp must call the functions the CPU tests exercise, not private copies of them."""
    src = open(os.path.join(os.path.dirname(HERE), "paper_2110_13005_amd", "csrc", "stage.cpp")).read()
    for fn in ("host::choose_message", "host::admit_forward", "host::commit_forward", "host::admit_backward",
               "host::commit_backward", "host::wgrad_action", "host::gradients_complete", "host::release_awaiting",
               "host::check_post", "host::stream_index", "host::WaitClock",
               "host::addressable_in_place", "host::bucket_plan", "host::chunk_span", "host::lowest_layer"):
        assert fn in src, fn


def test_gemm_test_shapes_reach_the_tiles_they_name(tmp_path):
    """The GPU tests of the ring kernel's tiles and of the head's split input gradient rely on the launcher's cost model
    for the kernel that their shapes run on."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "tiles")
    subprocess.run([gxx, "-std=c++17", "-O1", SRC, "-o", exe, "-pthread"], check=True, timeout=300)

    def choice(M, N, K):
        tile, parts = map(int, subprocess.run([exe, "tile", str(M), str(N), str(K)], capture_output=True, text=True,
                                              check=True).stdout.split())
        return ("64x64", "128x64", "128x128", "128x192", "128x256", "large")[tile], parts

    from test_gpu_lm_ends import SPLIT_PARTS
    from test_gpu_ops import RING_TILES
    assert {s: choice(*s)[0] for s in RING_TILES} == RING_TILES
    assert set(RING_TILES.values()) == {"64x64", "128x64", "128x128", "128x192", "128x256"}
    assert {s: choice(*s)[1] for s in SPLIT_PARTS} == SPLIT_PARTS
    gemm = open(os.path.join(os.path.dirname(HERE), "paper_2110_13005_amd", "csrc", "gemm.hip")).read()
    assert all(fn in gemm for fn in ("host::choose_ring_tile", "host::choose_split", "host::xcd_contiguous"))
