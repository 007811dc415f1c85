"""The host side of the batch calls and the server, without a GPU: csrc/batch.cpp and csrc/serve.cpp linked
with a runtime that only logs (units/batch_host.cpp).  Only a replay needs the captured graph, so a batch is launched before the capture
begins, other buffers alone cause none, and a capture that fails costs neither this batch nor the next one.
The server, which never replays, captures nothing.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1305_4376_amd", "csrc")
SIZES = {"teams": 100, "waves": 2048 * 2049}  # blocks of a batch on either side of the switch between its kernels


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "batch_host")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-value", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                           "-o", exe, os.path.join(ROOT, "tests", "units", "batch_host.cpp"), *(os.path.join(CSRC, f) for f in ("batch.cpp", "serve.cpp")),
                           "-pthread"])
    return lambda *args: subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60,
                                        check=True).stdout.splitlines()


@pytest.mark.parametrize("kernel", SIZES)
def test_a_batch_is_launched_before_its_graph_is_captured(run, kernel):
    direct, capture = ["launch plan", f"launch {kernel}"], [f"capture {kernel}", "instantiate"]
    assert run("ordinary", SIZES[kernel]) == [
        *direct, *capture, "batch 0",
        "launch graph", "replay 0",
        *direct, "batch 0",                                       # the same buffer
        *direct, "batch 0",                                       # another: its graph waits for a replay
        "drop graph", *capture, "launch graph", "replay 0",
        *direct, "batch 0",
        "drop graph"]


@pytest.mark.parametrize("kernel", SIZES)
@pytest.mark.parametrize("call", ["begin", "end", "instantiate"])
def test_a_failed_capture_does_not_fail_the_batch(run, kernel, call):
    direct = ["launch plan", f"launch {kernel}"]
    tried = [] if call == "begin" else [f"capture {kernel}"]
    assert run(call, SIZES[kernel]) == [
        *direct, *tried, "batch 0",
        *direct, *tried, "batch 0",
        *tried, "replay -8",                        # a replay has nothing else to launch
        f"capture {kernel}", "instantiate", "launch graph", "replay 0",
        "drop graph"]


@pytest.mark.parametrize("kernel", SIZES)
def test_the_server_captures_no_graphs(run, kernel):
    assert run("serve", SIZES[kernel]) == ["launch fill", "launch plan", f"launch {kernel}", "served 0 0"] * 2
