"""The host transfers' threads and waits on the CPU, against a stand-in for
the HIP runtime (tests/host/transfer_host.cpp): no GPU is involved."""
import os
import subprocess

import pytest

from paper_2604_22092_amd.build import hipcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host", "transfer_host.cpp")
SRC = os.path.join(ROOT, "paper_2604_22092_amd", "csrc", "fs_transfer.hip")


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("transfer") / "transfer_host")
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.dirname(SRC)]
    objs = []
    for src in (SRC, HOST):
        objs.append(f"{exe}_{len(objs)}.o")
        subprocess.run([hipcc(), "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none", "-x", "hip",
                        "-std=c++17", "-O1", "-fPIC", *inc, "-c", src, "-o", objs[-1]], check=True)
    # (host-only objects of one unit id each define its marker)
    subprocess.run(["g++", "-Wl,-z,muldefs", "-o", exe, *objs, "-lpthread"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.endswith("done\n"), res.stdout + res.stderr
    return res.stdout


def test_per_thread_stream_is_used_by_the_caller_alone(output):
    assert "failed" not in output and "differs" not in output
    assert "per-thread stream" not in output


def test_a_failed_history_read_waits_for_its_kernel(output):
    assert "error lost" not in output
    assert "buffer given up" not in output
