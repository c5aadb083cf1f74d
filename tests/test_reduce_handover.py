"""The count reduce hands its blocks' totals to the block that draws the last
ticket.  Up to four wavefronts of a block store totals (32 and 64 replicas) and
one thread draws the ticket after the workgroup's barrier, which does not wait
for other wavefronts' global stores: each storing wavefront has to wait for its
own before the barrier.  Read from the assembly of the kernels, compiled as the
library is but for a lower optimisation level (a matter of seconds)."""
import os
import re
import subprocess

import pytest

from paper_2604_22092_amd.build import HIPCC_FLAGS, PKG, ROOT, hipcc


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "fs_kernels.s")
    subprocess.run([hipcc(), *HIPCC_FLAGS, "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                    "--cuda-device-only", "-S", "-o", out, os.path.join(PKG, "csrc", "fs_kernels.hip")],
                   check=True, capture_output=True)
    text = open(out).read()
    return {m.group(1): m.group(0) for m in re.finditer(r"^_ZN3fsk\d+(\w+?)E\w*:.*?^\.Lfunc_end", text, re.M | re.S)}


@pytest.mark.parametrize("name", ["reduce_kernel", "reduce_batch_kernel"])
def test_totals_are_waited_for_before_the_barrier(kernels, name):
    body = next(v for k, v in kernels.items() if k.startswith(name))
    lines = [l.split(";")[0].strip() for l in body.splitlines()]
    # the totals: agent-scope stores (write-through, sc1) before the first ticket
    ticket = next(i for i, l in enumerate(lines) if l.startswith(("global_atomic_add", "flat_atomic_add")))
    stores = [i for i, l in enumerate(lines[:ticket]) if l.startswith(("global_store", "flat_store")) and l.endswith("sc1")]
    assert stores
    for i in stores:
        after = lines[i + 1:ticket]
        barrier = next(j for j, l in enumerate(after) if l.startswith("s_barrier"))
        assert any(re.match(r"s_waitcnt.*vmcnt\(0\)", l) for l in after[:barrier]), "\n".join(after[:barrier + 1])
