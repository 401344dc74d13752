"""The host copies phi as soon as it sees a read-out workgroup's word, so every
wave must have its values and flags out before the barrier that the word's store
follows.  Checked in the gfx950 assembly compiled from the source (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_0907_1720_amd import build as B


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "kernels.s")
    cmd = ([B.HIPCC] + B.DEVICE_FLAGS + [f"-I{B.INCLUDE}", f"-I{B.CSRC}", "-S", "--offload-device-only",
                                         os.path.join(B.CSRC, "kernels.hip"), "-o", out])
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    return open(out).read()


@pytest.mark.parametrize("kernel", ["6k_readIdE", "6k_readIfE"])
def test_every_wave_waits_for_its_stores_before_the_barrier(assembly, kernel):
    body = re.search(r"^_ZN3lbm%s\S*:.*?s_endpgm" % kernel, assembly, re.S | re.M).group(0)
    lines = [ln.split(";")[0].strip() for ln in body.splitlines()]
    bars = [i for i, ln in enumerate(lines) if ln.startswith("s_barrier")]
    assert len(bars) == 1
    stores = [i for i, ln in enumerate(lines[:bars[0]]) if re.match(r"(global|flat|buffer)_store", ln)]
    assert stores, "the values are stored before the barrier"
    # the wait lies in the barrier's own block, which every wave that stores runs through
    block = max(i for i, ln in enumerate(lines[:bars[0]]) if re.match(r"\.?L\w+:", ln) or ln.startswith("s_cbranch"))
    waits = [i for i in range(block, bars[0]) if re.match(r"s_waitcnt\b.*vmcnt\(0\)", lines[i])]
    assert waits and max([s for s in stores if s > block], default=block) < waits[-1], "\n".join(lines[block:bars[0] + 1])
    # of what the host reads, nothing stays in a cache: system-scope stores
    watched = [lines[i] for i in stores if "sc0 sc1" in lines[i]]
    assert any("dwordx2" in ln for ln in watched) and sum("dwordx2" not in ln for ln in watched) >= 2, lines
