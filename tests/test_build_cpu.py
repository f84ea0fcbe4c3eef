"""Checks of the compiled device code, no GPU: the build's guard against kernels
that use scratch memory, and the waits ahead of a hand-off between workgroups."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2402_15106_amd import build  # noqa: E402

REMARKS = """\
a.hip:1:1: remark: Function Name: k_one [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     VGPRs: 64 [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark: Function Name: k_two [-Rpass-analysis=kernel-resource-usage]
a.hip:9:1: remark:     ScratchSize [bytes/lane]: 240 [-Rpass-analysis=kernel-resource-usage]
"""


def test_scratch_kernels_names_only_the_spilling_kernel():
    assert build.scratch_kernels(REMARKS) == ["k_two (240 bytes/lane)"]
    assert build.scratch_kernels("") == []


@pytest.fixture(scope="module")
def core_asm(tmp_path_factory):
    """core.hip's gfx950 assembly, with the library's own flags."""
    out = str(tmp_path_factory.mktemp("asm") / "core.s")
    cmd = [build._hipcc()] + build.COMMON + ["--offload-device-only", "-S", os.path.join(build.CSRC, "core.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=300)
    return open(out).read()


@pytest.mark.parametrize("kernel", ["k_mid_hist", "k_mid_list"])
def test_every_wave_waits_for_its_writes_before_the_hand_off(core_asm, kernel):
    """One thread fences for its workgroup and counts it as done.  The barrier
    ahead of that fence orders LDS only, so each wave's own global writes have to
    be waited for before it."""
    body = re.search(r"^_ZN\S*%s\S*:.*?s_endpgm" % kernel, core_asm, re.M | re.S).group(0)
    code = [l.split(";")[0].strip() for l in body.splitlines()]
    fence = next(i for i, l in enumerate(code) if l.startswith("buffer_wbl2"))
    barrier = max(i for i, l in enumerate(code[:fence]) if l == "s_barrier")
    ops = [i for i, l in enumerate(code[:barrier]) if l.startswith(("global_", "flat_", "buffer_"))]
    waits = [i for i, l in enumerate(code[:barrier]) if l.startswith("s_waitcnt") and "vmcnt(0)" in l]
    assert ops and waits and waits[-1] > ops[-1], (kernel, code[ops[-1]], code[barrier])
    # and it is not skipped: no branch target between the wait and the barrier
    assert not any(l.endswith(":") for l in code[waits[-1]:barrier])


def test_outer_sums_refuse_an_edge_order_they_do_not_read(tmp_path):
    """The bf16 sums of d <= 64 take the edges in their stored order; a launch
    with another order is refused on the host (nothing runs on a GPU here)."""
    import paper_2402_15106_amd as dm
    exe, libdir = str(tmp_path / "outer_order"), os.path.dirname(dm.LIB_PATH)
    subprocess.run([build._hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    os.path.join(ROOT, "tests", "native", "outer_order.cpp"), "-o", exe, "-L" + libdir, "-ldsmpnn",
                    "-Wl,-rpath," + libdir], check=True, capture_output=True, timeout=300)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1")
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60, env=env).stdout.splitlines()
    assert len(out) == 2
    for line in out:
        assert line.startswith("%d " % dm.UNSUPPORTED) and "stored order" in line
