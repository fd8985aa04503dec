"""Registers and LDS that kernels may take and loads that they issue together,
from the compiler's own output for gfx950 (no GPU needed)."""
import os
import re
import subprocess

from paper_2606_24467_amd import build as B


def _resources(src, kernel):
    """(SGPRs, VGPRs, AGPRs, scratch bytes, LDS bytes) of a kernel as built."""
    r = subprocess.run([B._hipcc(), *B.FLAGS, *B.EXTRA.get(src, []), "-c",
                        "-Rpass-analysis=kernel-resource-usage", os.path.join(B.CSRC, src),
                        "-o", os.devnull], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    block = re.search(rf"Function Name: \S*{kernel}.*?LDS Size \[bytes/block\]: \d+", r.stderr,
                      re.S).group(0)
    num = lambda key: int(re.search(key + r": (\d+)", block).group(1))  # noqa: E731
    return (num("SGPRs"), num(" VGPRs"), num("AGPRs"), num(r"ScratchSize \[bytes/lane\]"),
            num(r"LDS Size \[bytes/block\]"))


def test_two_srh_score_workgroups_fit_a_cu():
    """Eight waves per SIMD: 512 registers / 8 VGPRs, 160 KB / 2 LDS, and 80
    SGPRs (800 / 8 = 100, less 16 for the trap handler, in steps of 16)."""
    sgprs, vgprs, agprs, scratch, lds = _resources("offline.hip", "srh_score_kernel")
    assert sgprs <= 80
    assert vgprs + agprs <= 64
    assert scratch == 0
    assert 2 * lds <= 160 * 1024


def test_srh_score_issues_a_batch_of_span_loads_together():
    """Every span load of a batch is issued before the first one is waited for
    and converted to fp64."""
    src = os.path.join(B.CSRC, "offline.hip")
    batch = int(re.search(r"kSrhBatch = (\d+);", open(src).read()).group(1))
    r = subprocess.run([B._hipcc(), *B.FLAGS, "--cuda-device-only", "-S", src, "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    body = re.search(r"^\S*srh_score_kernel\S*:(.*?)s_endpgm", r.stdout, re.S | re.M).group(1)
    # back from the first conversion to the start of its run of straight-line code
    before = body[:body.index("v_cvt_f64_f32")]
    run = re.split(r"^(?:\S+:|\s+s_c?branch\S*|\s+s_\w*saveexec\S*)", before, flags=re.M)[-1]
    assert len(re.findall(r"^\s+global_load_dword\s", run, re.M)) == batch
