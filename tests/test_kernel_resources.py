"""Compile-time checks of the gfx950 kernels (CPU only): no kernel keeps
private arrays in scratch memory or spills registers -- register stages that
fall back to scratch turn every streamed byte into extra memory traffic."""
import glob
import os
import re
import subprocess

import pytest

from paper_2609_32395_amd import build as B


def _resource_remarks(src):
    cmd = [B.HIPCC, *B.COMMON_FLAGS, "-c", src, "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = {}
    name = None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            kernels[name] = {}
            continue
        m = re.search(r"remark:\s+(.+?): (\d+)", line)
        if m and name:
            kernels[name][m.group(1).strip()] = int(m.group(2))
    return kernels


@pytest.mark.parametrize("src", sorted(glob.glob(os.path.join(B.CSRC, "*.hip"))), ids=os.path.basename)
def test_no_scratch_no_spills(src):
    ks = _resource_remarks(src)
    for name, res in ks.items():
        assert res.get("ScratchSize [bytes/lane]", 0) == 0, (name, res)
        assert res.get("VGPRs Spill", 0) == 0 and res.get("SGPRs Spill", 0) == 0, (name, res)


def test_encoder_waves_per_simd():
    """Every encoder kernel leaves registers for four waves on a SIMD (four
    workgroups on a CU): its workgroups wait for their own loads, and what the
    others compute meanwhile is all that hides it."""
    ks = _resource_remarks(os.path.join(B.CSRC, "attn_mfma.hip"))
    enc = {n: r for n, r in ks.items() if "k_encoder_mfma" in n}
    assert len(enc) == 12
    for name, res in enc.items():
        assert res["Occupancy [waves/SIMD]"] >= 4, (name, res)


def test_reader_folds_only_what_a_launch_reaches():
    """The folding reader is built for pages of at most 32 loads per lane, the
    ones its launch rule accepts: not for fp32 heads of 128 in 64-row pages."""
    ks = _resource_remarks(os.path.join(B.CSRC, "reader_valu.hip"))
    fold = [n for n in ks if re.search(r"k_reader_valuI[ft]Li\d+ELi\d+ELb[01]ELb1ELb1E", n)]
    assert len(fold) == 2 * (2 * 3 * 2 - 1)      # rotary or not; types x widths x blocks but that one
    assert not [n for n in fold if "IfLi128ELi64E" in n]
