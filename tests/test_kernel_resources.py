"""Compile-time guard (no GPU): the register-blocked min-plus kernel keeps its
table values in VGPRs, so a register spill in its loop costs a large factor.
Every instantiation must compile with zero scratch and reach the occupancy its
blocking table asks for."""
import os
import re
import subprocess

import pytest

from paper_2307_02031_amd import build as b


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    """The compiler's resource report, one text per kernel."""
    src = os.path.join(b.CSRC, "gbmw_kernels.hip")
    flags = [f for f in b.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [b.HIPCC, *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", src,
           "-o", str(tmp_path_factory.mktemp("resources") / "k.o")]
    out = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    return re.split(r"remark: Function Name: ", out)[1:]


def test_minplus_instantiations_do_not_spill(blocks):
    seen = 0
    for blk in blocks:
        name = blk.split()[0]
        m = re.match(r"_ZN4gbmw9k_minplusILi(\d+)ELi\d+ELi\d+ELi\d+ELi(\d+)E", name)
        if not m:
            continue
        seen += 1
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", blk).group(1))
        occ = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", blk).group(1))
        assert scratch == 0, f"{name}: {scratch} bytes of scratch per lane"
        assert occ >= int(m.group(2)), f"{name}: occupancy {occ} below the requested {m.group(2)}"
    assert seen == 288         # S' = 4..64 in steps of 4; first-layer and later-layer; with and without argmin records;
                               # three launch shapes (split, unsplit and the pruned step), and the
                               # counting twin of the last (measurements only, no occupancy target); S' = 68..128: with and
                               # without records


def test_the_wide_pruned_step_and_its_final_reduce_do_not_spill(blocks):
    """k_pruned_wide<2 | 4 chunks of 64 columns> for both layers' variants, with and without records (and the
    counting twins, which only have to exist), and k_final_pruned<1 | 2 | 4>: vector registers only, four and
    three waves per SIMD for the step."""
    wide = final = 0
    for blk in blocks:
        name = blk.split()[0]
        scratch = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", blk).group(1))
        occ = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", blk).group(1))
        vspill = int(re.search(r"VGPRs Spill: (\d+)", blk).group(1))
        m = re.match(r"_ZN4gbmw13k_pruned_wideILi(\d)ELb[01]ELb[01]ELb([01])E", name)
        if m:
            wide += 1
            if m.group(2) == "0":
                assert scratch == 0 and vspill == 0, f"{name}: {scratch} bytes of scratch, {vspill} spilled registers"
                assert occ >= (4 if m.group(1) == "2" else 3), f"{name}: {occ} waves per SIMD"
        if re.match(r"_ZN4gbmw14k_final_prunedILi[124]E", name):
            final += 1
            assert scratch == 0 and vspill == 0, f"{name}: {scratch} bytes of scratch, {vspill} spilled registers"
    assert wide == 16 and final == 3
