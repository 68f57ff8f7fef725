"""Host-side checks of the build's register accounting: the GEMM and attention kernels are written to a
budget of 256 VGPRs (two waves per SIMD) or 168 (three); the build records what the compiler reports and refuses spills."""
import os

import pytest

from paper_2605_17633_amd import build

SAMPLE = """\
a.hip:43:1: remark: Function Name: _Z3fooPf [-Rpass-analysis=kernel-resource-usage]
   43 | {
      | ^
a.hip:43:1: remark:     TotalSGPRs: 22 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     VGPRs: 250 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     AGPRs: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     ScratchSize [bytes/lane]: 140 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     Occupancy [waves/SIMD]: 2 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     VGPRs Spill: 34 [-Rpass-analysis=kernel-resource-usage]
a.hip:43:1: remark:     LDS Size [bytes/block]: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:90:1: remark: Function Name: _Z3barPf [-Rpass-analysis=kernel-resource-usage]
a.hip:90:1: remark:     VGPRs: 12 [-Rpass-analysis=kernel-resource-usage]
a.hip:90:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
"""


def test_resource_remarks_are_parsed():
    ks = build._resources(SAMPLE)
    assert [k["name"] for k in ks] == ["_Z3fooPf", "_Z3barPf"]
    assert ks[0]["VGPRs"] == 250 and ks[0]["VGPRs Spill"] == 34 and ks[0]["ScratchSize"] == 140
    assert ks[0]["Occupancy"] == 2 and ks[1]["VGPRs Spill"] == 0


@pytest.mark.parametrize("name,hot", [
    ("_Z19gemm_bf16_nt_kernelILi128ELi128EEv", True), ("_Z25gemm_bf16_nt_fused_kernelILi128EEv", True),
    ("_Z16gemm_ring_kernelILi64ELi64ELi3EEv", True), ("_Z18gemm_direct_kernelILi0ELb0EEv", True),
    ("_ZN12_GLOBAL__N_118attn_global_kernelILi80EEEv", True), ("_ZN12_GLOBAL__N_113select_kernelILi64EEEv", False)])
def test_spills_of_hot_kernels_are_refused(name, hot):
    assert bool(build.spilled([{"name": name, "VGPRs Spill": 3}])) == hot
    assert not build.spilled([{"name": name, "VGPRs Spill": 0}])


def recorded():
    path = os.path.join(build.ROOT, "_build", "kernel_resources.txt")
    if not os.path.exists(path):
        pytest.skip("library not built in this tree")
    for line in open(path):
        f = line.split()
        yield f[1], {k: int(v) for k, v in (x.split("=") for x in f[2:])}


def test_hot_kernels_keep_their_register_budget():
    hot = [(n, r) for n, r in recorded() if any(h in n for h in build.HOT)]
    # bf16_nt: tiles x epilogues x layouts; rings: 3 tiles x (4 epilogues x 2 layouts + 2 folded forms); direct: 4 epilogues + 2 folded forms;
    # wide: 12 tiles x (4 epilogues x 2 layouts + 2 folded forms) + 8 that read statistics in pieces x 2 + 8 that leave them; global: 4 d x ((patches or not) x 3 tables + 2 short last tiles); windows: d = 64 and 80 persistent, a wave to a tile at four d with any rows and near ones
    for family, count in (("gemm_bf16_nt_", 93), ("gemm_ring_kernel", 30), ("gemm_direct_kernel", 6), ("gemm_wide_kernel", 144), ("attn_global_kernel", 32),
                          ("attn_window_kernelI", 2), ("attn_window_kernel_wavesI", 8)):
        assert sum(family in n for n, _ in hot) >= count, f"expected every instantiation of {family} in the record"
    for name, r in hot:
        assert r["spill"] == 0 and r["scratch"] == 0, (name, r)
        # the row-major forms of the 128x256 and 256x128 tiles (forced choices only) keep both operands in LDS, 96 KB a
        # workgroup: they are alone on their CU with one wave per SIMD whatever their registers, so the two-waves
        # budget does not apply to them
        if ("gemm_bf16_nt_kernelILi128ELi256E" in name or "gemm_bf16_nt_kernelILi256ELi128E" in name) and "ELb0E" in name:
            continue
        # rings of 48 KB run three workgroups to a CU, three waves to a SIMD; so do windows up to d = 64, a wave to a tile
        three = ("gemm_ring_kernel" in name and "gemm_ring_kernelILi128ELi128E" not in name) or \
                ("attn_window_kernel_wavesI" in name and "ILi80E" not in name and "ELb0E" in name)
        # global attention at d = 16 with tables of 32 runs four (but for its form for short last tiles)
        four = "attn_global_kernelILi16E" in name and "ELi32E" in name and "ELb1EEE" not in name
        assert r["vgprs"] + r["agprs"] <= (128 if four else 168 if three else 256), (name, r)


def test_what_spills_elsewhere():
    """The selection over more than 16384 scores holds 64 keys a thread in 128 registers, the most a workgroup of 1024 has."""
    for name, r in recorded():
        if "select_kernelILi64E" in name:
            assert r["spill"] <= 48 and r["scratch"] <= 200, (name, r)
        else:
            assert r["spill"] == 0 and r["scratch"] == 0, (name, r)
