"""Host checks of the build script's kernel-resource rule (no GPU, no compiler run)."""
from paper_1904_03409_amd import build


def test_scratch_rule():
    assert build.may_spill("_Z4k_tnILi3ELb1EEv6TnArgs")
    for name in ("_Z4k_tnILi3ELb0EEv6TnArgs", "_Z4k_tnILi1ELb1EEv6TnArgs", "_Z9k_lev_bwdILi2ELi16ELb0EEv10LevBwdArgs",
                 "_Z9k_lev_fwdILi1ELi32ELb1EEv10LevFwdArgs", "_Z4k_ntILi3ELi1EEv6NtArgs", "_Z6k_planILb1EEv8PlanArgs"):
        assert not build.may_spill(name)


def test_resource_report_parse():
    text = "\n".join([
        "a.hip:1:1: remark: Function Name: _Z9k_lev_bwdILi2ELi16ELb0EEv10LevBwdArgs [-Rpass-analysis=kernel-resource-usage]",
        "a.hip:1:1: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]",
        "a.hip:1:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]",
        "a.hip:9:1: remark: Function Name: _Z4k_tnILi3ELb1EEv6TnArgs [-Rpass-analysis=kernel-resource-usage]",
        "a.hip:9:1: remark:     ScratchSize [bytes/lane]: 880 [-Rpass-analysis=kernel-resource-usage]",
    ])
    rep = build.resource_report(text)
    assert rep == {"_Z9k_lev_bwdILi2ELi16ELb0EEv10LevBwdArgs": 0, "_Z4k_tnILi3ELb1EEv6TnArgs": 880}


def _asm(nop_taken: str) -> str:
    return "\n".join([
        "_Z5k_xxxv:",
        "\tv_mfma_f32_16x16x32_f16 a[0:3], v[10:13], v[14:17], a[0:3]",
        "\tv_mfma_f32_16x16x32_f16 a[4:7], v[18:21], v[22:25], a[4:7]",
        *nop_taken.splitlines(),
        "\ts_cbranch_vccnz .LBB0_5",
        "; %bb.4:",
        "\ts_memrealtime s[10:11]",
        "\ts_waitcnt lgkmcnt(0)",
        ".LBB0_5:",
        "\ts_nop 1",
        "\tv_accvgpr_read_b32 v0, a7",
        "\tv_accvgpr_read_b32 v2, a3",
        "\tv_add_f32_e32 v13, v2, v0",
        "\ts_endpgm",
    ])


def test_mfma_branch_hazard_scan():
    # the pattern that returned a stale accumulator: 1 (branch) + 2 (s_nop 1) wait states on the taken path
    hz = build.mfma_branch_hazards(_asm(""))
    assert len(hz) == 1 and "after 3 wait states (needs 8)" in hz[0] and hz[0].startswith("_Z5k_xxxv")
    # enough wait states before the branch clear it: 1 + 2 + 5 is 8, one less is not
    assert build.mfma_branch_hazards(_asm("\ts_nop 4")) == []
    assert len(build.mfma_branch_hazards(_asm("\ts_nop 3"))) == 1
    assert build.mfma_branch_hazards(_asm("\ts_nop 4").replace("_f16 ", "_bf16 ")) == []
    # an MFMA the table does not name needs the longest wait
    assert "needs 19" in build.mfma_branch_hazards(_asm("\ts_nop 4").replace("16x16x32_f16 a[4:7]", "32x32x16_f16 a[4:7]"))[0]
    # a read of registers the MFMA did not write is no hazard
    assert build.mfma_branch_hazards(_asm("").replace("v0, a7", "v0, a9")) == []
