"""The build's checks on its kernels' device assembly (CPU: compiles only)."""
import pytest

from paper_2609_19116_amd import build

KERNEL = """
{name}:   ; @{name}
; Occupancy: {waves}
  - .agpr_count:     0
    .args:
      - .name:           P
    .name:           {name}
    .vgpr_spill_count: {spills}
"""


def test_resource_check_refuses_spills_and_lost_wavefronts():
    def asm(waves, spills, name="_ZN3msc12camps_kernelENS_9CampsArgsE"):
        return KERNEL.format(name=name, waves=waves, spills=spills)

    assert list(build.kernel_resources(asm(2, 7)).values()) == [{"waves": 2, "vgpr_spills": 7}]
    build.check_resources("camps.hip", asm(2, 0))
    build.check_resources("sampler.hip", "")           # nothing asked of it
    for bad in (asm(2, 1), asm(1, 0), "", asm(2, 0, name="_ZN3msc5otherEv")):
        with pytest.raises(RuntimeError):
            build.check_resources("camps.hip", bad)


def test_camps_kernel_keeps_two_workgroups_per_cu(tmp_path):
    asm = build.device_assembly(build.CSRC / "kernels" / "camps.hip", tmp_path / "camps.o")
    build.check_resources("camps.hip", asm)
    assert build.lost_lanes(asm) == []


JOIN = """
_Z6kernelv:
	s_and_saveexec_b64 s[0:1], vcc
	s_cbranch_execz .LBB0_2
; %bb.1:
	v_add_u32_e32 v1, v2, v3
.LBB0_2:                       ; join
{}	s_or_b64 exec, exec, s[0:1]
	v_mov_b32_e32 v5, v6
	s_endpgm
"""


def test_lost_lanes_are_found():
    assert build.lost_lanes(JOIN.format("")) == []
    # scalar spills in vector lanes do not depend on the mask
    assert build.lost_lanes(JOIN.format("\tv_writelane_b32 v167, s62, 9\n\ts_mov_b32 s62, s66\n")) == []
    for ins in ("v_mov_b32_e32 v101, v108", "scratch_store_dword off, v158, off offset:60"):
        bad = JOIN.format(f"\tv_writelane_b32 v167, s62, 9\n\t{ins} ; 4-byte Folded Spill\n")
        assert build.lost_lanes(bad) == [("_Z6kernelv", [ins])]
    # a loop's exit: no lane is left until the mask's restore
    loop = ".LBB0_1:\n\ts_andn2_b64 exec, exec, s[2:3]\n\ts_cbranch_execnz .LBB0_1\n; %bb.2:\n{}" \
           "\ts_or_b64 exec, exec, s[2:3]\n"
    assert build.lost_lanes(loop.format("")) == []
    assert len(build.lost_lanes(loop.format("\tv_mov_b32_e32 v1, v2\n"))) == 1
