"""The build's check on the compiler's resource report (CPU: compiles only)."""
import subprocess

import pytest

from paper_2609_19116_amd import build

REMARK = "x.hip:1:0: remark: {} [-Rpass-analysis=kernel-resource-usage]\n"


def _report(name, spill, waves):
    return "".join(REMARK.format(x) for x in (
        f"Function Name: {name}", "    VGPRs: 200", f"    VGPRs Spill: {spill}",
        f"    Occupancy [waves/SIMD]: {waves}"))


def test_resource_check_refuses_spills_and_lost_wavefronts():
    name = "_ZN3msc12camps_kernelENS_9CampsArgsE"
    assert build.kernel_resources(_report(name, 0, 2))[name]["VGPRs"] == 200
    build.check_resources("camps.hip", _report(name, 0, 2))
    build.check_resources("sampler.hip", "")           # nothing asked of it
    for bad in (_report(name, 1, 2), _report(name, 0, 1), "", _report("_ZN3msc5otherEv", 0, 2)):
        with pytest.raises(RuntimeError):
            build.check_resources("camps.hip", bad)


def test_camps_kernel_keeps_two_workgroups_per_cu(tmp_path):
    src = build.CSRC / "kernels" / "camps.hip"
    r = subprocess.run([build.HIPCC, "-x", "hip", *build.DEVICE, *build.COMMON, *build.REPORT,
                        "--cuda-device-only", "-c", str(src), "-o", str(tmp_path / "camps.o")],
                       capture_output=True, text=True, check=True)
    build.check_resources(src.name, r.stderr)
