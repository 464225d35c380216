"""Host-side logic of the library that needs no GPU: the block-id decoding of the kernels, compiled for the host
from the library's own header."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_block_decode_is_a_bijection_and_keeps_units_on_few_xcds(tmp_path):
    exe = tmp_path / "decode_check"
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "paper_2206_08888_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "decode_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and "bad 0" in out.stdout, out.stdout[-2000:]
    assert "agents 8, 9 on 4 and 4 XCDs; critics 16..19 on 2 2 2 2" in out.stdout


def test_workgroups_per_cu(tmp_path):
    exe = tmp_path / "lds_check"
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "paper_2206_08888_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "lds_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and "bad 0" in out.stdout, out.stdout[-2000:]


@pytest.mark.parametrize("check", ["act_grid_check", "spread_check"])
def test_rules_of_the_launches(tmp_path, check):
    exe = tmp_path / check
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(ROOT, "paper_2206_08888_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", check + ".cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and "bad 0" in out.stdout, out.stdout[-2000:]


def _asm(tmp, source):
    from paper_2206_08888_amd import build
    asm = tmp / (source + ".s")
    subprocess.run([build._hipcc(), *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(asm)],
                   check=True, capture_output=True)
    return asm.read_text()


@pytest.fixture(scope="module")
def k_chain_asm(tmp_path_factory):
    return _asm(tmp_path_factory.mktemp("asm"), "k_chain.hip")


# most SGPRs (arguments, mostly) and VGPRs spilled by the kernels of a file, where other than none: SAC's 64-row actor chains exist for tuning only
@pytest.mark.parametrize("source, kernels, sgprs, vgprs", [("k_few.hip", 10, 34, {}), ("k_sac.hip", 17, 16, {"k_sac_actorINS_12_GLOBAL__N_16Rows32ILi2E": 152}),
                                                            ("k_act.hip", 24, 0, {})])
def test_the_kernels_of_few_agents_of_sac_and_of_acting_spill_no_more_than_they_did(tmp_path, source, kernels, sgprs, vgprs):
    spills = {m[1]: (int(m[2]), int(m[3])) for m in re.finditer(r"\.name: +(_ZN3pop\S*).*?\.sgpr_spill_count: +(\d+).*?\.vgpr_spill_count: +(\d+)",
                                                                 _asm(tmp_path, source), re.S)}
    assert len(spills) == kernels, sorted(spills)
    for name, (s, v) in spills.items():
        assert s <= sgprs and v <= max((n for known, n in vgprs.items() if known in name), default=0), (name, s, v)


def test_critic_1_inside_the_target_workgroups_spills_no_arguments(k_chain_asm):
    """Arguments spilled at the kernel's start come in trips to memory one after the other."""
    spills = dict(re.findall(r"\.name: +(_ZN3pop\S*k_target_critic1INS_\S*Rows32ILi1E\S*).*?\.sgpr_spill_count: +(\d+)", k_chain_asm, re.S))
    assert len(spills) >= 2 and set(spills.values()) == {"0"}, spills


def test_wide_chains_that_have_a_cu_to_themselves_do_not_spill(k_chain_asm):
    """The wide-input kernels of k_chain.hip keep everything in registers, those that share a CU too."""
    spills = dict(re.findall(r"\.name: +(_ZN3pop\S*Rows\d+Deep\S*).*?\.vgpr_spill_count: +(\d+)", k_chain_asm, re.S))
    assert len(spills) >= 12 and sum("Rows32DeepILi1E" in k for k in spills) == 5, sorted(spills)      # five on eight wavefronts
    assert all(n == "0" for n in spills.values()), spills


def test_the_other_chains_spill_no_more_than_they_did(k_chain_asm):
    """Narrow actor chains, two workgroups to a CU, hold the actor's h2 tile across a product: their spills are known, the others have none."""
    spills = dict(re.findall(r"\.name: +(_ZN3pop\S*k_(?:target|critic|actor|act)\S*).*?\.vgpr_spill_count: +(\d+)", k_chain_asm, re.S))
    known = {"k_actorINS_12_GLOBAL__N_16Rows32ILi1ELb1ELi2ELb0EEELi2E": 40}
    for k, n in spills.items():
        assert int(n) <= max((m for name, m in known.items() if name in k), default=0), (k, n)
    assert all(any(name in k for k in spills) for name in known), sorted(spills)
