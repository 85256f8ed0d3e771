"""What the compiler gave the kernels of the built library: registers and spills, from the notes of its code object."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """Mangled kernel name -> its numbers."""
    at = tmp_path_factory.mktemp("code")
    tool = lambda name, *args: subprocess.run([os.path.join(LLVM, name), *args], check=True, capture_output=True, text=True).stdout  # noqa: E731
    tool("llvm-objcopy", f"--dump-section=.hip_fatbin={at}/bundle", os.path.join(ROOT, "paper_2106_16064_amd", "libdgsp.so"), f"{at}/copy")
    tool("clang-offload-bundler", "--unbundle", "--type=o", f"--input={at}/bundle", f"--output={at}/code",
         "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
    found, name = {}, None
    for line in tool("llvm-readelf", "--notes", f"{at}/code").splitlines():
        m = re.match(r"    \.(name|sgpr_spill_count|vgpr_count|vgpr_spill_count): +(\S+)", line)
        if m and m[1] == "name":
            name = m[2]
            found[name] = {}
        elif m:
            found[name][m[1]] = int(m[2])
    return found


def test_forms_that_share_no_rows_pay_nothing_for_those_that_do(resources):
    """nb_pr_kernel<V, KQ, SNAP, AXPBY, SHARES, ...>: with the choice left to the run, these spilled 22 scalar registers and more, and at
    two columns the plain form lost one of four waves a SIMD (128 vector registers)."""
    forms = {name: r for name, r in resources.items() if re.search(r"nb_pr_kernelILi\dELi2ELb\dELb\dELb0E", name)}
    assert len(forms) >= 4 * 8
    for name, r in forms.items():
        assert r["sgpr_spill_count"] == 0 and r["vgpr_spill_count"] == 0, name
    for v in (1, 2):
        plain, = [r for name, r in forms.items() if f"nb_pr_kernelILi{v}ELi2ELb0ELb0ELb0ELb0ELb0E" in name]
        assert plain["vgpr_count"] <= 128


def waves_a_simd(r):
    return min(8, 512 // (-(-r["vgpr_count"] // 8) * 8))


def test_forms_that_share_rows_or_queue_keep_as_many_workgroups(resources):
    """launch_nb_sr_run_v sizes the grid by the form without either, per lane layout and scaling."""
    plain = {name: r for name, r in resources.items() if re.search(r"nb_sr_run_kernelILi\dELb\dELb\dELb0ELb0E", name)}
    assert len(plain) >= 7 * 3
    others = 0
    for name, r in plain.items():
        for form in ("ELb1ELb0E", "ELb0ELb1E"):
            other = resources.get(re.sub(r"(nb_sr_run_kernelILi\dELb\dELb\d)ELb0ELb0E", r"\1" + form, name))
            if other:
                others += 1
                assert waves_a_simd(other) >= waves_a_simd(r), name
    assert others >= 7 * 3


def test_what_sharing_rows_costs_the_forms_that_do(resources):
    """Which of the rows at its ends a wave shares it keeps for the whole chunk.  As four booleans that was a pair of scalar registers each, and
    nb_pr_kernel took 131 vector registers at two columns, three waves a SIMD instead of four."""
    plain, scaled = ({v: r for name, r in resources.items() for v in "1234" if f"nb_pr_kernelILi{v}ELi2ELb0ELb{s}ELb1ELb0ELb0E" in name}
                     for s in "01")
    assert len(plain) == len(scaled) == 4
    assert plain["1"]["vgpr_count"] <= 128 and plain["2"]["vgpr_count"] <= 128 and scaled["1"]["vgpr_count"] <= 128
    for v in "1234":
        assert plain[v]["vgpr_spill_count"] == scaled[v]["vgpr_spill_count"] == 0
        assert plain[v]["sgpr_spill_count"] <= (4 if v in "12" else 12) and scaled[v]["sgpr_spill_count"] <= (15 if v in "12" else 22)
    hot = [r for name, r in resources.items() if re.search(r"nb_pr_kernelILi\dELi2ELb0ELb\dELb1ELb0ELb1E", name)]
    assert len(hot) == 8
    for r in hot:                                          # eight waves a CU, two a SIMD
        assert r["vgpr_count"] <= 256 and r["vgpr_spill_count"] == 0 and r["sgpr_spill_count"] <= 25
    assert all(r["vgpr_count"] <= 128 for name, r in resources.items() if "nb_sr_run_kernel" in name)      # four waves a SIMD
    runs = {name: r for name, r in resources.items() if re.search(r"nb_sr_run_kernelILi\dELb\dELb0ELb0ELb1E", name)}
    assert len(runs) == 14
    for name, r in runs.items():
        assert r["vgpr_count"] <= 128 and r["vgpr_spill_count"] == 0, name
        assert r["sgpr_spill_count"] <= (6 if "kernelILi0E" in name else 2), name
