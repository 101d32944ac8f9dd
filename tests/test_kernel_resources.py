"""Register spills of the search variants, from the metadata the compiler leaves in the objects of the last build (nothing to look at
where only the linked library is there)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"
OBJECTS = sorted(glob.glob(os.path.join(ROOT, "paper_2605_14929_amd", "csrc", "_build", "search_[01]_[012].o")))
NAME = re.compile(r"search_kernelILb(\d)ELi(\d+)ELi\dELi(\d)ELi(\d)ELb(\d)ELi(\d)ELi(\d)ELb(\d)E")


def _kernels(obj, tmp):
    fat, code = str(tmp / "fat"), str(tmp / "code")
    subprocess.check_call([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(tmp / "copy")], stderr=subprocess.DEVNULL)
    subprocess.check_call([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                           f"--input={fat}", f"--output={code}"])
    notes = subprocess.run([f"{LLVM}/llvm-readobj", "--notes", code], capture_output=True, text=True, check=True).stdout
    for part in re.split(r"\n\s+- \.a", notes)[1:]:
        f = dict(re.findall(r"\.?(\w+):\s+(\S+)", part))
        m = NAME.search(f.get("symbol", ""))
        if m:
            bf16, epl, sign, metric, emit, na, occ, multi = map(int, m.groups())
            yield (bf16, epl, sign, metric, emit, na), occ, int(f["vgpr_count"]), int(f["vgpr_spill_count"])


@pytest.mark.skipif(len(OBJECTS) != 6 or not shutil.which(f"{LLVM}/clang-offload-bundler"), reason="no objects of a build, or no tools to read them")
def test_no_variant_spills(tmp_path):
    seen = 0
    for obj in OBJECTS:
        for (bf16, epl, sign, metric, emit, na), occ, vgprs, spilled in _kernels(obj, tmp_path):
            seen += 1
            assert vgprs <= 512 // occ
            assert spilled == 0, ((bf16, epl, sign, metric, emit, na), spilled)
    assert seen == 576
