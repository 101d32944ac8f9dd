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


@pytest.mark.skipif(len(OBJECTS) != 6 or not shutil.which(f"{LLVM}/llvm-objdump"), reason="no objects of a build, or no tools to read them")
def test_a_step_waits_for_its_row_and_not_for_the_stores_before(tmp_path):
    """bf16 searches of one layer: the last wait before a step asks for the next row is the one for the row at hand (requested a step ago), and leaves that
    step's selector stores in flight: one, with up to eight atoms two."""
    def waits(obj):
        d = tmp_path / os.path.basename(obj)
        d.mkdir()
        list(_kernels(obj, d))                                    # (leaves the code object in d)
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(d / "code")], capture_output=True, text=True, check=True).stdout
        out = {}
        for part in re.split(r"\n[0-9a-f]+ <", text)[1:]:
            m = NAME.search(part.split(">")[0])
            if not m or m.group(5) == "1" or m.group(8) == "1" or "s_barrier" not in part:
                continue
            lines = part.split("s_barrier")[1].split("\n")        # from the loaded tables to the end of the row loop
            asks = [i for i, l in enumerate(lines) if "buffer_load_dwordx4" in l]
            while len(asks) > 1 and asks[-1] - asks[-2] < 14:     # (the requests of one row)
                asks.pop()
            out[m.group(0), m.group(6)] = int(re.findall(r"vmcnt\((\d+)\)", "\n".join(lines[:asks[-1]]))[-1])
        return out

    found = {k: v for obj in OBJECTS if "search_1_" in obj for k, v in waits(obj).items()}
    assert len(found) == 108
    late = {k: v for k, v in found.items() if v != (2 if k[1] == "8" else 1)}
    assert not late


PLANE = re.compile(r"plane_kernelILb(\d)ELi(\d+)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E")


@pytest.mark.skipif(len(OBJECTS) != 6 or not shutil.which(f"{LLVM}/llvm-objdump"), reason="no objects of a build, or no tools to read them")
def test_no_variant_of_one_plane_spills(tmp_path):
    """The searches that write one plane: no spilled vector register, no access to scratch memory (the frame that some of them reserve for scalar registers is kept in
    lanes of vector registers), and for bf16 weights the last wait before a step asks for its next row is not one for every store in flight."""
    seen = 0
    for obj in OBJECTS:
        list(_kernels(obj, tmp_path))                                # (leaves the code object)
        code = str(tmp_path / "code")
        notes = subprocess.run([f"{LLVM}/llvm-readobj", "--notes", code], capture_output=True, text=True, check=True).stdout
        limits = {}
        for part in re.split(r"\n\s+- \.a", notes)[1:]:
            f = dict(re.findall(r"\.?(\w+):\s+(\S+)", part))
            m = PLANE.search(f.get("symbol", ""))
            if m:
                limits[m.group(0)] = m
                assert int(f["vgpr_count"]) <= 512 // int(m.group(8)), m.group(0)
                assert int(f["vgpr_spill_count"]) == 0, m.group(0)
        if not limits:
            continue
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", code], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n[0-9a-f]+ <", text)[1:]:
            m = PLANE.search(part.split(">")[0])
            if not m or "s_barrier" not in part:
                continue
            assert "scratch_" not in part, m.group(0)
            seen += 1
            if m.group(1) == "0":
                continue
            lines = part.split("s_barrier")[1].split("\n")            # from the loaded tables to the end of the row loop
            asks = [i for i, l in enumerate(lines) if "buffer_load_dwordx4" in l]
            while len(asks) > 1 and asks[-1] - asks[-2] < 14:         # (the requests of one row)
                asks.pop()
            assert int(re.findall(r"vmcnt\((\d+)\)", "\n".join(lines[:asks[-1]]))[-1]) > 0, m.group(0)
    assert seen == 38
