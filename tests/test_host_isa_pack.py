"""The copy and transpose kernels that take any alignment, in the LLVM IR and
gfx950 assembly built here from source (no GPU needed): the compiler may assume
no alignment of their global accesses, and still uses one wide instruction."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_11718_amd import build as B

ANY = ("copy_kernel", "copy_stream_kernel", "pack_trans_any_kernel")


@pytest.fixture(scope="module")
def text(tmp_path_factory):
    if shutil.which(B.HIPCC) is None and not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not available")
    out, src = {}, os.path.join(B.CSRC, "kernels", "pack.hip")
    for kind, flags in (("ll", ["-emit-llvm"]), ("s", [])):
        path = tmp_path_factory.mktemp("pack") / ("pack." + kind)
        r = subprocess.run([B.HIPCC] + B.HIP_FLAGS + ["-x", "hip", "--cuda-device-only", "-S", *flags, src, "-o", str(path)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        out[kind] = path.read_text()
    return out


def _any_alignment(name: str) -> bool:
    ragged_reg = "pack_trans_reg_kernel" in name and re.search(r"kernelI\wLb1E", name)
    return bool(ragged_reg) or any(k in name for k in ANY)


def test_no_alignment_is_assumed(text):
    seen = 0
    for name, body in re.findall(r"define [^\n]*amdgpu_kernel [^\n]*@(\w+)\([^\n]*\{\n(.*?)\n\}", text["ll"], re.S):
        if not _any_alignment(name):
            continue
        for ln in body.splitlines():
            if re.search(r"(load|store) .*addrspace\(1\)", ln):
                seen += 1
                assert re.search(r"align 1(,|$)", ln), (name, ln)
    assert seen > 100


def test_units_move_in_one_instruction(text):
    names = [n for n in re.findall(r"^(\w+):", text["s"], re.M) if "IDv4_j" in n and _any_alignment(n)]
    assert names
    for name in names:
        i = text["s"].index(name + ":")
        body = text["s"][i:text["s"].index(".Lfunc_end", i)]
        assert "global_load_dwordx4" in body and "global_store_dwordx4" in body
        assert not re.search(r"(global|flat)_(load|store)_(u?byte|short|dword|dwordx2|dwordx3)\b", body), name
