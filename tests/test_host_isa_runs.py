"""The bf16 64-K-stage kernels' direct-to-LDS loads, in the gfx950 assembly
built here from source (no GPU needed): loads of one operand share an M0 write,
and load i of such a run must carry the instruction offset 1024 i, with no
other M0 write inside the run and the run's loads in order; and nothing spills."""
import re

import pytest

from tests.test_host_isa import KERNELS, _body, _lds_offset, asm  # noqa: F401


@pytest.mark.parametrize("bm,bn,lengths", [(256, 128, {2, 4}), (128, 256, {2, 4}), (128, 128, {2}), (128, 192, {2, 3}),
                                           (128, 320, {1, 2, 4})])
@pytest.mark.parametrize("ragged", [0, 1])
@pytest.mark.parametrize("nt", [0, 1])
def test_k64_runs(asm, bm, bn, lengths, ragged, nt):  # noqa: F811
    name = (f"_ZN3ccl12_GLOBAL__N_115gemm_k64_kernelILi{bm}ELi{bn}ELb{ragged}ELb{nt}EEEv"
            "NS0_10GemmParamsE")
    body = _body(asm, name)
    runs = []
    for ln in body:
        if re.match(r"s_\w+\s+m0\b", ln):
            runs.append([])
        elif "buffer_load" in ln and re.search(r"\blds\b", ln):
            runs[-1].append(_lds_offset(ln))
    assert {len(r) for r in runs} == lengths
    assert all(r == [1024 * i for i in range(len(r))] for r in runs)
    assert not any("scratch_" in ln for ln in body)


@pytest.mark.parametrize("kernel", list(KERNELS))
def test_pipelined_kernels_do_not_spill(asm, kernel):  # noqa: F811
    """No scratch access in the whole kernel: epilogues included, whose values
    must not stay live through the K loop."""
    assert not [ln for ln in _body(asm, kernel) if ln.startswith("scratch_")][:4]


def test_four_wave_kernel_spills_no_more_than_its_k_loop_needs(asm):  # noqa: F811
    """gemm_kernel<256, 256, 2> holds 256 accumulators per lane; 88 bytes of
    scratch with one staged epilogue, 120 with two."""
    name = "_ZN3ccl12_GLOBAL__N_111gemm_kernelILi256ELi256ELi2EEEvNS0_10GemmParamsE"
    size = re.search(rf"\.name:\s+{name}\n\s+\.private_segment_fixed_size:\s+(\d+)", asm)
    assert int(size.group(1)) <= 88


@pytest.mark.parametrize("name", [
    "15gemm_k64_kernelILi128ELi128ELb0ELb0EEEv", "15gemm_k64_kernelILi256ELi128ELb0ELb0EEEv",
    "15gemm_k64_kernelILi128ELi320ELb1ELb0EEEv", "16gemm_fp8s_kernelILi256ELi128ELi4ELi2EEEv",
    "14gemm_a2_kernelE", "11gemm_kernelILi256ELi256ELi4EEEv", "16gemm_fp8p_kernelE"])
def test_store_policy_of_c_stays_a_choice(asm, name):  # noqa: F811
    """C's non-temporal stores where the launch asks for them beside plain ones:
    alike, the compiler merges the two into a plain store."""
    name = re.search(rf"^(_ZN3ccl12_GLOBAL__N_1{name}\w*):", asm, re.M).group(1)
    stores = [ln for ln in _body(asm, name) if ln.startswith("global_store_dwordx4")]
    assert any(ln.endswith(" nt") for ln in stores) and any(not ln.endswith(" nt") for ln in stores)
