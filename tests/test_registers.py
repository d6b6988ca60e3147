"""Registers of the built kernels, from the metadata that the compiler leaves in the library: the
one-stream GEMM keeps everything of a wave in registers (a spill is traffic in its innermost loop
that no result shows)."""
import os
import re
import struct
import subprocess

import pytest

import paper_2502_02175_amd as V

AMDGPU_METADATA, ELF_AMDGPU, SHT_NOTE = 32, 224, 7


def kernels(code_objects=None):
    """-> {mangled name: its metadata} over all gfx code objects inside the library, which code_objects collects."""
    import msgpack
    data = open(V.lib_path(), "rb").read()
    out, at = {}, data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == ELF_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            entsize, count = struct.unpack_from("<HH", data, at + 58)
            if code_objects is not None:
                code_objects.append(data[at:at + shoff + entsize * count])
            for i in range(count):
                kind, _, _, offset, size = struct.unpack_from("<IQQQQ", data, at + shoff + i * entsize + 4)
                p, end = at + offset, at + offset + size
                while kind == SHT_NOTE and p < end:
                    name_len, desc_len, note = struct.unpack_from("<III", data, p)
                    desc = p + 12 + (name_len + 3) // 4 * 4
                    if note == AMDGPU_METADATA:
                        for k in msgpack.unpackb(data[desc:desc + desc_len])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    p = desc + (desc_len + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


def test_the_one_stream_gemm_does_not_spill():
    mine = {n: k for n, k in kernels().items() if "gemm_rows_kernel" in n}
    assert len(mine) == 27  # feature blocks, epilogues, operand types
    for n, k in mine.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, n


def test_the_embedding_of_few_patches_keeps_one_way_of_staging():
    """With the two-byte and the 16-byte staging in one instance it takes 224 registers and 0.5 us more of 10."""
    mine = {n: k for n, k in kernels().items() if "embed_patches_kernelILi1E" in n}
    two = [k[".vgpr_count"] for n, k in mine.items() if "ELb1EEv" in n]
    assert len(mine) == 4 and len(two) == 2
    assert max(two) <= 192 and all(k[".vgpr_spill_count"] == 0 for k in mine.values())


def test_the_embedding_of_many_workgroups_reads_its_list():
    """An instance without the LDS of the list that few workgroups work out for themselves: thousands of them (8 x 1024
    patches of 16 x 16 pixels at d_model 4096) took 193 us that way, 172 with the list of one launch."""
    mine = {n: k for n, k in kernels().items() if "embed_listed_kernel" in n}
    assert len(mine) == 4
    for n, k in mine.items():
        assert k[".group_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0 and k[".vgpr_count"] <= 224, n


def test_the_many_rows_gemm_keeps_its_sums_in_registers():
    """Copied behind the loop, out of the half of the registers that the products leave them in, they spill by 80 to 110
    registers; what holds them there is one empty instruction that a compiler may take otherwise.  (Output head:
    two words of addresses, outside the loop.)"""
    mine = {n: k for n, k in kernels().items() if "gemm_tall_kernel" in n}
    assert len(mine) == 18  # epilogues, items of 192 features, operand types
    for n, k in mine.items():
        head = "gemm_tall_kernelILi3E" in n
        assert k[".private_segment_fixed_size"] <= (8 if head else 0) and k[".vgpr_spill_count"] <= (1 if head else 0), n


def test_the_few_rows_gemm_of_several_feature_blocks_does_not_spill():
    mine = {n: k for n, k in kernels().items() if "gemm_few_wide_kernel" in n}
    assert len(mine) == 27  # two and three blocks (head: and four), epilogues, operand types
    for n, k in mine.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, n


def test_the_many_rows_gemm_waits_for_one_stage_of_copies_per_step(tmp_path):
    """The loop of a work item waits for all but the youngest copies, once per step.  A load of the epilogue before that not
    every path uses is still open there for the compiler, which then waits for it, and so for every copy, at each step: the
    items of 97 to 160 rows took up to 30 % more than those of 256 (8 heads of keys, d_model 8192, 1408 rows: QKV 216 -> 254 us)."""
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    objects, loops = [], 0
    kernels(objects)
    for i, code in enumerate(o for o in objects if b"gemm_tall_kernel" in o):
        path = tmp_path / ("%d.co" % i)
        path.write_bytes(code)
        text = subprocess.run([objdump, "-d", "--mcpu=gfx950", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands",
                               str(path)], capture_output=True, text=True, check=True).stdout
        for body in re.split(r"^<?.*gemm_tall_kernel.*>?:$", text, flags=re.M)[1:]:
            for block in re.split(r"^<L\d+>:$", body, flags=re.M):
                block = re.split(r"^\s*s_c?branch", block, flags=re.M)[0]
                if block.count("v_mfma") >= 4 and block.count("global_load_lds") >= 6:
                    loops += 1
                    waits = [int(w) for w in re.findall(r"vmcnt\((\d+)\)", block)]
                    assert len([w for w in waits if w < 63]) == 1 and min(waits) >= 21, waits
    assert loops >= 18 * 9
