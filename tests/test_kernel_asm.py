"""The gfx950 code the compiler emits for the kernels (CPU: hipcc
cross-compiles without a GPU), against what the sources claim of them: every
instantiation keeps its state in registers, and the attention pass as few of
them as the workgroups per CU that its comment states.
"""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2504_03775_amd", "csrc", "flowkv_attention.hip")


def hipcc():
    for c in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if c and os.path.exists(c):
            return c
    return None


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    cc = hipcc()
    if cc is None:
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("asm") / "attn.s"
    from paper_2504_03775_amd.build import HIP_FLAGS, INCLUDE, CSRC
    flags = [f for f in HIP_FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([cc, *flags, "--cuda-device-only", "-S", "-I", INCLUDE, "-I", CSRC, SRC,
                    "-o", str(out)], check=True, capture_output=True, timeout=600)
    return out.read_text()


def kernel_entries(asm, kernel):
    """The code object's kernel list (one YAML entry each), by name."""
    out = {}
    for e in re.split(r"\n  - ", asm):
        m = re.search(rf"\.name:\s+(\S*{kernel}\S*)", e)
        if m:
            out[m.group(1)] = e
    return out


def test_attention_kernels_use_no_scratch_and_keep_their_occupancy(asm):
    """Pass 1 is one kernel per head_dim, query heads per KV head, layout,
    source of the lengths and place of the output, whatever split_tokens is;
    the merge one per head_dim, source of the lengths and width.  None uses
    scratch memory or spills, and pass 1's registers (512 a SIMD lane, taken
    in eights) allow three workgroups of four waves per CU at head_dim 128 and
    four at 64, and no more."""
    split = kernel_entries(asm, "decode_attn_split")
    merge = kernel_entries(asm, "decode_attn_merge")
    assert len(split) == 2 * 4 * 2 * 2 * 2, sorted(split)
    assert len(merge) == 2 * 2 * 2, sorted(merge)
    for n, e in {**split, **merge}.items():
        assert re.search(r"\.private_segment_fixed_size:\s+0\b", e), n
        assert re.search(r"\.vgpr_spill_count:\s+0\b", e), n
        assert int(re.search(r"\.kernarg_segment_size:\s+(\d+)", e).group(1)) <= 4096, n
    for n, e in split.items():
        m = re.search(r"decode_attn_splitILi(64|128)E", n)
        assert m, n
        waves = 4 if m.group(1) == "64" else 3
        vgprs = int(re.search(r"\.vgpr_count:\s+(\d+)", e).group(1))
        lds = int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", e).group(1))
        assert waves * (-(-vgprs // 8) * 8) <= 512, (n, vgprs)
        assert waves * lds <= 160 * 1024, (n, lds)
        # what the launch allocates: at head_dim 64 a fifth workgroup must not fit
        m = re.search(rf"\.amdhsa_kernel {re.escape(n)}\n.*?\.amdhsa_next_free_vgpr (\d+)",
                      asm, re.S)
        taken = -(-int(m.group(1)) // 8) * 8
        assert waves * taken <= 512 < (waves + 1) * taken, (n, taken)


# ---- the transfer kernels: no scratch memory, no spills ------------------------

XFER_SRC = os.path.join(ROOT, "paper_2504_03775_amd", "csrc", "flowkv_transfer.hip")


@pytest.fixture(scope="module")
def xfer_asm(tmp_path_factory):
    cc = hipcc()
    if cc is None:
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("asm") / "xfer.s"
    from paper_2504_03775_amd.build import HIP_FLAGS, INCLUDE, CSRC
    flags = [f for f in HIP_FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([cc, *flags, "--cuda-device-only", "-S", "-I", INCLUDE, "-I", CSRC, XFER_SRC,
                    "-o", str(out)], check=True, capture_output=True, timeout=900)
    return out.read_text()


def test_transfer_kernels_use_no_scratch_and_spill_nothing(xfer_asm):
    """Every instantiation of kv_segment_copy -- both layouts on each side,
    every unroll and cache policy, both address paths, the device-plan form
    and the three argument forms -- keeps its state in registers: no private
    (scratch) segment and no vector registers spilled.  So the transfer needs
    no device memory beyond the pools and the caller's plan, which is why it
    has no variant that allocates nothing.  The default launch shape (unroll
    4) spills no scalar registers either; some unroll-16 forms spill a few
    into vector-register lanes, which costs no memory."""
    names = re.findall(r"\.name:\s+(\S*kv_segment_copy\S*)", xfer_asm)
    # 4 layout pairs x 4 unroll x 4 cache x 2 paths x (device plan, general
    # inline form), 32 between block-major pools and 96 with a layer-major
    # pool in the compact forms
    assert len(names) == 4 * 4 * 4 * 2 * 2 + 32 + 96, len(names)
    assert sum("XferArgsCompactILi1E" in n for n in names) == 32
    assert sum("XferArgsCompactILi32E" in n for n in names) == 96
    entries = kernel_entries(xfer_asm, "kv_segment_copy")
    assert len(entries) == len(names)
    for n, e in entries.items():
        assert re.search(r"\.private_segment_fixed_size:\s+0\b", e), n
        assert re.search(r"\.vgpr_spill_count:\s+0\b", e), n
        if "ELi4ELi" in n:    # unroll 4, the default
            assert re.search(r"\.sgpr_spill_count:\s+0\b", e), n
        size = int(re.search(r"\.kernarg_segment_size:\s+(\d+)", e).group(1))
        assert size <= 4096, (n, size)
