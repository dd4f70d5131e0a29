"""What the compiler made of the kernels, read from the metadata of the built library (llvm-readelf prints it): a
kernel that does not fit its registers spills to scratch memory, which nothing else would report."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    """The gfx950 code objects of the offload bundles inside a host library."""
    blob, magic, at = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        entries, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(entries):
            offset, size, name = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + name]:
                yield blob[at + offset:at + offset + size]
            p += 24 + name
        at += len(magic)


def kernels(tmp_path):
    """(mangled name, scratch bytes per work item) of every kernel in the library."""
    import paper_2209_09130_amd as P
    P.lib()
    found = []
    for n, obj in enumerate(code_objects(P.lib_path())):
        f = tmp_path / f"{n}.co"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for entry in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            field = lambda key: re.search(r"\.%s:\s+(\S+)" % key, entry).group(1)
            found.append((field("name"), int(field("private_segment_fixed_size"))))
    return found


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
@pytest.mark.parametrize("kernel", ["attention_i8_kernel", "attention_i8_p16_kernel", "attention_f16_kernel", "gemm_nt_stream_kernel"])
def test_kernels_use_no_scratch_memory(kernel, tmp_path):
    found = [(name, scratch) for name, scratch in kernels(tmp_path) if kernel in name]
    assert len(found) >= 4, found
    assert not [k for k in found if k[1]]


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf is not installed")
@pytest.mark.parametrize("kernel,least", [("qkv_attention_i8_packed_kernel", 2), ("gemm_nt_ln_kernel", 4), ("gemm_nt_small_kernel", 4),
                                          ("gemm_nt_small_f16_kernel", 3)])
def test_kernels_of_few_instances_use_no_scratch_memory(kernel, least, tmp_path):
    found = [(name, scratch) for name, scratch in kernels(tmp_path) if kernel in name]
    assert len(found) >= least, found
    assert not [k for k in found if k[1]]
