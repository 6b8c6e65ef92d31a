"""What the compiler made of the kernels, from the AMD metadata of the built
library's own code objects."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: {scratch, lds, threads}} of libmgemm.so."""
    from paper_2305_18236_amd import _native, build
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")) or not shutil.which("c++filt"):
        pytest.skip("no LLVM or binutils tools")
    _native.lib()
    tmp = tmp_path_factory.mktemp("objects")
    lib = shutil.copy(build.LIB, tmp)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], cwd=tmp, check=True, capture_output=True)
    found = []
    for name in sorted(os.listdir(tmp)):
        if build.ARCH not in name:
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", os.path.join(tmp, name)], check=True,
                               capture_output=True, text=True).stdout
        for block in re.split(r"\n  - \.a", notes)[1:]:
            field = {k: re.search(rf"\.{k}:\s+(\S+)", block) for k in
                     ("symbol", "private_segment_fixed_size", "group_segment_fixed_size", "max_flat_workgroup_size")}
            if all(field.values()):
                found.append([m.group(1) for m in field.values()])
    symbols = subprocess.run(["c++filt"], input="\n".join(f[0].removesuffix(".kd") for f in found),
                             check=True, capture_output=True, text=True).stdout.splitlines()
    out = {re.sub(r"^void |mg::|\(.*", "", s): dict(scratch=int(f[1]), lds=int(f[2]), threads=int(f[3]))
           for s, f in zip(symbols, found)}
    assert len(out) > 100
    return out


def test_fp32_kernels_use_no_scratch(kernels):
    """An accumulator block that is not kept in registers goes through memory
    on every K step."""
    fp32 = {k: v for k, v in kernels.items() if re.match(r"sgemm_|syr2k_|splitk_", k)}
    assert len(fp32) > 60
    assert {k: v["scratch"] for k, v in fp32.items() if v["scratch"]} == {}
