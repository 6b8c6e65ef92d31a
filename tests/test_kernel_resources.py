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


def launches(name):
    """{configuration id: [(launcher or kernel, template arguments), ...]} of a
    source file's dispatch over configurations."""
    from paper_2305_18236_amd import build
    text = open(os.path.join(build.CSRC, name)).read()
    out = {}
    for m in re.finditer(r"case (\d+):(.*?)(?=\n    case |\n    default)", text, re.S):
        found = re.findall(r"(launch_\w+_(?:cfg|direct|skinny)|gemm_\w+_ring_kernel)<([^<>]*)>", m.group(2))
        if found:
            out.setdefault(int(m.group(1)), found)
    return out


def names(launcher, args, kind):
    """Pattern of the kernels a launcher's template arguments instantiate."""
    a = [x.strip().replace("TERMS", kind) for x in args.split(",")]
    if launcher == "launch_sgemm_cfg":
        a = (a + ["false", "1"][len(a) - 5:]) if len(a) < 7 else a
        return rf"sgemm_mfma_kernel<{', '.join(a[:5])}, \w+, \w+, {a[5]}, {a[6]}>"
    if launcher == "launch_bf16_cfg":
        return rf"gemm_bf16_kernel<{', '.join(a[:5])}, \w+, \w+, {a[5]}>"
    if launcher == "launch_bf16_direct":
        return rf"gemm_bf16_direct_kernel<{', '.join(a[:5])}>"
    if launcher.endswith("ring_kernel"):
        return rf"{launcher}<{', '.join(a)}>"
    kernel = {"cfg": "", "direct": "direct_", "skinny": "skinny_"}[launcher.rsplit("_", 1)[1]]
    return rf"gemm_{launcher.split('_')[1]}_{kernel}kernel<{', '.join(a)}>"


@pytest.mark.parametrize("path,source,kind", [(0, "gemm_f32.hip", ""), (1, "gemm_bf16.hip", "3"), (2, "gemm_bf16.hip", "1"),
                                              (4, "gemm_bf16.hip", "16"), (3, "gemm_fp8.hip", ""), (5, "gemm_i8.hip", "")])
def test_blocking_model_knows_waves_and_lds(kernels, path, source, kind):
    """The planner's waves and LDS bytes of every configuration (the 16-bit
    direct ones on planes) are those of the kernel it launches."""
    from paper_2305_18236_amd import _native, blocking
    table, seen = launches(source), set()
    for c in blocking.library_configs(_native, path):
        if path == 0 and 8 <= c.id <= 11:   # unpacked and vector-ALU tiles: not planned
            continue
        for launcher, args in table[c.id]:
            if launcher == "launch_bf16_cfg" and c.bk == 64:
                continue                     # without planes
            pattern = names(launcher, args, kind)
            match = [v for k, v in kernels.items() if re.fullmatch(pattern, k)]
            assert match, (c.id, pattern)
            seen.add(c.id)
            ring = launcher.endswith("ring_kernel")
            lds = blocking.RING_STAGES * (c.bm + c.bn) * 128 if ring else c.lds_bytes
            assert not ring or c.ring(1, 1024), c.id
            assert {(v["threads"], v["lds"]) for v in match} == {(64 * c.waves, lds)}, (c.id, pattern)
            if len(args.split(",")) == 6 and launcher == "launch_bf16_direct":   # its last argument: the ring's stages
                (ring,) = [v for k, v in kernels.items()
                           if k == f"gemm_bf16_ring_kernel<{args.replace('TERMS', kind)}>"]
                assert c.ring(1, 64) and (ring["threads"], ring["lds"]) == (64 * c.waves, 5 * (c.bm + c.bn) * 128)
    assert len(seen) == _native.mg_num_configs(path) - (4 if path == 0 else 0)
