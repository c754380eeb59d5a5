"""What the compiler made of the kernels (read from the library built here): registers spilled to memory and the number of
vector instructions, for kernels whose time follows them.  A limit stands a little above what the kernel has."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

from paper_2402_03694_amd import build as hip_build

LLVM = "/opt/rocm/llvm/bin/"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    """The device code objects of a library: every bundle's entries for the GPU."""
    with open(path, "rb") as f:
        data = f.read()
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                yield data[at + offset:at + offset + size]
            p += 24 + length
        at = data.find(MAGIC, at + 1)


def _run(*cmd, **kw):
    return subprocess.run(cmd, check=True, capture_output=True, text=True, **kw).stdout


@pytest.fixture(scope="module")
def kernels():
    """{name: {"spilled": vector registers, "vector": vector instructions}}"""
    if not all(os.path.exists(LLVM + t) for t in ("llvm-readelf", "llvm-objdump")):
        pytest.skip("no llvm-readelf or llvm-objdump")
    found = {}
    for code in _code_objects(hip_build.build(force=False)):
        with tempfile.NamedTemporaryFile(suffix=".o") as f:
            f.write(code)
            f.flush()
            for block in _run(LLVM + "llvm-readelf", "--notes", f.name).split("\n  - "):
                name, spilled = re.search(r"\.symbol: +'?(\w+)\.kd", block), re.search(r"\.vgpr_spill_count: +(\d+)", block)
                if name:
                    found[name.group(1)] = {"spilled": int(spilled.group(1)), "vector": 0}
            name = None
            for line in _run(LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", f.name).splitlines():
                head = re.match(r"[0-9a-f]+ <(\w+)>:", line)
                if head:
                    name = head.group(1)
                elif name in found and line.lstrip().startswith("v_"):
                    found[name]["vector"] += 1
    plain = _run("c++filt", input="\n".join(found)).splitlines()
    return {n.replace("(anonymous namespace)::", "").replace("void ", "").split("(")[0]: v for n, v in zip(plain, found.values())}


@pytest.mark.parametrize("name,most", [("featurize_wave<8, false>", 1230), ("featurize_wave<16, false>", 3200)])
def test_vector_instructions(kernels, name, most):
    """The one-lane feature kernel up to 16 packets shares its comparisons between the statistics."""
    assert kernels[name]["vector"] <= most, kernels[name]


@pytest.mark.parametrize("name", ["featurize_wave<8, false>", "featurize_wave<16, false>", "featurize_wave<32, false>", "featurize_parts<8>",
                                  "featurize_parts<32>"] + ["mlp_wide_layer<%s>" % t for t in (
                                      "0, false, 0", "0, true, 0", "1, false, 0", "1, true, 0", "2, false, 0", "2, true, 0", "2, false, 1", "2, true, 1",
                                      "2, true, 2")] + [
                                      "mlp_rows<%s>" % t for t in ("4, 4, false", "8, 4, false", "12, 4, false", "16, 4, true", "16, 4, false", "4, 8, false",
                                                                   "8, 8, false", "12, 8, false", "16, 8, true")] + ["mlp_fused"] + [
                                      "forest_trees<%d, %d, false>" % t for t in ((4, 4), (4, 3), (2, 4), (2, 3), (1, 4))] + [
                                      "featurize_forest<128, 8, 0, 0, 8, %s>" % t for t in ("true", "false")])
def test_no_spills(kernels, name):
    assert kernels[name]["spilled"] == 0, kernels[name]


@pytest.mark.parametrize("name,most", [
    ("mlp_wide_layer<2, false, 2>", 4),   # header bits of 1 to 7 a packet, K streamed: outside the loop over K
    ("mlp_rows<16, 8, false>", 4),        # 14 with as many operands in accumulation registers as the narrower forms, and 4 % slower
    ("forest_trees<4, 4, true>", 4), ("forest_trees<4, 3, true>", 4), ("forest_trees<2, 4, true>", 4), ("forest_trees<2, 3, true>", 4),
    ("forest_trees<1, 4, true>", 4),      # behind the walk, the softmax in binary64
    ("featurize_forest<128, 8, 0, 0, 16, true>", 16), ("featurize_forest<128, 8, 0, 0, 16, false>", 16)])  # the feature phase of 16 packets
def test_few_spills(kernels, name, most):
    assert kernels[name]["spilled"] <= most, kernels[name]


SHORT_FORMS = ["featurize_forest_few<%s, 16, %s>" % (t, r) for t in ("128, 8, 0, 0", "128, 4, 5, 2", "64, 8, 3, 1") for r in ("true", "false")] + [
    "mlp_few<%d, %d, %d, sfsmall::%s>" % (k, n1, n2, g) for k in (4, 8) for n1 in (1, 2) for n2 in (1, 2) for g in ("GateRows", "NoGate")] + [
    "featurize_long<2>", "mlp_wide_last<true>", "mlp_last_layer<1>", "mlp_last_layer<2>", "f32_mlp<sfsmall::GateRows>",
    "f32_mlp<sfsmall::NoGate>"]


@pytest.mark.parametrize("name", SHORT_FORMS)
def test_no_spills_short_forms(kernels, name):
    """The forms for few rows, small batches and the wide models' last layer, which hold rings of operands in registers."""
    assert kernels[name]["spilled"] == 0, kernels[name]


@pytest.mark.parametrize("name,most", [("featurize_long<4>", 14),   # four blocks a unit: 128 registers
                                       ("mlp_wide_last<false>", 8)])  # once a tile, around the last layer
def test_few_spills_short_forms(kernels, name, most):
    assert kernels[name]["spilled"] <= most, kernels[name]


def test_slow_model_has_no_arrays_in_memory():
    """Bytes a lane of memory that are no spills: an array the compiler did not keep in registers."""
    held = {}
    for code in _code_objects(hip_build.build(force=False)):
        with tempfile.NamedTemporaryFile(suffix=".o") as f:
            f.write(code)
            f.flush()
            for block in _run(LLVM + "llvm-readelf", "--notes", f.name).split("\n  - "):
                name = re.search(r"\.symbol: +'?(\w+)\.kd", block)
                if name and ("mlp_" in name.group(1)):
                    count = lambda what: int(re.search(r"\.%s: +(\d+)" % what, block).group(1))
                    held[name.group(1)] = count("private_segment_fixed_size"), count("vgpr_spill_count")
    assert len(held) > 40
    assert not {n: v for n, v in held.items() if v[0] and not v[1]}
