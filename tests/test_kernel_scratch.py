"""Scratch memory (spilled registers) of the built attention kernels, from the
metadata of the code objects in libfqvit.so: a kernel that spills inside its
tile loop writes and reads device memory that no output needs."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 ELF images of the offload bundles in a shared library."""
    at = data.find(BUNDLE)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + length] and size:
                yield data[at + off:at + off + size]
            pos += 24 + length
        at = data.find(BUNDLE, at + 24)


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """(bytes of scratch a lane, vector registers) of every kernel, by demangled
    name."""
    from paper_2111_13824_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        pytest.fail("libfqvit.so is not built")
    with open(binding.LIB_PATH, "rb") as f:
        data = f.read()
    names, sizes = [], []
    path = tmp_path_factory.mktemp("code") / "object.elf"
    for elf in _code_objects(data):
        path.write_bytes(elf)
        text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                              check=True).stdout
        # one block per kernel; its keys are in alphabetical order
        for block in re.split(r"\n  - (?=\.)", text)[1:]:
            name = re.search(r"^\s*\.name:\s+(_Z\S+)$", block, re.M)
            size = re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)
            regs = re.search(r"\.vgpr_count:\s+(\d+)", block)
            if name and size and regs:
                names.append(name.group(1))
                sizes.append((int(size.group(1)), int(regs.group(1))))
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    return {n.split("(fqvit")[0].replace("void ", "").replace("fqvit::lis::", ""): s
            for n, s in zip(plain, sizes)}


@pytest.fixture(scope="module")
def scratch(resources):
    return {n: s for n, (s, _) in resources.items()}


def _spilling(scratch, kernel):
    found = {n: s for n, s in scratch.items() if n.startswith(kernel + "<")}
    assert found, f"no instance of {kernel} in the library"
    return {n: s for n, s in found.items() if s}


def test_qk_long_rows_hold_their_logits(scratch):
    """Attention from Q and K on the float path (fourth template argument): no
    instance spills, the longest rows included."""
    bad = {n: s for n, s in _spilling(scratch, "lis_qk_kernel").items()
           if n.split("<")[1].split(",")[3].strip() == "true"}
    assert not bad, bad


def test_qk_integer_rows_of_197_keys_hold_their_state(scratch):
    """The integer path holds a 32-bit and an 8-bit value per key: rows of 193
    to 208 keys without a bias (seven chunks, the last one half) fit the
    registers of three wavefronts per SIMD, full rows of 224 nearly do."""
    spill = {n: s for n, s in scratch.items()
             if n.startswith("lis_qk_kernel<") and n.split(",")[3].strip() == "false"}
    assert spill
    for n, s in spill.items():
        args = [x.strip(" >") for x in n.split("<")[1].split(",")]
        nc, half, bias = int(args[0]), args[2] == "true", args[6] == "true"
        limit = 0 if nc < 7 or (half and not bias) else 80
        assert s <= limit, (n, s)


def test_qk_integer_rows_keep_their_wavefronts(resources):
    """Integer path, rows of three and four chunks: at most the 96 and 128
    registers that five and four wavefronts a SIMD leave each.  With 129, 1000
    units of 100 x 100 took 19.4 us instead of 17.4."""
    seen = 0
    for n, (_, regs) in resources.items():
        args = [x.strip(" >") for x in n.split("<")[-1].split(",")]
        if n.startswith("lis_qk_kernel<") and args[3] == "false" and args[0] in ("3", "4"):
            assert regs <= (96 if args[0] == "3" else 128), (n, regs)
            seen += 1
    assert seen


def test_unit_kernels_hold_their_rows(scratch):
    """The unit kernel (fused head and stored codes): no instance spills."""
    bad = _spilling(scratch, "lis_unit_kernel")
    assert not bad, bad
