"""What the compiler made of the kernels, read from the built library (no GPU): the registers it spilled and the
scratch it takes, where the code says that there is none."""
import os
import re
import struct
import subprocess

import pytest

from paper_2402_16801_amd import binding, build

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: {field: value}} from the metadata of the device code in the library."""
    if not os.path.exists(binding.LIB_PATH):
        build.build_all()
    blob, found = open(binding.LIB_PATH, "rb").read(), {}
    where = tmp_path_factory.mktemp("code")
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob)):
        pos = at + 24
        (count,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" not in target:
                continue
            code = where / f"{at}.o"
            code.write_bytes(blob[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(code)], capture_output=True, text=True, check=True).stdout
            for entry in notes.split("  - .agpr_count:")[1:]:
                values = dict(re.findall(r"^ +\.(\w+): +(\S+)$", entry, re.M))
                found[values["name"].strip("'")] = {k: int(v) for k, v in values.items() if v.isdigit()}
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(found) > 100 and len(names) == len(found)
    return {re.sub(r"\(.*", "", n).replace("void ", ""): v for n, v in zip(names, found.values())}


def _spills(kernels, pattern):
    return {n: (k["sgpr_spill_count"], k["vgpr_spill_count"]) for n, k in kernels.items() if re.match(pattern, n)}


def test_floors_generated_by_blocks_spill_nothing(kernels):
    """A block covers a floor in one pass: seen as a loop, the compiler kept every kind of floor's constants in front of it."""
    spills = _spills(kernels, r"cf::(kf_reset|kf_import|kf_mutate_noise)<(\w+, )?320>")
    assert len(spills) == 5 and set(spills.values()) == {(0, 0)}, spills


def test_generators_of_the_full_game_spill_no_vector_register(kernels):
    """At the wavefronts per SIMD that they are bounded to (csrc/floor_route.hpp)."""
    spills = _spills(kernels, r"cf::(kf_reset|kf_import|kf_drain|kf_mutate_noise)<")
    assert len(spills) == 14 and {v for _, v in spills.values()} == {0}, spills


def test_step_kernels_use_no_scratch(kernels):
    scratch = {n: k["private_segment_fixed_size"] for n, k in kernels.items() if re.match(r"cx::k_step<|cf::kf_step<", n)}
    assert len(scratch) > 20 and set(scratch.values()) == {0}, scratch


def test_float_rollouts_of_sixteen_lanes_leave_registers_for_five_blocks(kernels):
    """512 vector registers per SIMD, handed out by eights: with more than 96 a compute unit holds four blocks, 16,384 environments on the chip."""
    assert kernels["cx::k_rollout<16, 2, false>"]["vgpr_count"] <= 96
