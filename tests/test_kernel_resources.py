"""Registers of the built kernels, from the metadata the compiler leaves in the library's code object; when it is out of date."""
import json
import os
import subprocess

import msgpack
import pytest

from paper_2511_22880_amd import build


def _kernels():
    """{kernel symbol: metadata} of every AMDGPU code object in the library (the notes hold MessagePack)."""
    data, found, at = open(build.LIB, "rb").read(), {}, 0
    while (at := data.find(b"AMDGPU\0\0", at)) >= 0:  # name of an NT_AMDGPU_METADATA note: sizes and type stand before it
        size, kind = (int.from_bytes(data[at - k:at - k + 4], "little") for k in (8, 4))
        if kind == 32:
            for k in msgpack.unpackb(data[at + 8:at + 8 + size])["amdhsa.kernels"]:
                found[k[".name"]] = k
        at += 8
    return found


@pytest.mark.parametrize("kernel, most", [
    # up to rank 64 (128 registers): the loop of 16 x 4 rank rows and 32 tokens takes them all but for one or two
    ("k_shrink_prefillE", 2),
    ("k_shrink_mixedILb0E", 2),
    ("k_shrink_prefill_anyE", 12),
    ("k_shrink_mixedILb1E", 12),
    ("k_apply_fusedE", 0),
    ("k_decode_fusedE", 0),
    # 254 of 256 registers; its waits count memory operations, and a spill's are among them
    ("k_linear_loraE", 0),
    ("k_shrink_halvesE", 0),
    ("k_expand_partsE", 0),
    # up to 126 of the 128 that four work groups on a compute unit leave; their waits count memory operations too
    ("k_expand_bigILb0E", 0),
    ("k_expand_bigILb1E", 0),
    ("k_expand_walkE", 0),  # 245 of 256
    ("k_expand_mixedILNS_6SlicesE0E", 0),
    ("k_expand_mixedILNS_6SlicesE1E", 0),
    ("k_linear_roundsILi4ELi4ELi2E", 0),  # 244 of 256
])
def test_spilled_registers(kernel, most):
    """A register spilled in a unit's k loop is a trip to memory in every pass of it."""
    hits = [k for name, k in _kernels().items() if "4lora" in name and kernel in name]
    assert len(hits) == 1
    assert hits[0][".vgpr_spill_count"] <= most, hits[0][".vgpr_spill_count"]


def _dynamic_symbols():
    """(offset of the code object, its sections' headers, symbol's entry, name) of every dynamic symbol of the library's AMDGPU code."""
    data, at = open(build.LIB, "rb").read(), 0
    num = lambda at, size: int.from_bytes(data[at:at + size], "little")
    while (at := data.find(b"\x7fELF", at)) >= 0:
        if num(at + 18, 2) == 224:  # EM_AMDGPU
            sections = [at + num(at + 40, 8) + k * num(at + 58, 2) for k in range(num(at + 60, 2))]
            for sec in sections:
                if num(sec + 4, 4) != 11:  # SHT_DYNSYM
                    continue
                names = at + num(sections[num(sec + 40, 4)] + 24, 8)
                for sym in range(at + num(sec + 24, 8), at + num(sec + 24, 8) + num(sec + 32, 8), 24):
                    name = data[names + num(sym, 4):data.index(b"\0", names + num(sym, 4))].decode()
                    yield num, at, sections, sym, name
        at += 4


def _code_bytes(kernel):
    hits = [num(sym + 16, 8) for num, _, _, sym, name in _dynamic_symbols() if "4lora" in name and kernel in name and not name.endswith(".kd")]
    assert len(hits) == 1
    return hits[0]


def test_expand_kernels_that_read_complete_v_hold_no_code_that_adds_slices_up():
    """With it, never run, they took other registers, and a mixed launch 4 % longer."""
    assert _code_bytes("k_expandILb0ELb0E") < _code_bytes("k_expand_partsE")
    assert _code_bytes("k_expand_mixedILNS_6SlicesE0E") < _code_bytes("k_expand_mixedILNS_6SlicesE1E")


def test_kernels_whose_profiles_are_quoted_exist():
    """bench.py names the kernel of a phase from profiles/measured.json."""
    with open(os.path.join(build.ROOT, "profiles", "measured.json")) as f:
        quoted = json.load(f)["phase_kernels"].values()
    names = subprocess.run(["c++filt", *_kernels()], capture_output=True, text=True, check=True).stdout.splitlines()
    assert set(quoted) <= {name.removeprefix("void ").split("(")[0] for name in names}


def _preloaded():
    """{kernel symbol: scalar registers of arguments that are there when a wavefront starts} from the kernel descriptors."""
    found = {}
    for num, at, sections, sym, name in _dynamic_symbols():
        if name.endswith(".kd"):
            home = sections[num(sym + 6, 2)]
            kd = at + num(home + 24, 8) + num(sym + 8, 8) - num(home + 16, 8)
            found[name[:-3]] = num(kd + 58, 2) & 127
    return found


@pytest.mark.parametrize("kernel, dwords", [
    # pointers and 64-bit strides take two; an argument that no longer fits the 14 ends the list, as does a struct
    ("k_decode_fusedE", 14),
    ("k_shrinkE", 13),
    ("k_shrink_wideILi8E", 14),
    ("k_expandILb0ELb0E", 12),
    ("k_apply_fusedE", 14),
    ("k_shrink_prefillE", 14),
    ("k_linear_smallILi4ELi4ELi2E", 14),
    ("k_linear_loraE", 12),
])
def test_arguments_that_arrive_in_registers(kernel, dwords):
    """The unit list, the arena and x (k_linear_lora: the rows, the pieces and the arena) need no load of their own."""
    hits = [n for name, n in _preloaded().items() if "4lora" in name and kernel in name]
    assert hits == [dwords]


@pytest.mark.parametrize("newer", ["a source", "a header", "the compile command"])
def test_a_library_older_than_what_it_is_built_from_is_stale(monkeypatch, newer):
    path = {"a source": build.SOURCES[0], "a header": build.HEADERS[0], "the compile command": build.__file__}[newer]
    times = {build.LIB: 2.0}
    monkeypatch.setattr(os.path, "getmtime", lambda p: times.get(p, 1.0))
    assert not build.is_stale()
    times[os.path.abspath(path)] = 3.0
    assert build.is_stale()
