"""Registers of the built kernels, from the metadata the compiler leaves in the library's code object; when it is out of date."""
import os

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
])
def test_spilled_registers(kernel, most):
    """A register spilled in a unit's k loop is a trip to memory in every pass of it."""
    hits = [k for name, k in _kernels().items() if "4lora" in name and kernel in name]
    assert len(hits) == 1
    assert hits[0][".vgpr_spill_count"] <= most, hits[0][".vgpr_spill_count"]


@pytest.mark.parametrize("newer", ["a source", "a header", "the compile command"])
def test_a_library_older_than_what_it_is_built_from_is_stale(monkeypatch, newer):
    path = {"a source": build.SOURCES[0], "a header": build.HEADERS[0], "the compile command": build.__file__}[newer]
    times = {build.LIB: 2.0}
    monkeypatch.setattr(os.path, "getmtime", lambda p: times.get(p, 1.0))
    assert not build.is_stale()
    times[os.path.abspath(path)] = 3.0
    assert build.is_stale()
