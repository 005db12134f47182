"""What the compiler made of kernels that rely on their registers, read from the metadata of the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_1907_03329_amd import binding, build

READELF = os.environ.get("LLVM_READELF", "/opt/rocm/llvm/bin/llvm-readelf")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    """{kernel: (bytes of scratch per lane, bytes of static LDS, registers)}"""
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    data = open(binding.LIB_PATH, "rb").read()
    d, out, at = tmp_path_factory.mktemp("code_objects"), {}, data.find(BUNDLE)
    while at >= 0:      # one bundle per translation unit: entries of offset, size, length of the triple, triple
        n, pos = struct.unpack_from("<Q", data, at + len(BUNDLE))[0], at + len(BUNDLE) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<3Q", data, pos)
            triple = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in triple or not size:
                continue
            path = d / "code"
            path.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            names = re.findall(r"^\s+\.name:\s+(_Z\S+)\s*$", notes, re.M)
            sizes = [[int(v) for v in re.findall(rf"^\s+\.{kind}:\s+(\d+)\s*$", notes, re.M)]
                     for kind in ("private_segment_fixed_size", "group_segment_fixed_size", "vgpr_count")]
            assert all(len(names) == len(s) for s in sizes)
            out.update(zip(names, zip(*sizes)))
        at = data.find(BUNDLE, at + 1)
    return out


@pytest.fixture(scope="module")
def resources(notes):
    """{kernel: (bytes of scratch per lane, bytes of static LDS)}"""
    return {k: v[:2] for k, v in notes.items()}


def test_rows_requested_ahead_stay_in_registers(resources):
    """Smoothing recursions: a wave's requests for observations, chunks of steps ahead, have constant places.  In scratch
    (as when their steps are calls and not inlined) every one of them is waited for: 43 -> 82 us for 240 steps at period 1."""
    kernels = {k: v for k, (v, _) in resources.items() if re.search(r"es_(forward|forward_long|backward)_kernel", k)}
    assert len(kernels) == 14       # forward: 9 of seasonalities and steps per group, 2 for long periods; reverse: 3
    assert not {k: v for k, v in kernels.items() if v}


def test_static_lds_stays_within_128_kb(resources):
    """An output-stage shape with 135 KB of static LDS has launched without an error and computed wrong outputs."""
    assert not {k: lds for k, (_, lds) in resources.items() if lds > 128 * 1024}


def test_forward_workgroups_of_several_streams_share_a_compute_unit(notes):
    """4-series forward kernels, eight waves each: two fit into the 160 KB and 512 registers a SIMD, so that streams run side by side."""
    kernels = {k: v for k, v in notes.items() if re.search(r"lstm_forward_narrow_kernel|lstm_forward_together_kernelI(Li\d+E){2}Lb\dELi0E", k)}
    assert len(kernels) == 14 * (4 + 2)
    assert not {k: (lds, registers) for k, (_, lds, registers) in kernels.items() if lds > 80 * 1024 or registers > 128}


def test_twelve_wave_workgroups_have_a_compute_unit_each(notes):
    kernels = {k: lds for k, (_, lds, _) in notes.items() if re.search(r"lstm_backward_(narrow_kernelI(Li\d+E){2}Lb\dELb1E|together)", k)}
    assert len(kernels) == 14 * (2 + 2)
    assert not {k: lds for k, lds in kernels.items() if lds <= 80 * 1024}


def test_recurrences_of_4_series_layers_have_no_scratch(resources):
    kernels = {k: v for k, (v, _) in resources.items() if re.search(r"lstm_(forward|backward)_(narrow|together)_kernel", k)}
    assert len(kernels) == 14 * (4 + 4 + 5 + 2)
    assert not {k: v for k, v in kernels.items() if v}
