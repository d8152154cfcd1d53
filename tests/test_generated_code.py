"""The generated code of the kernels: what the compiler may do to a source without a word and no output or an output now and then tells.

Shift amounts of 64-bit shifts:
a 64-bit shift whose amount sits in the last register a wavefront has (the last of its eight-register granule, with none behind it) uses a wrong
amount now and then when other wavefronts share the SIMD: port_round_robin's 88-register kernel, amount in v87, gave one position of sixteen
wrong in one tile of twenty, and only with the chip full.  The compiler does not avoid that register, so the code is looked at.
"""
import functools
import os
import re
import subprocess

import pytest

from paper_2510_19262_amd import build


def _shifts_by_the_last_register(text):
    for name, body, kernel in re.findall(r"^(\w+):\s*; @\1\n(.*?)\.amdhsa_kernel \1\n(.*?)\.end_amdhsa_kernel", text, re.S | re.M):
        last = -(-int(re.search(r"amdhsa_next_free_vgpr (\d+)", kernel)[1]) // 8) * 8 - 1
        for line, amount in re.findall(r"(v_(?:lshlrev|lshrrev|ashrrev)_[bi]64\S* v\[\d+:\d+\], v(\d+), .*)", body):
            if int(amount) == last:
                yield f"{name}: {line}"


def test_the_search_finds_such_a_shift():
    text = ("k: ; @k\n\tv_lshlrev_b64 v[18:19], v{0}, v[44:45]\n\t.amdhsa_kernel k\n\t\t.amdhsa_next_free_vgpr {1}\n\t.end_amdhsa_kernel\n")
    assert list(_shifts_by_the_last_register(text.format(87, 88))) == ["k: v_lshlrev_b64 v[18:19], v87, v[44:45]"]
    assert not list(_shifts_by_the_last_register(text.format(87, 89))) and not list(_shifts_by_the_last_register(text.format(86, 88)))


@functools.lru_cache(maxsize=None)
def _assembly(src):
    flags = [f for f in build.FLAGS if f != "-Wall"] + build.EXTRA_FLAGS.get(src, [])
    return subprocess.run([build.HIPCC, *flags, "-w", "-S", "--cuda-device-only", os.path.join(build.CSRC, src), "-o", "-"], check=True,
                          stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout


@pytest.mark.parametrize("src", build.SOURCES)
def test_no_64_bit_shift_by_the_last_register(src):
    text = _assembly(src)
    assert src == "api.hip" or ".amdhsa_kernel" in text
    assert not list(_shifts_by_the_last_register(text))


@pytest.mark.parametrize("registers", [1, 2])
def test_the_port_kernels_leave_their_last_register_alone(registers):
    body, kernel = re.search(r"^_ZN2rs18port_packed_kernelILb1ELi%dEE\w+:\s*; @\w+\n(.*?)\.amdhsa_kernel (.*?)\.end_amdhsa_kernel" % registers, _assembly("extras.hip"), re.S | re.M).groups()
    last = int(re.search(r"amdhsa_next_free_vgpr (\d+)", kernel)[1]) - 1
    assert last % 8 == 7
    instructions = re.sub(r";.*", "", body)
    for lo, hi in re.findall(r"\bv(?:\[(\d+):)?(\d+)\b", instructions):
        assert int(hi) < last


def test_indices_of_the_list_kernels_are_streamed():
    # a plain store beside them under the same condition would make them plain: 4 194 304 rows of 64 logits, top-6: 209 us streaming, 222 plain
    bodies = re.findall(r"^(_ZN2rs24route_topk_insert_kernel\w+):\s*; @\1\n(.*?)\.amdhsa_kernel \1\n", _assembly("route_topk.hip"), re.S | re.M)
    assert len(bodies) >= 14
    for name, body in bodies:
        assert re.search(r"global_store_dword v.* nt$", body, re.M), name
