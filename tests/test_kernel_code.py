"""The machine code of kernels whose compilation once went wrong without any
wrong result: operands spilled into vector lanes, loads no longer issued
ahead.  Reads the gfx950 code of the built library; the bounds lie between the
counts of the slow and of the present code."""

import os
import re
import shutil
import subprocess

import pytest

import paper_2401_06132_amd as frmi

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """blocks(name): the instruction lists between branches of the kernels whose mangled name holds `name`."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(frmi.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(frmi.LIB_PATH)], cwd=d, check=True, capture_output=True)
    objs = [str(d / f) for f in sorted(os.listdir(d)) if "gfx950" in f]
    syms = {}
    for o in objs:
        for line in subprocess.run([OBJDUMP, "-t", o], check=True, capture_output=True, text=True).stdout.splitlines():
            if " F .text" in line:
                syms[line.split()[-1]] = o

    def blocks(name):
        found = [s for s in syms if name in s]
        assert found, name
        out = []
        for s in found:
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + s, syms[s]], check=True,
                                  capture_output=True, text=True).stdout
            ops = [m.group(1) for m in re.finditer(r"^\s+([sv]_\S.*|ds_\S.*|global_\S.*|scratch_\S.*)$", text, re.M)]
            cur = []
            for op in ops:
                cur.append(op)
                if op.startswith(("s_cbranch", "s_branch", "s_barrier")):
                    out.append(cur)
                    cur = []
            out.append(cur)
        return out

    return blocks


def count(block, prefix):
    return sum(op.startswith(prefix) for op in block)


@pytest.mark.parametrize("diag", [0, 1])
def test_hex_fp64_p4_projection_operands(code, diag):
    """hex_volume<4, double> with flux anti-aliasing: the y projection once read its operators back from vector
    lanes for every line (406 lane reads)."""
    assert max(count(b, "v_readlane") for b in code("hex_volumeILi4EdLi1ELi64ELb%dELb0ELb1ELb0ELb0E" % diag)) < 200


@pytest.mark.parametrize("diag", [0, 1])
def test_hex_fp64_p4_face_fields_read_ahead(code, diag):
    """hex_volume<4, double> with surface-flux anti-aliasing: the face quadrature points once waited for each LDS
    read by itself (53 waits for 56 reads, once per axis)."""
    face = [b for b in code("hex_volumeILi4EdLi1ELi64ELb%dELb0ELb1ELb1ELb0E" % diag)
            if count(b, "v_rcp") and 40 <= count(b, "ds_read") <= 100]
    assert len(face) == 3  # one per axis
    for b in face:
        assert count(b, "s_waitcnt") < 30, (count(b, "ds_read"), count(b, "s_waitcnt"))


def test_hex_warp_fp32_p4_one_wave_groups(code):
    """Curved hexahedra, FP32 p = 4: one element per one-wave workgroup (five per four waves were 19% slower on
    small meshes)."""
    code("hex_volumeILi4EfLi1ELi64ELb0ELb0ELb1ELb0ELb1E")


def test_pyr_fp64_p4_projection_loads_ahead(code):
    """dense_volume_mf<pyramid, 4, double> with flux anti-aliasing: the projection once waited for most operator
    loads right after issuing them."""
    proj = [b for b in code("dense_volume_mfILi3ELi4EdLi1ELi256ELb1E") if count(b, "v_mfma") >= 90]
    assert len(proj) == 1
    waits = [op for op in proj[0] if op.startswith("s_waitcnt") and "vmcnt(0)" in op]
    assert len(waits) < 10, len(waits)
