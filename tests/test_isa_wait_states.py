"""Wait states between dependent vector instructions on gfx950, in the assembly
of every kernel source.  The compiler keeps them between its own instructions
but does not look inside inline assembly, so its listing is checked as a whole:

* a scalar register or VCC written by a vector instruction (compare, carry,
  lane read) and read by one: 2 wait states (4 as a lane select);
* a vector register written by a vector instruction and read across lanes by
  DPP or a lane swap: 2; by a lane read: 1.

Every instruction in between counts one, ``s_nop n`` n + 1.  And the occupancy
that a kernel's attributes state is one its registers allow."""
import concurrent.futures
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2603_25260_amd import build as B

KERNEL_SOURCES = ["octree.hip", "model.hip", "rc.hip"]
REG = re.compile(r"\b([sv])(\d+)\b|\b([sv])\[(\d+):(\d+)\]|\b(vcc)(_lo|_hi)?\b")
CARRY_OUT = re.compile(r"v_(add|addc|sub|subb|subrev|subbrev)_co_|v_mad_[ui]64_")
LANE = re.compile(r"v_(readlane|writelane)_b32")
SWAP = re.compile(r"v_permlane(16|32)_swap")
READ_LANE = re.compile(r"v_read(first)?lane")


def regs(text):
    out = set()
    for m in REG.finditer(text):
        if m.group(6):
            out |= {"vcc_lo", "vcc_hi"} if not m.group(7) else {"vcc" + m.group(7)}
        elif m.group(1):
            out.add(m.group(1) + m.group(2))
        else:
            out |= {f"{m.group(3)}{k}" for k in range(int(m.group(4)), int(m.group(5)) + 1)}
    return out


def violations(body):
    """(distance, needed, writer, reader) of every pair that is too close."""
    bad, age = [], {}  # age: register -> (wait states since written by a vector instruction, writer)
    for line in body.split("\n"):
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", rest)]
        if op == "s_nop":
            step = int(args[0], 0) + 1
        else:
            step = 1
            vector = op.startswith("v_") and not op.startswith("v_mfma")
            ndef = 2 if CARRY_OUT.match(op) else 1
            defs, uses = regs(",".join(args[:ndef])), args[ndef:]
            if SWAP.match(op):  # both operands are read and written
                defs, uses = regs(rest), args
            close = set()
            if vector:
                for k, a in enumerate(uses):
                    for r in regs(a):
                        if r not in age:
                            continue
                        need = 0
                        if r[0] == "s" or r.startswith("vcc"):
                            need = 4 if LANE.match(op) and k == 1 else 2
                        elif READ_LANE.match(op):
                            need = 1
                        elif re.search(r"\b(quad_perm|row_|wave_)", rest) and k == 0:
                            need = 2
                        elif SWAP.match(op):
                            need = 2
                        if age[r][0] < need:
                            close.add((age[r][0], need, age[r][1], line))
            bad += sorted(close)
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                age = {}
                continue
        age = {r: (n + step, w) for r, (n, w) in age.items() if n + step < 4}
        if op != "s_nop":
            for r in defs:
                age.pop(r, None)
            if vector:
                age.update({r: (0, line) for r in defs})
    return bad


def _asm(src, out):
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-Wall")]
    cmd = [B.HIPCC, *flags, "--cuda-device-only", "-S", "-o", out, os.path.join(B.CSRC, src)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return open(out).read(), r.stderr


@pytest.fixture(scope="module")
def asm():
    if not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as d:
        with concurrent.futures.ThreadPoolExecutor(len(KERNEL_SOURCES)) as ex:
            texts = list(ex.map(lambda s: _asm(s, os.path.join(d, s + ".s")), KERNEL_SOURCES))
    return dict(zip(KERNEL_SOURCES, texts))


@pytest.mark.parametrize("src", KERNEL_SOURCES)
def test_dependent_vector_instructions_keep_their_distance(asm, src):
    kernels = re.findall(r"^(_Z\w+):(.*?)^\.Lfunc_end\d+:", asm[src][0], re.S | re.M)
    assert kernels
    bad = [(name, *v) for name, body in kernels for v in violations(body)]
    assert not bad, (len(bad), bad[:5])


@pytest.mark.parametrize("src", KERNEL_SOURCES)
def test_stated_occupancy_is_reached(asm, src):
    missed = [line for line in asm[src][1].split("\n") if "failed to meet occupancy target" in line]
    assert not missed, missed[:3]


@pytest.mark.parametrize("body,n", [
    ("v_cmp_le_u32_e32 vcc, v1, v2\nv_addc_co_u32_e32 v0, vcc, v3, v4, vcc", 1),
    ("v_cmp_le_u32_e32 vcc, v1, v2\ns_nop 1\nv_addc_co_u32_e32 v0, vcc, v3, v4, vcc", 0),
    ("v_cmp_le_u32_e32 vcc, v1, v2\nv_mov_b32_e32 v5, v6\nv_cndmask_b32_e32 v0, v3, v4, vcc", 1),
    ("v_cmp_le_u32_e32 vcc, v1, v2\nv_mov_b32_e32 v5, v6\nv_mov_b32_e32 v7, v6\nv_cndmask_b32_e32 v0, v3, v4, vcc", 0),
    ("v_readlane_b32 s4, v1, s5\nv_add_u32_e32 v2, s4, v3", 1),
    ("v_max_u32_e32 v1, v2, v3\nv_readlane_b32 s4, v1, s5", 1),
    ("v_max_u32_e32 v1, v2, v3\ns_ff1_i32_b64 s5, s[6:7]\nv_readlane_b32 s4, v1, s5", 0),
    ("v_max_u32_e32 v1, v2, v3\nv_nop\nv_min_u32_dpp v4, v1, v5 wave_shr:1 row_mask:0xf bank_mask:0xf", 1),
    ("v_add_u32_e32 v1, v2, v3\nv_mov_b32_e32 v4, v5\nv_permlane16_swap_b32_e32 v1, v6", 1),
    ("v_add_u32_e32 v1, v2, v3\ns_nop 1\nv_permlane16_swap_b32_e32 v1, v6", 0),
    ("v_cmp_le_u32_e64 s[0:1], v1, v2\ns_and_b64 vcc, s[0:1], s[2:3]", 0),
])
def test_detector(body, n):
    assert len(violations(body)) == n
