"""Build check: a vector instruction that reads a lane mask (vcc or a scalar pair) stands at least two wait states behind
the vector instruction that wrote it, in every kernel of the library.  gfx950 needs that distance and the compiler keeps it
in the code that it can see; inside an inline asm statement nobody does, and no parity test shows a mask read too early
reliably.  Every source is compiled to assembly for the device and read; nothing runs, no GPU involved."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

from paper_2010_00704_amd import build

WAIT_STATES = 2


def scalars(operands):
    """Scalar registers named in an operand text; vcc counts as one."""
    got = set()
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", operands):
        got |= set(range(int(lo), int(hi) + 1))
    got |= {int(n) for n in re.findall(r"\bs(\d+)\b", operands)}
    if re.search(r"\bvcc(_lo|_hi)?\b", operands):
        got.add("vcc")
    return got


def early_reads(lines):
    """Vector instructions that read a scalar register which a vector instruction wrote too shortly before."""
    found, written = [], []                  # written: (registers, wait states since), youngest last
    kernel = ""
    for line in lines:
        text = line.split(";")[0].strip()
        if re.match(r"[A-Za-z_.][\w.$]*:$", text):
            if text.startswith("_Z"):
                kernel = text[:-1]
                written = []
            continue                         # (falling through a label keeps what was written)
        if not text or text[0] == ".":
            continue
        op = text.split()[0]
        args = text[len(op):].split(",")
        reads, writes = set(), set()
        if op.startswith("v_"):
            if op.startswith("v_cmp"):
                writes, reads = scalars(args[0]), scalars(",".join(args[1:]))
            elif "_co_" in op or op.startswith(("v_mad_i64", "v_mad_u64", "v_div_scale")):
                writes, reads = scalars(args[1]), scalars(",".join(args[2:]))
            elif op.startswith(("v_readlane", "v_readfirstlane")):
                writes, reads = scalars(args[0]), scalars(",".join(args[1:]))
            else:
                reads = scalars(",".join(args[1:]))
            for regs, age in written:
                if regs & reads:
                    found.append("%s: %s" % (kernel, text))
                    break
        elif op.startswith("s_") and op != "s_nop" and args:
            gone = scalars(args[0])          # written anew by a scalar instruction: no longer the vector's result
            written = [(regs - gone, age) for regs, age in written]
        step = 1 + int(args[0]) if op == "s_nop" else 1
        written = [(regs, age + step) for regs, age in written if regs and age + step < WAIT_STATES]
        if writes:
            written.append((writes, 0))
    return found


def test_the_reader_sees_an_early_read():
    early = ["_Zk:", "v_cmp_le_f32_e32 vcc, 0, v1", "v_addc_co_u32 v0, vcc, v0, v0, vcc"]
    assert len(early_reads(early)) == 1
    assert not early_reads(early[:2] + ["s_nop 1"] + early[2:])
    assert len(early_reads(early[:2] + ["s_nop 0"] + early[2:])) == 1
    assert not early_reads(["v_cmp_le_f32_e64 s[2:3], 0, v1", "v_mov_b32_e32 v4, v5", "v_mov_b32_e32 v6, v5",
                            "v_cndmask_b32_e64 v0, 0, 1, s[2:3]"])
    assert not early_reads(["v_cmp_le_f32_e64 s[2:3], 0, v1", "s_and_b64 s[2:3], s[2:3], vcc", "v_writelane_b32 v0, s2, 1"])


def test_no_mask_is_read_early(tmp_path):
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    root = os.path.dirname(os.path.dirname(os.path.abspath(build.__file__)))
    include = ["-I", os.path.join(root, "include"), "-I", os.path.join(root, "paper_2010_00704_amd", "csrc")]

    def read(src):
        out = str(tmp_path / (os.path.basename(src) + ".s"))
        rc, log = build._run([build.HIPCC] + flags + ["--cuda-device-only", "-S"] + include + [src, "-o", out])
        assert rc == 0, log
        with open(out) as f:
            return early_reads(f)

    with ThreadPoolExecutor(max_workers=8) as pool:
        found = [hit for hits in pool.map(read, build.sources()) for hit in hits]
    assert not found, "%d masks read early, the first: %s" % (len(found), found[:5])
