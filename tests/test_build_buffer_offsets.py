"""Build check: every access through a buffer descriptor has all of its offset in the vector register and the instruction, none in the
scalar register.  LLVM leaves the scalar offset of the raw buffer builtins out of the bounds check, and these kernels count on that check:
rows past the end of a ragged tile store nothing, words past a tensor's end read as zero.  Every source is compiled to assembly for
the device and read; nothing runs, no GPU involved."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

from paper_2010_00704_amd import build


def scalar_offsets(lines):
    """Buffer accesses with a scalar offset other than zero, and how many accesses there are."""
    found, seen, kernel = [], 0, ""
    for line in lines:
        text = line.split(";")[0].strip()
        if re.match(r"_Z[\w.$]*:$", text):
            kernel = text[:-1]
        if not text.startswith(("buffer_load", "buffer_store", "buffer_atomic")):
            continue
        at = re.search(r"\b(?:s|ttmp)\[\d+:\d+\],\s*(\S+)", text)
        assert at, text
        seen += 1
        if at.group(1) != "0":
            found.append("%s: %s" % (kernel, text))
    return found, seen


def test_the_reader_sees_a_scalar_offset():
    good = ["_Zk:", "buffer_store_dword v0, v1, s[4:7], 0 offen offset:16", "buffer_store_dwordx4 v[0:3], off, s[4:7], 0 nt",
            "buffer_load_dwordx4 v[0:3], v1, s[4:7], 0 offen nt", "buffer_load_dword v1, s[0:3], 0 offen lds"]
    assert scalar_offsets(good) == ([], 4)
    assert len(scalar_offsets(good + ["buffer_store_dword v0, v1, s[4:7], s9 offen"])[0]) == 1
    assert len(scalar_offsets(["buffer_load_dword v0, v1, s[4:7], 16 offen"])[0]) == 1


def test_no_access_has_a_scalar_offset(tmp_path):
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    root = os.path.dirname(os.path.dirname(os.path.abspath(build.__file__)))
    include = ["-I", os.path.join(root, "include"), "-I", os.path.join(root, "paper_2010_00704_amd", "csrc")]

    def read(src):
        out = str(tmp_path / (os.path.basename(src) + ".s"))
        rc, log = build._run([build.HIPCC] + flags + ["--cuda-device-only", "-S"] + include + [src, "-o", out])
        assert rc == 0, log
        with open(out) as f:
            return scalar_offsets(f)

    with ThreadPoolExecutor(max_workers=8) as pool:
        results = list(pool.map(read, build.sources()))
    assert sum(seen for _, seen in results) > 10000
    found = [hit for hits, _ in results for hit in hits]
    assert not found, "%d accesses with a scalar offset, the first: %s" % (len(found), found[:5])
