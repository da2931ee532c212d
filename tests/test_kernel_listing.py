"""The listing of the kernels built here: no register is copied, and none goes
to or comes from scratch, between the end of a branch's instructions and the
instruction that brings the other lanes back.  Under register pressure the
compiler has put copies of live registers there, for all lanes but run by the
branch's only, and the others went on with stale values.  A block made of
nothing but such copies is that form.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2407_18304_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LIB = os.path.join(build.PKG, "libmgrhd.so")
COPY = re.compile(r"v_mov_b(32|64)_e(32|64) v\S+, v|v_accvgpr_|scratch_(load|store)_")
SCALAR = re.compile(r"s_(?!or_b64 exec|\w*branch|endpgm|\w*saveexec|\w+ exec\b)|v_(read|write)lane")


def misplaced(lines):
    """(kernel, block) of every run of copies that an exec restore ends."""
    kernel, run, pure, found = None, [], False, []
    for line in lines:
        t = line.split("//")[0].strip()
        if not t:
            continue
        if t.endswith(">:"):
            name = t[t.rindex("<") + 1:-2]
            if not re.fullmatch(r"L\d+", name):
                kernel = name
            run, pure = [], True
        elif t.startswith("s_or_b64 exec, exec,"):
            if run and pure:
                found.append((kernel, run))
            run, pure = [], True
        elif COPY.match(t):
            run.append(t)
        elif "branch" in t:
            run, pure = [], True
        elif not SCALAR.match(t):
            pure = False
    return found


def test_the_form_is_found():
    listing = """
0000000000001000 <kernel>:
    v_add_f64 v[0:1], v[2:3], v[4:5] // 00
    s_and_saveexec_b64 s[10:11], vcc
    s_cbranch_execz L2
0000000000001010 <L1>:
    s_or_b64 exec, exec, s[16:17]
0000000000001020 <L2>:
    v_mov_b64_e32 v[66:67], v[80:81]
    v_mov_b32_e32 v17, v119
    s_mov_b64 s[6:7], s[98:99]
    s_or_b64 exec, exec, s[10:11]
""".split("\n")
    assert misplaced(listing) == [("kernel", ["v_mov_b64_e32 v[66:67], v[80:81]",
                                                   "v_mov_b32_e32 v17, v119"])]
    # the same copies behind the restore, and a branch that computes
    fine = [l for l in listing if "v_mov" not in l] + ["v_mul_f64 v[0:1], v[2:3], v[4:5]",
                                                            "v_mov_b32_e32 v1, v2",
                                                            "s_or_b64 exec, exec, s[2:3]"]
    assert misplaced(fine) == []


def test_no_copies_before_the_other_lanes_return(tmp_path):
    if not (os.path.exists(OBJDUMP) and os.path.exists(LIB)):
        pytest.skip("no built library, or no listing tool")
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True,
                   capture_output=True)
    objects = sorted(p for p in os.listdir(tmp_path) if "gfx950" in p)
    assert objects
    found = []
    for p in objects:
        proc = subprocess.Popen([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", p],
                                cwd=tmp_path, stdout=subprocess.PIPE, text=True)
        found += misplaced(proc.stdout)
        assert proc.wait() == 0
    assert found == []
