"""The assembly of the kernels with the most live state, built here: no register move or spill stands between the
label where lanes that parted meet again and the instruction that turns them back on. The compiler has put moves
there in a gradient kernel whose lanes branched around a load: they ran for part of the lanes, the others kept a
stale address."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2110_11866_amd", "_build")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MOVE = re.compile(r"v_accvgpr_|v_mov_b|scratch_|buffer_")
OTHER = re.compile(r"v_readlane|v_writelane|s_")


def moves_before_exec(lines):
    """(kernel, moves) for every join whose exec restore follows moves."""
    kernel, block, joined, found = "", [], False, []
    for line in lines:
        t = line.split("//")[0].strip()
        if not t:
            continue
        label = re.match(r"(?:[0-9a-f]+ )?<(\S+)>:$", t)
        if label:
            kernel = label.group(1) if label.group(1).startswith("_Z") else kernel
            block, joined = [], True
        elif t.startswith("s_or_b64 exec, exec,"):
            if joined and all(MOVE.match(x) or OTHER.match(x) for x in block) and any(MOVE.match(x) for x in block):
                found.append((kernel, block))
            block, joined = [], False
        elif t.startswith(("s_branch", "s_cbranch", "s_endpgm", "s_setpc")) or "exec" in t.split(",")[0]:
            block, joined = [], False
        else:
            block.append(t)
    return found


def test_finds_moves():
    good = ["<_Zk>:", "s_cbranch_execz L1", "v_mov_b32_e32 v1, v2", "<L1>:", "s_or_b64 exec, exec, s[0:1]", "v_accvgpr_write_b32 a9, v1"]
    bad = ["<_Zk>:", "s_cbranch_execz L1", "v_mov_b32_e32 v1, v2", "<L1>:", "v_accvgpr_write_b32 a9, v1", "s_or_b64 exec, exec, s[0:1]"]
    assert moves_before_exec(good) == []
    assert moves_before_exec(bad) == [("_Zk", ["v_accvgpr_write_b32 a9, v1"])]


@pytest.mark.parametrize("name", ["scan_k%d_r%d" % (k, r) for k in (9, 12) for r in (4, 8, 16, 32)] + ["granule_scan", "carry_scan"])
def test_no_moves_before_exec(name, tmp_path):
    obj = os.path.join(BUILD, name + ".o")
    tools = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")]
    if not os.path.exists(obj) or any(shutil.which(t) is None for t in tools):
        pytest.skip("no built object or no LLVM tools")
    fat, code = str(tmp_path / "fat"), str(tmp_path / "code")
    subprocess.run([tools[0], "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], check=True)
    subprocess.run([tools[1], "--unbundle", "--type=o", "--input=" + fat, "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + code],
                   check=True)
    with subprocess.Popen([tools[2], "-d", "--no-show-raw-insn", "--symbolize-operands", code], stdout=subprocess.PIPE, text=True) as p:
        found = moves_before_exec(p.stdout)
    assert p.returncode == 0 and not found, [(k, b[:4]) for k, b in found[:4]]
