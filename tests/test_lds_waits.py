"""Every LDS access of the built kernels is waited for in front of the next block barrier (CPU only).

On gfx950 neither s_barrier nor the compiler waits for outstanding LDS accesses there: a barrier that hands LDS data to other
wavefronts, or gives up a buffer they will refill, needs a wait of its own, and a kernel without it gives the right values as
long as the accesses happen to be quick.  So no test of values shows that it lacks.  Here the instructions of the library built
from this tree are followed along all paths of control: LDS accesses complete in order, so s_waitcnt lgkmcnt(n) waits for one
behind which at least n others were issued."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2102_08481_amd", "libthia.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
OBJDUMP = shutil.which("llvm-objdump") or os.path.join(ROCM, "llvm", "bin", "llvm-objdump")

READS = ("ds_read", "ds_bpermute", "ds_permute", "ds_swizzle")   # the others write
NONE, MOST = 99, 15   # state: no access outstanding; lgkmcnt counts to 15


def kernels_of(listing):
    """(name, [(address, operation, operands, comment)]) of a disassembly."""
    name, code = None, []
    for line in listing.splitlines():
        head = re.match(r"^[0-9a-f]+ <(.+)>:$", line)
        if head:
            if code:
                yield name, code
            name, code = head.group(1), []
            continue
        ins = re.match(r"^\s+(\S+)(.*?)\s*//\s*([0-9A-F]+):(.*)$", line)
        if ins and name:
            code.append((int(ins.group(3), 16), ins.group(1), ins.group(2).strip(), ins.group(4)))
    if code:
        yield name, code


def unwaited_at_barriers(code, accesses):
    """Addresses of the barriers that an LDS access for which accesses(operation) holds can reach without having been waited
    for.  State in front of an instruction: how many LDS accesses at least were issued behind the newest such one."""
    index = {a: i for i, (a, *_) in enumerate(code)}
    state, todo, bad = {0: NONE}, [0], set()
    while todo:
        i = todo.pop()
        s = state[i]
        address, op, args, comment = code[i]
        following = [i + 1]
        if op == "s_barrier" and s != NONE:
            bad.add(hex(address))
        elif op == "s_waitcnt":
            count = re.search(r"lgkmcnt\((\d+)\)", args)
            if s != NONE and ((count and int(count.group(1)) <= s) or args in ("0", "0x0")):
                s = NONE
        elif op.startswith("ds_"):
            if accesses(op):
                s = 0
            elif s != NONE:
                s = min(s + 1, MOST)
        elif op == "s_endpgm":
            following = []
        elif op == "s_branch" or op.startswith("s_cbranch"):
            to = re.search(r"<.*?(?:\+0x([0-9a-f]+))?>$", comment)
            target = index[code[0][0] + int(to.group(1) or "0", 16)]
            following = [target] if op == "s_branch" else [i + 1, target]
        else:
            assert op not in ("s_setpc_b64", "s_swappc_b64", "s_call_b64"), (op, "calls are not followed")
        for j in following:
            if j < len(code) and (j not in state or s < state[j]):
                state[j] = s
                todo.append(j)
    return bad


def _code(*lines):
    return [(16 * i, l.split()[0], " ".join(l.split()[1:]), "") if "->" not in l else
            (16 * i, l.split()[0], "", " <k+0x%x>" % (16 * int(l.split("->")[1]))) for i, l in enumerate(lines)]


@pytest.mark.parametrize("lines,found", [
    (["ds_write_b64 v0", "s_barrier", "s_endpgm"], True),
    (["ds_write_b64 v0", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_endpgm"], False),
    (["ds_write_b64 v0", "s_waitcnt vmcnt(3)", "s_barrier", "s_endpgm"], True),
    (["ds_write_b64 v0", "ds_read_b64 v2", "s_waitcnt lgkmcnt(1)", "s_barrier", "s_endpgm"], False),   # one behind it may be out
    (["ds_read_b64 v2", "ds_write_b64 v0", "s_waitcnt lgkmcnt(1)", "s_barrier", "s_endpgm"], True),
    (["s_cbranch_scc1 ->2", "ds_write_b64 v0", "s_barrier", "s_endpgm"], True),                        # one of two paths
    (["s_barrier", "ds_write_b64 v0", "s_cbranch_scc1 ->0", "s_endpgm"], True),                        # around a loop
    (["s_branch ->2", "ds_write_b64 v0", "s_barrier", "s_endpgm"], False),                             # not reached
])
def test_the_paths_are_followed(lines, found):
    assert bool(unwaited_at_barriers(_code(*lines), lambda op: not op.startswith(READS))) == found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not installed")
def test_lds_accesses_are_waited_for_at_every_barrier(tmp_path):
    if not os.path.exists(LIB):
        from paper_2102_08481_amd import build
        build.build()
    shutil.copy(LIB, tmp_path / "libthia.so")
    subprocess.run([OBJDUMP, "--offloading", "libthia.so"], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    assert objects
    barriers, bad = 0, []
    for f in objects:
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for name, code in kernels_of(listing):
            barriers += sum(op == "s_barrier" for _, op, *_ in code)
            for what, accesses in (("write", lambda op: not op.startswith(READS)), ("read", lambda op: op.startswith(READS))):
                bad += [(name, what, at) for at in sorted(unwaited_at_barriers(code, accesses))]
    assert barriers > 500, "the listing was not understood"
    assert not bad, bad
