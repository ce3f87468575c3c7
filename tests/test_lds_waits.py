"""LDS reads around the barriers of kernels that fill LDS with direct loads.

A barrier does not wait for a wave's LDS reads, and after it another wave's
direct global->LDS load may overwrite what they read. In the built library's
gfx950 code, on every path, each LDS read of such a kernel therefore has to be
waited for (lgkmcnt) before the next s_barrier; LDS answers in order, so a
wait for n leaves at most the last n reads outstanding."""
import os
import re
import subprocess

import pytest

from paper_2507_01021_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\t(\S+)(.*?)\s*// ([0-9A-F]+):(.*)$")
LGKM = re.compile(r"lgkmcnt\((\d+)\)")


def functions(tmp_path):
    lib = tmp_path / "lib.so"
    lib.symlink_to(binding.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in sorted(tmp_path.iterdir()):
        if "gfx950" not in f.name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], check=True, capture_output=True,
                              text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"^([0-9a-f]+) <(.*)>:$", line)
            if m:
                name, base = m.group(2), int(m.group(1), 16)
                out[name] = []
                continue
            m = LINE.match(line)
            if m and name:
                target = re.search(r"<" + re.escape(name) + r"(?:\+0x([0-9a-f]+))?>", m.group(4))
                out[name].append((int(m.group(3), 16), m.group(1), m.group(2),
                                  base + int(target.group(1) or "0", 16) if target else None))
    return out


def unwaited(code, crossings=0):
    """Addresses of the barriers that some path reaches with an LDS read
    outstanding that has already crossed `crossings` barriers."""
    index = {a: i for i, (a, *_) in enumerate(code)}
    seen = [set() for _ in code]  # outstanding reads before the instruction: barriers crossed, oldest first
    work = [(0, ())]
    bad = set()
    while work:
        i, s = work.pop()
        if s in seen[i]:
            continue
        seen[i].add(s)
        assert len(seen[i]) < 1000
        _, op, args, target = code[i]
        if re.match(r"ds_(read|load)", op):
            s = (s + (0,))[-16:]
        elif op == "s_waitcnt" and LGKM.search(args):
            n = int(LGKM.search(args).group(1))
            s = s[len(s) - n:] if n < len(s) else s
        elif op == "s_barrier":
            if any(c >= crossings for c in s):
                bad.add(code[i][0])
            s = tuple(min(c + 1, crossings) for c in s)
        if op.startswith("s_cbranch") or op == "s_branch":
            assert target in index, (op, args)
            work.append((index[target], s))
        if op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
            work.append((i + 1, s))
    return bad


def test_reads_are_waited_for_before_barriers(tmp_path):
    if not os.path.exists(binding.LIB_PATH) or not os.path.exists(OBJDUMP):
        pytest.skip("library not built, or no disassembler")
    direct = {n: c for n, c in functions(tmp_path).items() if any("load_lds" in op for _, op, *_ in c)}
    for kind in ("gemm_bf16_kernel", "gemm_bf16_h_kernel", "gemm_tile_kernelINS_4bf16", "gemm_tile_kernelIf",
                 "enc_attn_bf16_kernel", "enc_attn_f32_kernel"):
        assert any(kind in n for n in direct), kind
    for n, c in direct.items():
        # the 256 x 256 kernel's two wave groups refill a buffer two barriers after its reads
        bad = unwaited(c, 1 if "gemm_bf16_kernel" in n else 0)
        assert not bad, (n, [hex(a) for a in sorted(bad)])


def test_analysis_sees_an_unwaited_read():
    code = [(0, "ds_read_b128", " v[0:3], v4", None), (4, "s_barrier", "", None), (8, "s_endpgm", "", None)]
    assert unwaited(code) == {4}
    code.insert(1, (2, "s_waitcnt", " lgkmcnt(0)", None))
    assert not unwaited(code)
    # a read at a loop's end, waited for only after the barrier at its head
    loop = [(0, "s_barrier", "", None), (4, "s_waitcnt", " lgkmcnt(0)", None), (8, "ds_read_b128", " v[0:3], v4", None),
            (12, "s_cbranch_scc1", " 0", 0), (16, "s_endpgm", "", None)]
    assert unwaited(loop) == {0}
    # outstanding across one barrier, waited for before the second
    two = [(0, "ds_read_b128", " v[0:3], v4", None), (4, "s_barrier", "", None), (8, "s_waitcnt", " lgkmcnt(0)", None),
           (12, "s_barrier", "", None), (16, "s_endpgm", "", None)]
    assert unwaited(two) == {4} and not unwaited(two, 1)
    del two[2]
    assert unwaited(two, 1) == {12}
